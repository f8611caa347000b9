// Pass B of the local backward: the carried adjoint, walked back through a unit's
// chunks with the fp32 adjoint in registers.
//
// The walk of one unit is cut by hidden unit into slices of HS = 128 columns, one
// workgroup of 8 waves each: wave w of slice s owns hidden columns
// [128 s + 16 w, + 16) of W1bar, S1bar, W2bar, S2bar, held as 16 x 16 MFMA tiles
// (rows d, column hidden: W1bar^T, S1bar^T, W2bar, S2bar).  Of a chunk's quantities
// only Rbar (and the outputs dk and the gate row sums, which nothing in the walk
// reads) contract over the hidden units, so the slices meet once per chunk:
//
//   T3 = D1 W1bar', T4 = D1 S1bar', T5 = Hk W2bar'^T, T6 = Hk S2bar'^T   (from bf16
//       copies of the slice's adjoint in LDS), the adjoint . state products, the gate
//       row sums -K.T3 - R.T5 and -K.T4 - R.T6
//   D1bar = -Pz^T Zbar - cC K W1bar'^T - b K S1bar'^T -> Gbar = D1bar s'(Zk),
//   Hkbar = -Q1^T H - cC R W2bar' - b R S2bar'   (the wave's own columns, the adjoint
//       tiles taken as MFMA operands from the registers)
//   Rbar = -Po^T dO - cC T5 - b T6 + Gbar W2^T   the slice's part, exchanged;
//       meanwhile the adjoint update's terms that do not need it
//   Ykbar = (2/d) Rbar (dv = -Ykbar), Zkbar = (Hkbar + Ykbar W2) s'(Zk) + D1bar G s''(Zk),
//       the rest of the update, the LDS copies of the new adjoint
//   dk = -cC T3 - b T4 + Zkbar W1                the slice's part, summed by pass C.
//
// Exchange: every partial sum travels with its tag in one 8-byte word (agent-scope
// relaxed atomics), so a word that carries the chunk's tag is the whole message: no
// fence, no flag, one trip.  Two buffers in turn: a slice that publishes a chunk has
// received the others' chunk before it, which they sent after they had read the one
// before that, the last in the same buffer.
// Pass A clears the tags in every call.
//
// A workgroup learns its slice from a counter of the workgroups that have started (eight
// counters, by residue of the block index; pass A clears them, too).  Those that have
// started are therefore whole groups and at most one slice more per counter, in whatever
// order the device starts them and whatever else runs there: a whole group waits for
// nobody outside it, and the next workgroup to start on a place that it leaves completes
// a pair.  The grid is never larger than the CUs (groups of slices take several units in
// turn).  The wait ends after WAIT_ROUNDS in any case; the gradients are NaN then.
//
// Bound by latency (one memory round trip, four barriers and one exchange a chunk).
// Chunks of up to 32 rows: 10.8 us a chunk at 16 rows (32 units of 512 chunks), where
// the walk on one CU per unit with the adjoint in memory took 36.  The 32-row instance
// already spills 66 to 71 of its vector registers; at 64 rows the tiles do not fit beside
// the adjoint at all, and that walk stays.
#include "tnt_local_bwd_helpers.h"
#include "tnt_local_bwd_split.h"
#include "tnt_regtile.h"

#include <algorithm>

namespace tnt {

using namespace bwdh;

namespace {

constexpr int WAIT_ROUNDS = 1 << 25;  // a poll takes about a microsecond

template <int D, int H, int CP>
struct BWalk {
  static constexpr int HS = rec::walk_hs(H), G = rec::walk_slices(CP, H);
  static_assert(G == 2, "two slices a unit: each has one other to wait for");
  static constexpr int NW = HS / 16, NT = NW * WAVE;
  static constexpr int DT = D / 16, TM = CP / 16;
  static constexpr int NCI = (CP + 31) / 32;  // K steps of a contraction over the chunk
  // LDS, bf16 elements.  Rows read 8 bytes a lane are padded by 8 bytes, rows read
  // 16 bytes a lane by 16.
  static constexpr int LK = D + 4, LC4 = CP + 4, LC8 = CP + 8, LD8 = D + 8, LH = HS + 8;
  static constexpr int cmax(int x, int y) { return x > y ? x : y; }
  // region A: the operands of the slice's own columns; then K^T, Ykbar, Ykbar^T
  static constexpr int PzT = 0, Q1T = PzT + CP * LC8, K = Q1T + CP * LC8, R = K + CP * LK;
  static constexpr int endA1 = R + CP * LK;
  static constexpr int Yk = 0, YkT = Yk + CP * LD8, KT = YkT + D * LC8, endA2 = KT + D * LC4;
  // dO^T and, scaled by A_i and by E_i, X^T and dO^T
  static constexpr int dOT = (cmax(endA1, endA2) + 7) / 8 * 8;
  static constexpr int XAT = dOT + D * LC8, XET = XAT + D * LC8, dOAT = XET + D * LC8,
                       dOET = dOAT + D * LC8, RT = dOET + D * LC8;
  static constexpr int adj = (RT + D * LC4 + 7) / 8 * 8;  // W1bar^T, S1bar^T, W2bar, S2bar [D][LH]
  static constexpr int sG = adj + 4 * D * LH;             // Gbar, then Zkbar [CP][LH]
  static constexpr int total = sG + CP * LH;
  static_assert(Q1T % 8 == 0 && YkT % 8 == 0 && K % 4 == 0 && R % 4 == 0 && KT % 4 == 0 &&
                    XAT % 8 == 0 && RT % 4 == 0 && sG % 8 == 0,
                "aligned rows");
  static_assert(2 * DT <= NW && D % 32 == 0, "a wave per column strip of T3, T4 and of T5, T6");
  static_assert(CP * CP / 8 <= NT && CP * D / 8 <= NT && 2 * CP <= NT, "one vector per thread");
};

// 16 bytes of a row at contraction offset k0 + 8 g, zero past K
template <int K>
__device__ __forceinline__ bf16x8 frag16(const __bf16* row, int k0, int g) {
  if (K % 32 == 0 || k0 + 8 * g < K) return *reinterpret_cast<const bf16x8*>(row + k0 + 8 * g);
  bf16x8 z;
#pragma unroll
  for (int j = 0; j < 8; ++j) z[j] = (__bf16)0.f;
  return z;
}

// The thread's index through an opaque move, as lane_id_local: no address made from
// it is hoisted out of the chunk loop or kept from one phase to the next.
__device__ __forceinline__ int tid_local() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}
struct Lane {
  int l, g, lc;
  __device__ __forceinline__ Lane() : l(lane_id_local()), g(l >> 4), lc(l & 15) {}
};

// a vector at a 32-bit element offset from a wave-uniform base (scalar base, one
// address register per load)
template <typename V>
__device__ __forceinline__ V at(const __bf16* base, uint32_t e) {
  return *reinterpret_cast<const V*>(reinterpret_cast<const char*>(base) + e * 2u);
}
template <int K>
__device__ __forceinline__ bf16x8 gfrag(const __bf16* base, uint32_t row, int k0, int g) {
  if (K % 32 == 0 || k0 + 8 * g < K) return at<bf16x8>(base, row + k0 + 8 * g);
  bf16x8 z;
#pragma unroll
  for (int j = 0; j < 8; ++j) z[j] = (__bf16)0.f;
  return z;
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
  return x + __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}
// sum over the 16 lanes of a row: quads, then mirrors of 8 and 16 lanes
__device__ __forceinline__ float row_sum16(float x) {
  x = dpp_add<0xB1>(x);
  x = dpp_add<0x4E>(x);
  x = dpp_add<0x141>(x);
  return dpp_add<0x140>(x);
}

}  // namespace

// LO: the adjoint . state products in fp32, from the registers and the two state copies
template <int D, int H, int CP, bool LO>
__global__ void __launch_bounds__((BWalk<D, H, CP>::NT)) local_bwd_walk_kernel(LocalBwdArgs a, SplitPtrs P) {
  using CT = __bf16;
  using B = BWalk<D, H, CP>;
  constexpr int HS = B::HS, G = B::G, NW = B::NW, NT = B::NT, DT = B::DT, TM = B::TM, NCI = B::NCI;
  constexpr int LK = B::LK, LC4 = B::LC4, LC8 = B::LC8, LD8 = B::LD8, LH = B::LH;
  constexpr size_t hd = (size_t)H * D;
  constexpr rec::RecLayout RL = rec::make_rec_layout(CP, D, H);
  extern __shared__ __align__(16) unsigned char smem[];
  __shared__ __align__(16) float sC[CP], sB[CP];
  __shared__ int role;
  __shared__ float sc3[4], dpart[3][NW], pC[2 * DT][CP], pB[2 * DT][CP];
  CT* const L = reinterpret_cast<CT*>(smem);
  CT *sPzT = L + B::PzT, *sQ1T = L + B::Q1T, *sK = L + B::K, *sR = L + B::R, *sYk = L + B::Yk,
     *sYkT = L + B::YkT, *sKT = L + B::KT, *sdOT = L + B::dOT, *sXAT = L + B::XAT, *sXET = L + B::XET, *sdOAT = L + B::dOAT,
     *sdOET = L + B::dOET, *sRT = L + B::RT,
     *sAdj = L + B::adj, *sGz = L + B::sG;

  // this workgroup's group and slice, by the order in which those of its residue modulo
  // WALK_LANES have started (one counter for all of them: 1135 us for 1120 at B 2, H 4, L 2048)
  if (threadIdx.x == 0) {
    const int lane8 = (int)blockIdx.x % WALK_LANES, part = P.n0 + P.nc == a.D.S / a.D.C ? 0 : 1;
    role = (int)__hip_atomic_fetch_add(P.tickets + (part * WALK_LANES + lane8) * TICKET_STRIDE, 1u,
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) * WALK_LANES + lane8;
  }
  __syncthreads();
  const int place = __builtin_amdgcn_readfirstlane(role);
  const int blk = place / (WALK_LANES * G), rem = place % (WALK_LANES * G);
  const int sl = rem / WALK_LANES, grp = blk * WALK_LANES + rem % WALK_LANES;
  if (grp >= P.groups) return;  // (every slice of the group)
  const Dims Dm = a.D;
  const int C = Dm.C, nshard = Dm.L / Dm.S, nch = Dm.S / C;
  const int w = wave_id_uniform();
  const int h0 = sl * HS;                    // the slice's first hidden column
  const int pair = w / DT, strip = w % DT;   // column strip of T3, T4 (0) or T5, T6 (1)
  const float rscale = 2.0f / (float)D;
  unsigned long long* const xg = P.xch + (size_t)grp * 2 * G * CP * D;

  f4 w1[DT], s1[DT], w2[DT], s2[DT];  // the adjoint: rows 16 dt + 4 g + r, column h0 + 16 w + lc
  // bf16 copies of the adjoint in LDS, [D][LH]
  auto write_copies = [&]() {
    const int l = lane_id_local(), g = l >> 4, lc = l & 15, q = lc & 3;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      CT* p = sAdj + (16 * dt + 4 * g + q) * LH + 16 * w + lc - q;
      *reinterpret_cast<bf16x4*>(p) = cvt4(quad_transpose(w1[dt]));
      *reinterpret_cast<bf16x4*>(p + D * LH) = cvt4(quad_transpose(s1[dt]));
      *reinterpret_cast<bf16x4*>(p + 2 * D * LH) = cvt4(quad_transpose(w2[dt]));
      *reinterpret_cast<bf16x4*>(p + 3 * D * LH) = cvt4(quad_transpose(s2[dt]));
    }
  };
  auto put_dots = [&](float pa, float pe, float pb) {  // summed after the chunk's first barrier
    pa = wave_sum(pa);
    pe = wave_sum(pe);
    pb = wave_sum(pb);
    if (lane_id_local() == 0) {
      dpart[0][w] = pa;
      dpart[1][w] = pe;
      dpart[2][w] = pb;
    }
  };
  // LO: a chunk's adjoint . state products, taken at the end of the chunk before (in the
  // order of the walk), where the adjoint is final and few registers are in use (beside
  // the chunk's first products, or requested ahead of the last barrier, they spilled 80
  // registers at 16 rows; here none).  The state at the lane's adjoint
  // tiles: copy and remainder of W1, S1 (by rows, transposed within the quad) and W2, S2.
  struct StatePairs {
    bf16x4 v[LO ? 4 : 1][DT];
    rem2 r[LO ? 2 : 1][DT];
  };
  auto load_pairs = [&](int u, int n, StatePairs& L) {
    const size_t slot = (size_t)u * a.nslots + n;
    const CT* hi = launder_global((const CT*)a.statesT + slot * (4 * hd + (size_t)D * D));
    const rem2* lo = launder_global((const rem2*)a.statesLo + slot * (hd / 2));
    const Lane y;
    const int q = y.lc & 3, h = h0 + 16 * w + y.lc;
#pragma unroll
    for (int m = 0; m < (LO ? 4 : 0); ++m)  // W1, W2, S1, S2
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const uint32_t e = m % 2 ? h * D + 16 * dt + 4 * y.g : (16 * dt + 4 * y.g + q) * H + h - q;
        L.v[m][dt] = at<bf16x4>(hi + m * hd, e);
        if (m < 2) L.r[m][dt] = lo[m * hd / 4 + rem_ofs(DT, dt, h0 / 16 + w, m ? y.l : rem_lane1(y.l))];
      }
  };
  auto exact_dots = [&](const StatePairs& L) {
    float pa = 0.f, pe = 0.f, pb = 0.f;
    auto value = [&](int m, int dt) {
      const f4 x = rem_unpack(L.v[m][dt], L.r[m % 2][dt][m / 2]);
      return m % 2 ? x : quad_transpose(x);
    };
#pragma unroll
    for (int m = 0; m < (LO ? 2 : 0); ++m)
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const f4 y0 = value(m, dt), y1 = value(m + 2, dt), x0 = m ? w2[dt] : w1[dt], x1 = m ? s2[dt] : s1[dt];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          pa += x0[r] * y0[r];
          pe += x0[r] * y1[r];
          pb += x1[r] * y1[r];
        }
      }
    put_dots(pa, pe, pb);
  };
  // a chunk's shared operands and coefficients, one vector of each per thread
  struct Stage {
    bf16x8 pz, q1, k, r, rt;
    float cf, sc;
  };
  auto prefetch = [&](size_t t, Stage& S) {
    const CT* rc = launder_global((const CT*)a.frec + t * RL.fc.n);
    const CT* bq = launder_global((const CT*)P.brec + t * RL.bc.n);
    const float* rf = launder_global(a.frec_f + t * RL.ff.n);
    const int tid = tid_local();
    if (tid < CP * CP / 8) {
      S.pz = *reinterpret_cast<const bf16x8*>(rc + RL.fc.o[rec::PzT] + 8 * tid);
      S.q1 = *reinterpret_cast<const bf16x8*>(bq + RL.bc.o[rec::Q1T] + 8 * tid);
    }
    if (tid < CP * D / 8) {
      S.k = *reinterpret_cast<const bf16x8*>(rc + RL.fc.o[rec::K] + 8 * tid);
      S.r = *reinterpret_cast<const bf16x8*>(rc + RL.fc.o[rec::R] + 8 * tid);
      S.rt = *reinterpret_cast<const bf16x8*>(rc + RL.fc.o[rec::RT] + 8 * tid);
    }
    if (tid < 2 * CP) S.cf = rf[(tid < CP ? RL.ff.o[rec::cC] : RL.ff.o[rec::bb]) + tid % CP];
    if (tid < 3) S.sc = rf[RL.ff.o[rec::sc] + tid];
  };
  auto put8 = [](CT* p, const bf16x8& v) {  // rows that are only 8-byte aligned
    *reinterpret_cast<bf16x4*>(p) = bf16x4{v[0], v[1], v[2], v[3]};
    *reinterpret_cast<bf16x4*>(p + 4) = bf16x4{v[4], v[5], v[6], v[7]};
  };
  auto stage = [&](const Stage& S) {
    const int tid = tid_local(), e = 8 * tid;
    if (tid < CP * CP / 8) {
      const int i = e / CP, c = e % CP;
      *reinterpret_cast<bf16x8*>(sPzT + i * LC8 + c) = S.pz;
      *reinterpret_cast<bf16x8*>(sQ1T + i * LC8 + c) = S.q1;
    }
    if (tid < CP * D / 8) {
      const int i = e / D, c = e % D, j = e / CP, ct = e % CP;
      put8(sK + i * LK + c, S.k);
      put8(sR + i * LK + c, S.r);
      put8(sRT + j * LC4 + ct, S.rt);
    }
    if (tid < 2 * CP) (tid < CP ? sC : sB)[tid % CP] = S.cf;
    if (tid < 3) sc3[tid] = S.sc;
  };
  // Ykbar = (2/d) Rbar of tile (it, strip) into LDS, row-wise and transposed; dv = -Ykbar
  auto put_y = [&](int it, const f4& rb, float* dvp) {
    const int l = lane_id_local(), g = l >> 4, lc = l & 15, q = lc & 3;
    const int i = 16 * it + 4 * g, j = 16 * strip + lc;
    f4 y;
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = i + r < C ? rscale * rb[r] : 0.f;
    const f4 yt = quad_transpose(y);
    *reinterpret_cast<bf16x4*>(sYk + (i + q) * LD8 + j - q) = cvt4(yt);
    *reinterpret_cast<bf16x4*>(sYkT + j * LC8 + i) = cvt4(y);
    if (sl == 0 && i + q < C)
      *reinterpret_cast<f32x4*>(dvp + (size_t)(i + q) * D + j - q) = f32x4{-yt[0], -yt[1], -yt[2], -yt[3]};
  };

  unsigned tag0 = 0;   // tags of this unit's chunks: tag0 + n + 1
  unsigned turn = 0;   // chunks walked by this launch: the exchange buffers in turn
  bool lost = false;   // a wait ran out: later ones are skipped
  for (int u = grp; u < P.units; u += P.groups, tag0 += nch) {
    const int b = u / (Dm.H * nshard), hh = (u / nshard) % Dm.H, s = u % nshard;
    const size_t cbase = ((size_t)b * Dm.H + hh) * Dm.L;
    float* const adj0 = a.adj + (size_t)u * 4 * hd;
    const int nlast = P.n0 + P.nc - 1;
    {
      const int l = lane_id(), g = l >> 4, lc = l & 15, h = h0 + 16 * w + lc;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        w1[dt] = s1[dt] = w2[dt] = s2[dt] = zero4();
        if (nlast != nch - 1) {  // the adjoint that the launch for the later chunks left
          const int d0 = 16 * dt + 4 * g;
          w1[dt] = *reinterpret_cast<const f32x4*>(adj0 + (size_t)h * D + d0);
          s1[dt] = *reinterpret_cast<const f32x4*>(adj0 + 2 * hd + (size_t)h * D + d0);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            w2[dt][r] = adj0[hd + (size_t)(d0 + r) * H + h];
            s2[dt][r] = adj0[3 * hd + (size_t)(d0 + r) * H + h];
          }
        }
      }
    }
    write_copies();
    if constexpr (LO) {
      StatePairs L;
      load_pairs(u, nlast, L);
      exact_dots(L);
    }
    __syncthreads();

    for (int n = nlast; n >= P.n0; --n, ++turn) {
      const size_t t = (size_t)u * nch + n;
      const int tok0 = s * Dm.S + n * C;
      const CT* rc = launder_global((const CT*)a.frec + t * RL.fc.n);
      const CT* bq = launder_global((const CT*)P.brec + t * RL.bc.n);
      float* bqf = launder_global(P.brec_f + t * RL.bf.n);
      const CT* pk = launder_global((const CT*)a.statesT + ((size_t)u * a.nslots + n) * (4 * hd + (size_t)D * D));
      const CT *W1T = pk, *W2T = pk + hd, *S1T = pk + 2 * hd, *S2T = pk + 3 * hd;
      const int hw = h0 + 16 * w;  // the wave's first hidden column

      // ---- T3, T4 (D1 with W1bar', S1bar') or T5, T6 (Hk with W2bar', S2bar') on the wave's
      // strip, and the adjoint . state products (W1bar, S1bar from their LDS copies, W2bar,
      // S2bar from the registers, the state from its compute-type copies; LO: done already).
      // Every load of the phase is requested ahead of the first product: one memory round
      // trip.
      f4 t0[TM], t1[TM];
#pragma unroll
      for (int it = 0; it < TM; ++it) t0[it] = t1[it] = zero4();
      bf16x4 mx[TM];           // K or R at the strip's tiles (row sums)
      bf16x8 zb[NCI], ht[NCI];  // the own columns of Zbar and H
      {
        const Lane y;
        const int tid = tid_local(), l = y.l, g = y.g, lc = y.lc, hrow = hw + lc;
        constexpr int NKH = HS / 32, KG = NKH / 2;
        const CT* Ar = rc + RL.fc.o[pair ? rec::Hk : rec::D1] + h0;
        bf16x8 fa[KG][TM];
        auto load_fa = [&](int k0) {
#pragma unroll
          for (int ks = 0; ks < KG; ++ks)
#pragma unroll
            for (int it = 0; it < TM; ++it) fa[ks][it] = gfrag<HS>(Ar, (16 * it + lc) * H, 32 * (k0 + ks), g);
        };
        if (pair < 2) {
          load_fa(0);
          const CT* MT = rc + RL.fc.o[pair ? rec::RT : rec::KT];
#pragma unroll
          for (int it = 0; it < TM; ++it) mx[it] = at<bf16x4>(MT, (16 * strip + lc) * CP + 4 * g + 16 * it);
        }
        constexpr int IT = D * HS / 8 / NT;
        static_assert(D * HS / 8 % NT == 0, "whole vectors per thread");
        bf16x8 y0[IT], y1[IT];
        bf16x4 v0[DT], v1[DT];
        if constexpr (!LO) {
#pragma unroll
          for (int p = 0; p < IT; ++p) {
            const int v = tid + p * NT, j = v / (HS / 8), c = 8 * (v % (HS / 8));
            y0[p] = at<bf16x8>(W1T, j * H + h0 + c);
            y1[p] = at<bf16x8>(S1T, j * H + h0 + c);
          }
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            v0[dt] = at<bf16x4>(W2T, hrow * D + 16 * dt + 4 * g);
            v1[dt] = at<bf16x4>(S2T, hrow * D + 16 * dt + 4 * g);
          }
        }
        Stage S;
        prefetch(t, S);
#pragma unroll
        for (int c = 0; c < NCI; ++c) {
          zb[c] = gfrag<CP>(bq + RL.bc.o[rec::ZbT], hrow * CP, 32 * c, g);
          ht[c] = gfrag<CP>(rc + RL.fc.o[rec::HT], hrow * CP, 32 * c, g);
        }
        if (pair < 2) {
          const CT* Bc = sAdj + (pair ? 2 * D * LH : 0) + (16 * strip + lc) * LH;
#pragma unroll
          for (int k0 = 0; k0 < NKH; k0 += KG) {
#pragma unroll
            for (int ks = 0; ks < KG; ++ks) {
              const bf16x8 b0 = frag16<HS>(Bc, 32 * (k0 + ks), g), b1 = frag16<HS>(Bc + D * LH, 32 * (k0 + ks), g);
#pragma unroll
              for (int it = 0; it < TM; ++it) {
                mma32(t0[it], fa[ks][it], b0);
                mma32(t1[it], fa[ks][it], b1);
              }
            }
            if (k0 + KG < NKH) load_fa(k0 + KG);
          }
        }
        if constexpr (!LO) {
          float pa = 0.f, pe = 0.f, pb = 0.f;
#pragma unroll
          for (int p = 0; p < IT; ++p) {
            const int v = tid + p * NT, j = v / (HS / 8), c = 8 * (v % (HS / 8));
            const bf16x8 x0 = *reinterpret_cast<const bf16x8*>(sAdj + j * LH + c);
            const bf16x8 x1 = *reinterpret_cast<const bf16x8*>(sAdj + D * LH + j * LH + c);
#pragma unroll
            for (int q = 0; q < 8; ++q) {
              pa += (float)x0[q] * (float)y0[p][q];
              pe += (float)x0[q] * (float)y1[p][q];
              pb += (float)x1[q] * (float)y1[p][q];
            }
          }
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              pa += w2[dt][r] * (float)v0[dt][r];
              pe += w2[dt][r] * (float)v1[dt][r];
              pb += s2[dt][r] * (float)v1[dt][r];
            }
          put_dots(pa, pe, pb);
        }
        stage(S);
      }
      // s'(Zk), G, s''(Zk) of the own columns, requested ahead of the barrier
      bf16x4 spv[TM], gg[TM], spp[TM];
#pragma unroll
      for (int it = 0; it < TM; ++it) {
        const uint32_t fo = (uint32_t)frag_ofs<CP, H>(16 * it, hw, lane_id_local());
        spv[it] = at<bf16x4>(rc + RL.fc.o[rec::Sp], fo);
        gg[it] = at<bf16x4>(rc + RL.fc.o[rec::G], fo);
        spp[it] = at<bf16x4>(rc + RL.fc.o[rec::Spp], fo);
      }
      __syncthreads();  // the chunk's operands and coefficients are in LDS

      // ---- the strip's row sums and -cC T - b T'
      f4 kr[TM];
      if (pair < 2) {
        const Lane y;
        const int g = y.g, lc = y.lc;
#pragma unroll
        for (int it = 0; it < TM; ++it) {
          const int i = 16 * it + 4 * g;
          const f4 cc = *reinterpret_cast<const f4*>(sC + i), cb = *reinterpret_cast<const f4*>(sB + i);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float m = (float)mx[it][r];
            const float x0 = row_sum16(m * t0[it][r]), x1 = row_sum16(m * t1[it][r]);
            if (lc == 0) {
              pC[w][i + r] = x0;
              pB[w][i + r] = x1;
            }
            kr[it][r] = -cc[r] * t0[it][r] - cb[r] * t1[it][r];
          }
        }
      }
      if (const int tid = tid_local(); tid < 3) {
        float x = 0.f;
#pragma unroll
        for (int v = 0; v < NW; ++v) x += dpart[tid][v];
        bqf[RL.bf.o[rec::dots] + 4 * sl + tid] = x;
      }

      // ---- the wave's own columns: D1bar -> Gbar, the Zkbar terms known now
      bf16x4 gb[TM];
      f4 zkp[TM];
      bf16x8 kt;  // K^T of the chunk, into LDS once region A is dead
      bf16x8 xa, xe, da, de, dO;  // X^T and dO^T (scaled), into LDS before the next barrier
      if (const int tid = tid_local(); tid < CP * D / 8) {
        kt = at<bf16x8>(rc + RL.fc.o[rec::KT], 8 * tid);
        xa = at<bf16x8>(rc + RL.fc.o[rec::XAT], 8 * tid);
        xe = at<bf16x8>(rc + RL.fc.o[rec::XET], 8 * tid);
        da = at<bf16x8>(bq + RL.bc.o[rec::dOAT], 8 * tid);
        de = at<bf16x8>(bq + RL.bc.o[rec::dOET], 8 * tid);
        if (sl == 0) dO = at<bf16x8>(bq + RL.bc.o[rec::dOT], 8 * tid);
      }
      {
        const Lane y;
        const int g = y.g, lc = y.lc;
        bf16x8 bw[DT / 2], bs[DT / 2];
#pragma unroll
        for (int c = 0; c < DT / 2; ++c) {
          bw[c] = join(cvt4(w1[2 * c]), cvt4(w1[2 * c + 1]));
          bs[c] = join(cvt4(s1[2 * c]), cvt4(s1[2 * c + 1]));
        }
#pragma unroll
        for (int it = 0; it < TM; ++it) {
          const int row = 16 * it + lc, i = 16 * it + 4 * g;
          f4 ap = zero4(), k1 = zero4(), k2 = zero4();
#pragma unroll
          for (int c = 0; c < DT / 2; ++c) {
            const bf16x8 ak = a_pair(sK, LK, row, 32 * c, g);
            mma32(k1, ak, bw[c]);
            mma32(k2, ak, bs[c]);
          }
#pragma unroll
          for (int c = 0; c < NCI; ++c) mma32(ap, frag16<CP>(sPzT + row * LC8, 32 * c, g), zb[c]);
          const f4 cc = *reinterpret_cast<const f4*>(sC + i), cb = *reinterpret_cast<const f4*>(sB + i);
          f4 gv;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float d1b = -ap[r] - cc[r] * k1[r] - cb[r] * k2[r];
            gv[r] = d1b * (float)spv[it][r];
            zkp[it][r] = d1b * (float)gg[it][r] * (float)spp[it][r];
          }
          gb[it] = cvt4(gv);
          const int q = lc & 3;
          *reinterpret_cast<bf16x4*>(sGz + (i + q) * LH + 16 * w + lc - q) = cvt4(quad_transpose(gv));
        }
#pragma unroll
        for (int c = 0; c < DT / 2; ++c) {
          bw[c] = join(cvt4(w2[2 * c]), cvt4(w2[2 * c + 1]));
          bs[c] = join(cvt4(s2[2 * c]), cvt4(s2[2 * c + 1]));
        }
#pragma unroll
        for (int it = 0; it < TM; ++it) {
          const int row = 16 * it + lc, i = 16 * it + 4 * g;
          f4 aq = zero4(), r1 = zero4(), r2 = zero4();
#pragma unroll
          for (int c = 0; c < DT / 2; ++c) {
            const bf16x8 ar = a_pair(sR, LK, row, 32 * c, g);
            mma32(r1, ar, bw[c]);
            mma32(r2, ar, bs[c]);
          }
#pragma unroll
          for (int c = 0; c < NCI; ++c) mma32(aq, frag16<CP>(sQ1T + row * LC8, 32 * c, g), ht[c]);
          const f4 cc = *reinterpret_cast<const f4*>(sC + i), cb = *reinterpret_cast<const f4*>(sB + i);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            zkp[it][r] += (-aq[r] - cc[r] * r1[r] - cb[r] * r2[r]) * (float)spv[it][r];
        }
      }
      bf16x8 wf[HS / 32];  // W2 rows (T5, T6 waves) for Gbar W2^T; W1^T rows (T3, T4) for Zkbar W1
      auto load_wf = [&](const CT* p) {
        const int l = lane_id_local();
#pragma unroll
        for (int ks = 0; ks < HS / 32; ++ks) wf[ks] = gfrag<HS>(p + h0, (16 * strip + (l & 15)) * H, 32 * ks, l >> 4);
      };
      if (pair == 1) load_wf(rc + RL.fc.o[rec::W2r]);
      if (const int t8 = 8 * tid_local(); t8 < CP * D) {
        const int e = (t8 / CP) * LC8 + t8 % CP;
        *reinterpret_cast<bf16x8*>(sXAT + e) = xa;
        *reinterpret_cast<bf16x8*>(sXET + e) = xe;
        *reinterpret_cast<bf16x8*>(sdOAT + e) = da;
        *reinterpret_cast<bf16x8*>(sdOET + e) = de;
        if (sl == 0) *reinterpret_cast<bf16x8*>(sdOT + e) = dO;
      }
      __syncthreads();  // Gbar, X^T and dO^T complete; region A is dead

      const int tid = tid_local();
      if (tid < CP * D / 8) put8(sKT + (8 * tid / CP) * LC4 + 8 * tid % CP, kt);
      if (tid < CP) {  // gate row sums of the slice, fixed order
        float x = 0.f, y = 0.f;
#pragma unroll
        for (int v = 0; v < 2 * DT; ++v) {
          x += pC[v][tid];
          y += pB[v][tid];
        }
        bqf[RL.bf.o[rec::gCC] + CP * sl + tid] = -x;
        bqf[RL.bf.o[rec::gB] + CP * sl + tid] = -y;
      }
      const unsigned tag = tag0 + (unsigned)n + 1;
      unsigned long long* const xb = xg + (size_t)(turn & 1) * G * CP * D;
      float* const dvp = a.dv_part + (cbase + tok0) * D;
      // ---- the slice's part of Rbar
      if (pair == 1) {
        const Lane y;
        const int g = y.g, lc = y.lc;
#pragma unroll
        for (int it = 0; it < TM; ++it) {
          f4 acc = zero4();
#pragma unroll
          for (int ks = 0; ks < HS / 32; ++ks)
            mma32(acc, frag16<HS>(sGz + (16 * it + lc) * LH, 32 * ks, g), wf[ks]);
#pragma unroll
          for (int r = 0; r < 4; ++r) kr[it][r] += acc[r];
        }
        if (sl == 0) {  // the term that no slice shares
#pragma unroll
          for (int it = 0; it < TM; ++it) {
            f4 po = zero4();
#pragma unroll
            for (int c = 0; c < NCI; ++c)
              mma32(po, gfrag<CP>(rc + RL.fc.o[rec::PoT], (16 * it + lc) * CP, 32 * c, g),
                    frag16<CP>(sdOT + (16 * strip + lc) * LC8, 32 * c, g));
#pragma unroll
            for (int r = 0; r < 4; ++r) kr[it][r] -= po[r];
          }
        }
#pragma unroll
        for (int it = 0; it < TM; ++it) {
          unsigned long long* const p = xb + (uint32_t)(sl * CP * D + (16 * it + 4 * g) * D + 16 * strip + lc);
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float v = kr[it][r];
            __hip_atomic_store(p + r * D, ((unsigned long long)tag << 32) | __builtin_bit_cast(unsigned, v),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
        }
      }
      // ---- the adjoint update's terms without Ykbar
      const float AC = sc3[0], BC = sc3[1], EC = sc3[2];
      {
        const Lane y;
        const int g = y.g, lc = y.lc;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          f4 nw = AC * w1[dt], ns = EC * w1[dt] + BC * s1[dt];
#pragma unroll
          for (int c = 0; c < NCI; ++c) {
            mma32(nw, frag16<CP>(sXAT + (16 * dt + lc) * LC8, 32 * c, g), zb[c]);
            mma32(ns, frag16<CP>(sXET + (16 * dt + lc) * LC8, 32 * c, g), zb[c]);
          }
          w1[dt] = nw;
          s1[dt] = ns;
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const int row = 16 * dt + lc;
          f4 nw = AC * w2[dt], ns = EC * w2[dt] + BC * s2[dt];
#pragma unroll
          for (int c = 0; c < NCI; ++c) {
            mma32(nw, frag16<CP>(sdOAT + row * LC8, 32 * c, g), ht[c]);
            mma32(ns, frag16<CP>(sdOET + row * LC8, 32 * c, g), ht[c]);
            const bf16x8 bg = TM == 1 ? join(gb[0], zero_bf4()) : join(gb[(2 * c) % TM], gb[(2 * c + 1) % TM]);
            mma32(nw, a_pair(sRT, LC4, row, 32 * c, g, TM > 1), bg);
          }
          w2[dt] = nw;
          s2[dt] = ns;
        }
      }
      // W2's hidden column of the lane (for Ykbar W2) and Hk^T, requested ahead of the wait
      bf16x8 w2f[DT / 2], hkf[NCI];
      {
        const Lane y;
#pragma unroll
        for (int c = 0; c < DT / 2; ++c) w2f[c] = gfrag<D>(W2T, (hw + y.lc) * D, 32 * c, y.g);
#pragma unroll
        for (int c = 0; c < NCI; ++c) hkf[c] = gfrag<CP>(rc + RL.fc.o[rec::HkT], (hw + y.lc) * CP, 32 * c, y.g);
      }
      // ---- the other slice's part of Rbar added to this one's (from the registers: a
      // workgroup never reads words that it may still be writing; two terms, so their order
      // does not matter) -> Ykbar
      if (pair == 1) {
        const Lane y;
        const unsigned long long* const p = xb + (uint32_t)((1 - sl) * CP * D + 4 * y.g * D + 16 * strip + y.lc);
#pragma unroll
        for (int it = 0; it < TM; ++it) {  // a tile at a time (the later ones have mostly arrived)
          unsigned long long x[4];
          bool all = false;  // of the wave
          for (int round = lost ? WAIT_ROUNDS - 1 : 0; !all && round < WAIT_ROUNDS; ++round) {
            bool ok = true;
#pragma unroll
            for (int r = 0; r < 4; ++r)
              x[r] = __hip_atomic_load(p + (16 * it + r) * D, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int r = 0; r < 4; ++r) ok = ok && (unsigned)(x[r] >> 32) == tag;
            all = __builtin_amdgcn_readfirstlane(__all(ok)) != 0;
            if (!all) __builtin_amdgcn_s_sleep(1);
          }
          lost = lost || !all;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            kr[it][r] += all ? __builtin_bit_cast(float, (unsigned)x[r]) : __builtin_nanf("");
        }
#pragma unroll
        for (int it = 0; it < TM; ++it) put_y(it, kr[it], dvp);
      }
      __syncthreads();  // Ykbar, K^T complete

      // ---- Zkbar, the rest of the update
      if (pair == 0) load_wf(W1T);
      bf16x4 zk[TM];
      const Lane y4;
      const int g = y4.g, lc = y4.lc;
#pragma unroll
      for (int it = 0; it < TM; ++it) {
        f4 acc = zero4();
#pragma unroll
        for (int c = 0; c < DT / 2; ++c)
          mma32(acc, frag16<D>(sYk + (16 * it + lc) * LD8, 32 * c, g), w2f[c]);
        f4 zv;
#pragma unroll
        for (int r = 0; r < 4; ++r) zv[r] = acc[r] * (float)spv[it][r] + zkp[it][r];
        zk[it] = cvt4(zv);
        const int q = lc & 3;
        *reinterpret_cast<bf16x4*>(sGz + (16 * it + 4 * g + q) * LH + 16 * w + lc - q) = cvt4(quad_transpose(zv));
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const int row = 16 * dt + lc;
#pragma unroll
        for (int c = 0; c < NCI; ++c) {
          const bf16x8 bz = TM == 1 ? join(zk[0], zero_bf4()) : join(zk[(2 * c) % TM], zk[(2 * c + 1) % TM]);
          mma32(w1[dt], a_pair(sKT, LC4, row, 32 * c, g, TM > 1), bz);
          mma32(w2[dt], frag16<CP>(sYkT + row * LC8, 32 * c, g), hkf[c]);
        }
      }
      write_copies();
      __syncthreads();  // Zkbar and the adjoint's copies complete

      // ---- the slice's part of dk
      if (pair == 0) {
        const Lane y;
        const int g = y.g, lc = y.lc;
        float* const dk = P.dks + (t * G + sl) * CP * D;
#pragma unroll
        for (int it = 0; it < TM; ++it) {
          f4 acc = kr[it];
#pragma unroll
          for (int ks = 0; ks < HS / 32; ++ks)
            mma32(acc, frag16<HS>(sGz + (16 * it + lc) * LH, 32 * ks, g), wf[ks]);
          const int i = 16 * it + 4 * g, j = 16 * strip + lc, q = lc & 3;
          const f4 v = quad_transpose(acc);
          *reinterpret_cast<f32x4*>(dk + (size_t)(i + q) * D + j - q) = f32x4{v[0], v[1], v[2], v[3]};
        }
      }
      if (LO && n > P.n0) {
        StatePairs L;
        load_pairs(u, n - 1, L);
        exact_dots(L);
      }
    }
    // the adjoint for the launch of the earlier chunks, or of the learned init
    {
      float* const o1 = P.n0 == 0 ? a.dWinit_part + (size_t)u * 2 * hd : adj0;
      const int l = lane_id(), g = l >> 4, lc = l & 15, h = h0 + 16 * w + lc;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const int d0 = 16 * dt + 4 * g;
        *reinterpret_cast<f32x4*>(o1 + (size_t)h * D + d0) = f32x4{w1[dt][0], w1[dt][1], w1[dt][2], w1[dt][3]};
#pragma unroll
        for (int r = 0; r < 4; ++r) o1[hd + (size_t)(d0 + r) * H + h] = w2[dt][r];
        if (P.n0) {
          *reinterpret_cast<f32x4*>(adj0 + 2 * hd + (size_t)h * D + d0) = f32x4{s1[dt][0], s1[dt][1], s1[dt][2], s1[dt][3]};
#pragma unroll
          for (int r = 0; r < 4; ++r) adj0[3 * hd + (size_t)(d0 + r) * H + h] = s2[dt][r];
        }
      }
    }
  }
}

namespace {
template <int D, int H, int CP, bool LO>
bool try_walk(const LocalBwdArgs& a, const SplitPtrs& P, hipStream_t st, hipError_t* err) {
  if (a.D.d != D || a.D.hid != H || a.D.Cp != CP || (a.statesLo != nullptr) != LO) return false;
  using B = BWalk<D, H, CP>;
  constexpr size_t lds = (size_t)B::total * sizeof(__bf16);
  auto kern = local_bwd_walk_kernel<D, H, CP, LO>;
  if (!lds_fits((const void*)kern, lds)) {
    *err = hipErrorInvalidConfiguration;
    return true;
  }
  set_lds_limit((const void*)kern);
  const int grid = (P.groups + WALK_LANES - 1) / WALK_LANES * WALK_LANES * B::G;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(B::NT), lds, st, a, P);
  *err = hipGetLastError();
  return true;
}
}  // namespace

bool launch_local_bwd_walk(const LocalBwdArgs& a, const SplitPtrs& P, hipStream_t st, hipError_t* err) {
  return try_walk<64, 256, 32, false>(a, P, st, err) || try_walk<64, 256, 16, false>(a, P, st, err) ||
         try_walk<64, 256, 32, true>(a, P, st, err) || try_walk<64, 256, 16, true>(a, P, st, err);
}

}  // namespace tnt
