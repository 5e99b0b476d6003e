// Refinement below the roots (bf16 caches; App. A.3 "Recursive refinement
// rule", App. B.4 eq:app_tree_split_candidates).
//
// A node's refinement needs nothing of another node but its own distortion, so
// nodes are refined in any order and numbered at the end:
//   * k_sub_first lists the children of the refined roots: nodes of more than
//     ST_N tokens for the split kernel, smaller ones for the subtree kernel;
//   * the split kernels (split.hip, their LV form) refine the long nodes, one
//     workgroup per node, class by class (128, 64 and 32 tokens at most); a
//     workgroup goes on with the child of its own class and lists the others;
//   * k_subtree takes a node of at most ST_N tokens to its singletons, one wave
//     per node, with no barrier;
//   * k_number gives every unit its breadth-first order.
// Whoever refines a node appends its children to the unit's node slots (a
// counter per unit), in any order, with the depth in node_parent.  Breadth-first
// order is (depth, start): parents come in order of their starts, children are
// contiguous and left to right, so k_number ranks the starts of a depth by
// population counts over a 128-bit mask.  (One launch of the split kernel and
// one numbering pass per depth, up to 48 of each, took 347 + 62 ms of a
// complete build over 8.4 million tokens, at 42 ns per node whatever its size.)
//
// Pruned build: a node is refined when the utility bound of the op that creates
// it (the least utility on its path, the high word of the effective key)
// reaches that of theta: every node that the 64-bit comparison would take.
#include "common.h"

namespace gkv {

constexpr int ST_T = 256;                 // four waves, each on its own subtree

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// The region of the lists: offsets of its arrays and its size, the one place that both
// the plan and the view take them from.  The nodes of a list are disjoint, of at
// least ST_N + 1 and 2 tokens: 22 bytes a token, and six roundings.
BelowLists below_lists(int64_t LG, int64_t N_c) {
  BelowLists b;
  b.long_cap = LG * (N_c / (ST_N + 1)) + 1;
  size_t o = 0;
  auto put = [&](size_t& off, size_t bytes) { off = o; o = al256(o + bytes); };
  for (int c = 0; c < LONG_CLASSES; ++c) put(b.long_items[c], (size_t)b.long_cap * 32);
  put(b.sub_items, (size_t)(LG * short_capacity(N_c)) * 32);
  put(b.sub_ctr, (size_t)LG * 4);
  put(b.lv_ctr, 16 * 4);
  b.bytes = o;
  return b;
}

static __device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

__global__ void k_sub_reset(const Dims* __restrict__ dmp, const TreeView* __restrict__ tvp) {
  const TreeView& tv = *tvp;
  const int LG = dmp->L * dmp->G;
  if (threadIdx.x < 16) tv.lv_ctr[threadIdx.x] = 0;
  for (int i = threadIdx.x; i < LG; i += blockDim.x) tv.sub_ctr[i] = 0;
}

// The children of every refined root, one unit per thread; the lanes of a wave
// that list into the same place take one block of it.
__global__ __launch_bounds__(256) void k_sub_first(const Dims* __restrict__ dmp, const TreeView* __restrict__ tvp,
                                                   int full) {
  const Dims& dm = *dmp;
  const TreeView& tv = *tvp;
  const int nunits = tv.wctr[8];
  const int J = *tv.nslots;
  const uint64_t theta = full ? 0ull : tv.theta[0];
  const int lane = threadIdx.x & 63;
  const int64_t scap = short_capacity(dm.N_c);
  for (int k0 = (int)(blockIdx.x * blockDim.x + (threadIdx.x & ~63u)); k0 < nunits; k0 += (int)(gridDim.x * blockDim.x)) {
    const int k = k0 + lane;
    int unit = 0, lg = 0, cnt = 0;
    int64_t base = 0;
    uint64_t Ef = 0ull;
    if (k < nunits) {
      unit = tv.work[8 * (int64_t)k];
      lg = unit / dm.J_cap;
      const int j = unit % dm.J_cap;
      if (j < J) {
        base = (int64_t)lg * 2 * dm.N_c + 2 * (int64_t)tv.slots[j];
        cnt = tv.unit_nn[unit];
        Ef = full ? ~0ull : tv.sp_E[base];                   // the root's Split
        if (cnt < 2 || cnt > 4 || Ef < theta) cnt = 0;
      }
    }
    const float w = cnt ? tv.omega[lg] : 0.f;
    for (int c = 1; c < 4; ++c) {
      const int n = c < cnt ? tv.node_n[base + c] : 0;
      const int dest = n < 2 ? -1 : list_of(n, lg);
      uint64_t todo = __ballot(dest >= 0);
      while (todo != 0ull) {
        const int lead = __builtin_ctzll(todo);
        const int d = __builtin_amdgcn_readlane(dest, lead);
        const uint64_t same = __ballot(dest == d);
        todo &= ~same;
        int first = 0;
        if (lane == lead) first = atomicAdd(list_counter(tv, d), __popcll(same));
        first = __builtin_amdgcn_readlane(first, lead);
        if (dest == d) {
          int32_t* dst = list_item(tv, d, scap, first + __popcll(same & ((1ull << lane) - 1ull)));
          if (dst) {
            ((int4*)dst)[0] = make_int4(unit, tv.node_a[base + c], n | (1 << 8) | (c << 16), __float_as_int(tv.node_D[base + c]));
            ((int4*)dst)[1] = make_int4(__float_as_int(tv.node_R[base + c]), __float_as_int(w), (int32_t)(Ef >> 32), 0);
          } else {
            atomicOr(tv.status, STATUS_CAPACITY);
          }
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Subtrees of at most 16 tokens, one wave each.
//
// Every child of every node below is an interval [a, x) of the subtree's
// tokens, at most 119 of them, so the wave computes the distortion of each
// interval once, left end by left end from the last to the first, and the
// refinement rule then runs over a table.  (Interval by interval a node's
// prefix and suffix children repeat those of its parent; the table is also what
// makes the work regular: no list of candidates, no masked sums.)
//   * lane = probe: the probe exponentials e_t of the 16 tokens in registers;
//     with Y_t = sum G_tt' e_t' over [a, t) kept per token and updated by one
//     term per left end, the sums over [a, t] of the increments
//     e_t (Z), e_t (Y_t + u_t) (||M||^2), R_t u_t + e_t a_t and u_t + e_t g_t
//     (<M, sum R v>, <M, sum v>), u_t = Y_t + e_t G_tt, run down the tokens;
//   * lane = token: ||sum w v||^2, sum R, sum ||k|| of the intervals, by scans
//     along the 16-lane rows;
//   * lane = rotation pair: k° of the 16 tokens in registers; the key of every
//     interval that starts at a goes to LDS in three bf16 parts, and one tile of
//     matrix products gives its logits against every probe (exact products) and
//     its norm (the diagonal of the tile with itself);
//   * four 4 x 4 exchanges of lane rows turn the product tiles (lane = probe of
//     one tile, token or child in registers) into lane = probe of the wave.
// Sums are fp32 as in the split kernel.  Bound by VALU issue: about 75
// instructions per interval.
template <int D>
struct StLds {
  static constexpr int H2 = D / 2;
  static constexpr int KPS = D + 8;                       // child key row stride (bf16)
  static constexpr int oTab = 0;                          // rotation rows 0 .. 15 (cos, sin)
  static constexpr int oWave = oTab + ST_N * H2 * 8;
  // per wave
  static constexpr int wK = 0;                            // three planes of child keys [16][KPS]
  static constexpr int wG = wK + 3 * ST_N * KPS * 2;      // Gram matrix [16][20]
  static constexpr int wD = wG + ST_N * 20 * 4;           // distortions [a][x], row stride 17
  static constexpr int wC = wD + (ST_N * 17 + 3) / 4 * 16;   // per child (beta, 1/den, ||v~||^2, m_eff)
  static constexpr int wA = wC + ST_N * 16;               // (a_t, g_t)
  static constexpr int wN = wA + ST_N * 8;                // nodes: a | b << 8 | nch << 16 | kind << 20, cut | depth << 8, D, R
  static constexpr int wU = wN + 32 * 16;                 // their utility bounds
  static constexpr int wBytes = wU + 32 * 4;
  static constexpr int bytes = oWave + (ST_T / 64) * wBytes;
  static_assert(wBytes % 16 == 0, "16-byte rows");
};
static_assert(StLds<128>::bytes <= 80 * 1024, "two workgroups per CU");

// (value, index) of the largest value of each row, ties to the smaller index
__device__ __forceinline__ void row_argmax(float& v, int& i) {
#pragma unroll
  for (int sh = 8; sh > 0; sh >>= 1) {
    const float v2 = dpp_ror_f(v, sh);
    const int i2 = dpp_ror_i(i, sh);
    if (v2 > v || (v2 == v && i2 < i)) { v = v2; i = i2; }
  }
}

__device__ __forceinline__ float readlane_f(float v, int l) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

template <int D>
__global__ __launch_bounds__(ST_T, 2) void k_subtree(const Dims* __restrict__ dmp, const TreeView* __restrict__ tvp,
                                                      int full, int chunks, const uint16_t* __restrict__ K,
                                                      const uint16_t* __restrict__ V, const uint16_t* __restrict__ Q,
                                                      const float* __restrict__ cosT, const float* __restrict__ sinT,
                                                      const float* __restrict__ kappa) {
  using Lay = StLds<D>;
  constexpr int H2 = D / 2, KS = D / 32, KPS = Lay::KPS;
  constexpr float LOG2E = 1.44269504088896341f;
  extern __shared__ __align__(16) char smem[];
  const Dims& dm = *dmp;
  const TreeView& tv = *tvp;
  float2* sTab = (float2*)(smem + Lay::oTab);
  for (int e = threadIdx.x; e < ST_N * H2; e += ST_T)
    sTab[e] = e / H2 < dm.T ? make_float2(cosT[e], sinT[e]) : make_float2(1.f, 0.f);
  __syncthreads();
  const int wave = uni((int)threadIdx.x >> 6);
  char* wb = smem + Lay::oWave + wave * Lay::wBytes;
  uint16_t* sK = (uint16_t*)(wb + Lay::wK);
  float* sG = (float*)(wb + Lay::wG);
  float* sD = (float*)(wb + Lay::wD);
  float4* sC = (float4*)(wb + Lay::wC);
  float2* sA = (float2*)(wb + Lay::wA);
  int4* sN = (int4*)(wb + Lay::wN);
  uint32_t* sU = (uint32_t*)(wb + Lay::wU);
  const float sc2 = LOG2E / sqrtf((float)D);
  const float invW = 1.0f / (float)dm.W;
  const float invn = 1.0f / (float)((threadIdx.x & 15) + 1);   // lane i: 1 / (i + 1)
  const int LG = dm.L * dm.G;
  const uint32_t thi = full ? 0u : (uint32_t)(tv.theta[0] >> 32);
  const int nw = (int)gridDim.x * (ST_T / 64);
  for (int task = uni((int)blockIdx.x * (ST_T / 64) + wave); task < LG * chunks; task += nw) {
    const int lg = task / chunks, ch = task - lg * chunks;
    const int64_t cnt = min((int64_t)uni(tv.sub_ctr[lg]), short_capacity(dm.N_c));
    const int i0 = (int)(cnt * ch / chunks), i1 = (int)(cnt * (ch + 1) / chunks);
    if (i0 >= i1) continue;
    const int l = lg / dm.G, g = lg % dm.G;
    // per-lane indices are formed inside the loops: what the compiler derives from
    // them would else be held across items, past the register budget
    int lane = threadIdx.x & 63;
    asm volatile("" : "+v"(lane));
    const int i16 = lane & 15, g4 = lane >> 4;
    // probe rows as the products' column operand, probe shift and normaliser of probe `lane`
    uint4 qf[4][KS];
    {
      const uint16_t* Qp = Q + ((int64_t)l * dm.H + (int64_t)g * dm.hpg) * dm.W * D;
#pragma unroll
      for (int pt = 0; pt < 4; ++pt) {
        const int q0 = 16 * pt + i16, q = q0 < dm.W ? q0 : 0;
        const uint16_t* row = Qp + ((int64_t)(q % dm.hpg) * dm.W + q) * D + 8 * g4;
#pragma unroll
        for (int s = 0; s < KS; ++s) qf[pt][s] = *(const uint4*)(row + 32 * s);
      }
    }
    // a lane without a probe has e = z = 0 in every interval
    const float mq2 = lane < dm.W ? tv.probe_m[(int64_t)lg * dm.W + lane] * LOG2E : INFINITY;
    const float izc = lane < dm.W ? 1.0f / tv.probe_ZC[(int64_t)lg * dm.W + lane] : 0.f;
    const float w = tv.omega[lg];
    for (int it = i0; it < i1; ++it) {
      int lane = threadIdx.x & 63;
      asm volatile("" : "+v"(lane));
      const int i16 = lane & 15, g4 = lane >> 4, pi = lane & (H2 - 1);   // pi: rotation pair
      const int4* ip = (const int4*)(tv.sub_items + 8 * ((int64_t)lg * short_capacity(dm.N_c) + it));
      const int4 d0 = ip[0], d1 = ip[1];
      const int unit = uni(d0.x), a0 = uni(d0.y), word = uni(d0.z);
      const int n = word & 255, depth = (word >> 8) & 255, idx = (word >> 16) & 255;
      const int j = unit - lg * dm.J_cap;
      const int64_t tok0 = (int64_t)lg * dm.N_c + a0;
      // token i16 in every 16-lane row
      const bool tok = i16 < n;
      const int ti = tok ? i16 : n - 1;
      const float tR = tok ? tv.tok_R[tok0 + ti] : 0.f;
      float tA = tok ? tv.tok_A[tok0 + ti] : -INFINITY;
      if (tA != tA) tA = -INFINITY;                       // the choices below stay the same in every lane
      const float tkap = kappa[a0 + ti];
      const bool tfl = tv.fl_flag && tok && tv.fl_flag[tok0 + ti];
      if (n > 2) {
        const uint16_t* Kp = K + ((int64_t)lg * dm.T + a0) * D;
        const uint16_t* Vp = V + ((int64_t)lg * dm.T + a0) * D;
        uint4 kf[KS], vf[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) kf[s] = *(const uint4*)(Kp + (int64_t)ti * D + 32 * s + 8 * g4);
#pragma unroll
        for (int s = 0; s < KS; ++s) vf[s] = *(const uint4*)(Vp + (int64_t)ti * D + 32 * s + 8 * g4);
        uint16_t r1[ST_N], r2[ST_N];
#pragma unroll
        for (int t = 0; t < ST_N; ++t) {
          const int tt = t < n ? t : n - 1;
          r1[t] = Kp[(int64_t)tt * D + pi];
          r2[t] = Kp[(int64_t)tt * D + pi + H2];
        }
        // logits of the tokens, ||k_t||^2 and the Gram matrix of the values
        float e[ST_N];
        {
          f32x4 acc[4];
#pragma unroll
          for (int pt = 0; pt < 4; ++pt) {
            acc[pt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) acc[pt] = mfma_bf16_16x16x32(pk8(kf[s]), pk8(qf[pt][s]), acc[pt]);
          }
          mfma_done(acc);
          tiles_to_columns(acc, e);
#pragma unroll
          for (int t = 0; t < ST_N; ++t) e[t] = __builtin_amdgcn_exp2f(e[t] * sc2 - mq2);
        }
        f32x4 kk = {0.f, 0.f, 0.f, 0.f}, gg = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
          kk = mfma_bf16_16x16x32(pk8(kf[s]), pk8(kf[s]), kk);
          gg = mfma_bf16_16x16x32(pk8(vf[s]), pk8(vf[s]), gg);
        }
        mfma_done(kk);
        mfma_done(gg);
        // the diagonal of a tile sits at lane (i, i / 4), element i % 4; every row gets it
        const int rs = i16 & 3;
        auto diagonal = [&](const f32x4& x) {
          const float v = rs == 0 ? x[0] : (rs == 1 ? x[1] : (rs == 2 ? x[2] : x[3]));
          return g4 == (i16 >> 2) ? v : 0.f;
        };
        const float tkn = tok ? sqrtf(col_sum4(diagonal(kk))) : 0.f;
        const float tGd = col_sum4(diagonal(gg));
#pragma unroll
        for (int r = 0; r < 4; ++r) sG[(4 * g4 + r) * 20 + i16] = gg[r];
        float uR[ST_N], uG[ST_N];                        // the same for every lane
#pragma unroll
        for (int t = 0; t < ST_N; ++t) {
          uR[t] = readlane_f(tR, t);
          uG[t] = readlane_f(tGd, t);
        }
        // k° of every token, turned back to the subtree's start
        float k1[ST_N], k2[ST_N];
#pragma unroll
        for (int t = 0; t < ST_N; ++t) {
          const float2 cs = sTab[t * H2 + pi];
          const float x = __uint_as_float((uint32_t)r1[t] << 16), y = __uint_as_float((uint32_t)r2[t] << 16);
          k1[t] = x * cs.x + y * cs.y;
          k2[t] = y * cs.x - x * cs.y;
        }
        float Y[ST_N];
#pragma unroll
        for (int t = 0; t < ST_N; ++t) Y[t] = 0.f;
        // lane = last token t of the interval [a, t]: sums over its tokens
        float sR = 0.f, sKn = 0.f, RR = 0.f, RG = 0.f, GG = 0.f, at = 0.f, gt = 0.f;
        // a singleton's sums (left end n - 1)
        if (i16 == n - 1) {
          sR = tR; sKn = tkn;
          RR = tR * tR * tGd; RG = tR * tGd; GG = tGd;
        }
        wave_lds_order();
#pragma unroll 1
        for (int a = n - 2; a >= 0; --a) {
          const int tl = a == 0 ? n - 2 : n - 1;          // last t evaluated: the subtree's root is known
          // ---- keys of the intervals [a, t]: mean k° turned to the representative position ----
          {
            // representative position of [a0 + a, a0 + t + 1) less a0
            auto rep = [&](int t) {
              const int m = 2 * a0 + a + t, h = m >> 1;
              return ((m & 1) ? h + (h & 1) : h) - a0;
            };
            float s1 = 0.f, s2 = 0.f;
            float2 csn = sTab[rep(a + 1) * H2 + pi];
#pragma unroll
            for (int t = 0; t < ST_N; ++t) {
              if (t >= a && t <= tl) {
                s1 += k1[t];
                s2 += k2[t];
                if (t > a) {
                  const float2 cs = csn;
                  csn = sTab[(rep(t + 1) & (ST_N - 1)) * H2 + pi];
                  const float inv = readlane_f(invn, t - a);
                  const float m1 = s1 * inv, m2 = s2 * inv;
                  const float o[2] = {m1 * cs.x - m2 * cs.y, m2 * cs.x + m1 * cs.y};
#pragma unroll
                  for (int h = 0; h < 2; ++h) {
                    // o = hi + mid + lo exactly, each a bf16
                    const uint32_t hi = __float_as_uint(o[h]);
                    const float d1 = o[h] - __uint_as_float(hi & 0xffff0000u);
                    const uint32_t mi = __float_as_uint(d1);
                    const uint32_t lo = __float_as_uint(d1 - __uint_as_float(mi & 0xffff0000u));
                    uint16_t* dst = sK + t * KPS + pi + h * H2;
                    dst[0] = (uint16_t)(hi >> 16);
                    dst[ST_N * KPS] = (uint16_t)(mi >> 16);
                    dst[2 * ST_N * KPS] = (uint16_t)(lo >> 16);
                  }
                }
              }
            }
          }
          // ---- lane = t: sums over [a, t], from those over [a + 1, t] ----
          const float ra = readlane_f(tR, a), ka = readlane_f(tkn, a), ga = readlane_f(tGd, a);
          const float gat = sG[a * 20 + i16];
          const bool past = i16 > a;
          const float c1 = row_scan16(past ? gat * tR : 0.f), c0 = row_scan16(past ? gat : 0.f);
          if (i16 >= a) {
            sR += ra;
            sKn += ka;
            RR += ra * (ra * ga + 2.f * c1);
            RG += ra * ga + (ra * c0 + c1);
            GG += ga + 2.f * c0;
          }
          if (past) { at += gat * ra; gt += gat; }
          if (lane < ST_N) sA[i16] = make_float2(at, gt);
          wave_lds_order();
          // ---- logits of the interval keys (rows t) against every probe, and the keys' norms ----
          f32x4 acc[4], nn2 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int pt = 0; pt < 4; ++pt) acc[pt] = f32x4{0.f, 0.f, 0.f, 0.f};
          s16x8 kx[3][KS];
          // the low parts first: the matrix cores truncate at the size of the sum so far
#pragma unroll
          for (int part = 2; part >= 0; --part)
#pragma unroll
            for (int s = 0; s < KS; ++s) {
              kx[part][s] = pk8(*(const uint4*)(sK + (part * ST_N + i16) * KPS + 32 * s + 8 * g4));
#pragma unroll
              for (int pt = 0; pt < 4; ++pt) acc[pt] = mfma_bf16_16x16x32(kx[part][s], pk8(qf[pt][s]), acc[pt]);
            }
#pragma unroll
          for (int o = 0; o < 6; ++o) {
            constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int s = 0; s < KS; ++s) nn2 = mfma_bf16_16x16x32(kx[pa[o]][s], kx[pb[o]][s], nn2);
          }
          mfma_done(nn2);
          mfma_done(acc);
          // constants of the child [a, t]: lane (t, t / 4) holds its key's norm
          {
            const float ss = rs == 0 ? nn2[0] : (rs == 1 ? nn2[1] : (rs == 2 ? nn2[2] : nn2[3]));
            const float nch = (float)(i16 - a + 1);
            const float inv = __shfl(invn, (i16 - a) & 15, 64);
            const float km = sKn * inv + dm.eps;
            const float me = fminf(fmaxf(nch * (ss / (km * km)), 1.0f), nch);
            const float beta = dm.beta_frac * sR * inv;
            const float iden = 1.0f / (sR + nch * beta + dm.eps);
            const float vv = (RR + beta * (2.f * RG + beta * GG)) * (iden * iden);
            if (past && g4 == (i16 >> 2)) sC[i16] = make_float4(beta, iden, vv, me);
          }
          float z[ST_N];
          tiles_to_columns(acc, z);
          wave_lds_order();
          // ---- lane = probe: running sums over [a, t] and D_q of each interval ----
          const float4* grow = (const float4*)(sG + a * 20);
          const float4 gr[4] = {grow[0], grow[1], grow[2], grow[3]};
          float ea = 0.f, Z = 0.f, S = 0.f, P = 0.f, Qs = 0.f;
          float con[ST_N];
          float4 c4n = sC[(a + 1) & (ST_N - 1)];
          float2 agn = sA[(a + 1) & (ST_N - 1)];
#pragma unroll
          for (int t = 0; t < ST_N; ++t) {
            con[t] = 0.f;
            if (t == a) {
              ea = e[t];
              const float u = ea * uG[t];
              Z = ea;
              S = ea * u;
              P = uR[t] * u;
              Qs = u;
            }
            if (t > a && t <= tl) {
              const float4 c4 = c4n;
              const float2 ag = agn;
              c4n = sC[(t + 1) & (ST_N - 1)];
              agn = sA[(t + 1) & (ST_N - 1)];
              const float gv = (t & 3) == 0 ? gr[t >> 2].x : ((t & 3) == 1 ? gr[t >> 2].y : ((t & 3) == 2 ? gr[t >> 2].z : gr[t >> 2].w));
              const float y = Y[t] + gv * ea;
              Y[t] = y;
              const float et = e[t];
              const float u = y + et * uG[t];
              Z += et;
              S += et * (y + u);
              P += uR[t] * u + et * ag.x;
              Qs += u + et * ag.y;
              const float zt = __builtin_amdgcn_exp2f(z[t] * sc2 - mq2) * c4.w;
              const float xv = (P + c4.x * Qs) * c4.y;
              const float s1 = fmaxf(S + zt * (zt * c4.z - 2.f * xv), 0.f);
              const float dz = Z - zt;
              const float Dq = dm.lam_Z * dz * dz * __builtin_amdgcn_rcpf(Z * Z + dm.eps) +
                               dm.lam_M * s1 * __builtin_amdgcn_rcpf(S + dm.eps);
              con[t] = (Z * izc) * Dq;
            }
          }
          // sums over the probes: row g, element k of v holds interval t = 4 g + k
          float v[4];
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const auto p0 = __builtin_amdgcn_permlane32_swap(__float_as_uint(con[k]), __float_as_uint(con[k + 8]), false, false);
            const auto p1 = __builtin_amdgcn_permlane32_swap(__float_as_uint(con[k + 4]), __float_as_uint(con[k + 12]), false, false);
            const float x = __uint_as_float(p0[0]) + __uint_as_float(p0[1]);
            const float y = __uint_as_float(p1[0]) + __uint_as_float(p1[1]);
            const auto p2 = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
            v[k] = row_sum16(__uint_as_float(p2[0]) + __uint_as_float(p2[1]));
          }
          if (i16 < 4) {
            const float dv = i16 == 0 ? v[0] : (i16 == 1 ? v[1] : (i16 == 2 ? v[2] : v[3]));
            sD[a * 17 + 4 * g4 + i16 + 1] = dv * invW;
          }
          wave_lds_order();
        }
      }
      // ---- the refinement rule over the table: four nodes at a time, one per
      // 16-lane row; cut x = a + 1 + i16, token i16 ----
      if (lane == 0) {
        sN[0] = make_int4(0 | (n << 8), depth << 8, d0.w, d1.x);
        sU[0] = (uint32_t)d1.z;
      }
      wave_lds_order();
      int head = 0, tail = 1;
      while (head < tail) {
        const int q = head + g4;
        const bool on = q < tail;
        const int4 nd = sN[on ? q : head];
        const uint32_t uc = sU[on ? q : head];
        const int a = nd.x & 255, b = (nd.x >> 8) & 255, m = b - a, dep = (nd.y >> 8) & 255;
        const float Dv = __int_as_float(nd.z), Rv = __int_as_float(nd.w);
        const bool go = on && m >= 2 && (full || uc >= thi);
        // D of [x, y): 0 for a singleton
        auto dist = [&](int x, int y) { return y - x >= 2 ? sD[x * 17 + y] : 0.f; };
        const bool in = i16 >= a && i16 < b;
        // extraction token: largest probe mass; a node of three or more tokens that
        // holds a floor candidate is extracted at the one of largest value, with no choice
        float pa = in ? tA : -INFINITY, pf = in && tfl && tR == tR ? tR : -INFINITY;
        int p = in ? i16 : 0x7fffffff, fp = in && tfl ? i16 : 0x7fffffff;
        row_argmax(pa, p);
        bool forced = false;
        if (tv.fl_flag) {
          row_argmax(pf, fp);
          forced = m >= 3 && fp != 0x7fffffff;
          if (forced) p = fp;
        }
        p = p < ST_N ? p : a;
        float kmn = in ? tkap : INFINITY, kmx = in ? tkap : -INFINITY;
#pragma unroll
        for (int sh = 8; sh > 0; sh >>= 1) {
          kmn = fminf(kmn, dpp_ror_f(kmn, sh));
          kmx = fmaxf(kmx, dpp_ror_f(kmx, sh));
        }
        const float kr = kmx - kmn;
        // curvature position t = a + i16 proposes the cut t + 1: the k_curv largest
        // over [a, b - 2], ties to the smaller t; the midpoint
        const int t = a + i16;
        const float kt = __shfl(tkap, 16 * g4 + (t & 15), 64);
        bool cand = t < b - 1;
        if (dm.k_curv < ST_N - 1) {
          int rank = 0;
#pragma unroll
          for (int k = 0; k < ST_N; ++k) {
            const float k2v = __shfl(tkap, k, 64);
            rank += (int)(k >= a && k < b - 1 && (k2v > kt || (k2v == kt && k < t)));
          }
          cand = cand && (rank < dm.k_curv || t + 1 == a + m / 2);
        }
        float best = -INFINITY;
        int bk = 0x7fffffff;
        if (cand && !forced) {
          const float kh = kr > 0.f ? (kt - kmn) / kr : 0.f;
          best = ((Dv - dist(a, t + 1)) - dist(t + 1, b)) + dm.lam_kappa * kh;
          if (best != best) best = -INFINITY;
          bk = t + 1;
        }
        row_argmax(best, bk);
        const float dl = p > a ? dist(a, p) : 0.f, dr = p + 1 < b ? dist(p + 1, b) : 0.f;
        const int kids = 1 + (p > a) + (p + 1 < b);
        const float gext = m > 2 ? (Dv - (dl + dr)) / (float)(kids - 1) : -INFINITY;
        const bool bin = m == 2 || (bk < ST_N && best >= gext);
        const int x = m == 2 ? a + 1 : bk;
        // children [c0, c1), [c1, c2), [c2, c3)
        const int nk = go ? (bin ? 2 : kids) : 0;
        const int c0 = a;
        const int c1 = bin ? x : (p > a ? p : p + 1);
        const int c2 = bin ? b : (p > a ? p + 1 : b);
        const int c3 = b;
        const float D0 = dist(c0, c1), D1 = dist(c1, c2), D2 = nk > 2 ? dist(c2, c3) : 0.f;
        const float Us = utility(split_gain(w, Rv, Dv, (D0 + D1) + D2), nk - 1);
        const uint32_t ub = min(uc, __float_as_uint(Us));
        const float R0 = row_sum16(i16 >= c0 && i16 < c1 ? tR : 0.f), R1 = row_sum16(i16 >= c1 && i16 < c2 ? tR : 0.f);
        const float R2 = row_sum16(i16 >= c2 && i16 < c3 ? tR : 0.f);
        const int n0 = __builtin_amdgcn_readlane(nk, 0), n1 = __builtin_amdgcn_readlane(nk, 16);
        const int n2 = __builtin_amdgcn_readlane(nk, 32), n3 = __builtin_amdgcn_readlane(nk, 48);
        const int pos = tail + (g4 > 0 ? n0 : 0) + (g4 > 1 ? n1 : 0) + (g4 > 2 ? n2 : 0) + i16;
        if (i16 < nk && pos < 32) {
          const int ka = i16 == 0 ? c0 : (i16 == 1 ? c1 : c2), kb = i16 == 0 ? c1 : (i16 == 1 ? c2 : c3);
          sN[pos] = make_int4(ka | (kb << 8), (dep + 1) << 8, __float_as_int(i16 == 0 ? D0 : (i16 == 1 ? D1 : D2)),
                              __float_as_int(i16 == 0 ? R0 : (i16 == 1 ? R1 : R2)));
          sU[pos] = ub;
        }
        if (i16 == 0 && nk > 0) {
          sN[q].x = nd.x | (nk << 16) | ((bin ? 1 : 2) << 20);
          sN[q].y = nd.y | (bin ? x : p);
        }
        head = min(head + 4, tail);
        tail = min(tail + n0 + n1 + n2 + n3, 32);
        wave_lds_order();
      }
      // ---- the subtree's nodes into the unit's slots ----
      if (tail > 1 && j >= 0 && j < dm.J_cap) {
        const int sl = tv.slots[j], nslot = tv.slots[j + 1] - sl;
        const int64_t base = (int64_t)lg * 2 * dm.N_c + 2 * (int64_t)sl;
        int pos = 0;
        if (lane == 0) pos = atomicAdd(&tv.unit_nn[unit], tail - 1);
        pos = uni(pos);
        if (pos + tail - 1 > 2 * nslot - 1) {            // a tree over n tokens has at most 2n - 1 nodes
          if (lane == 0) atomicOr(tv.status, STATUS_CAPACITY);
        } else if (lane < tail) {
          const int4 nd = sN[lane];
          const int a = nd.x & 255, b = (nd.x >> 8) & 255, nk = (nd.x >> 16) & 15, kind = (nd.x >> 20) & 15;
          const int64_t s = lane == 0 ? base + idx : base + pos + lane - 1;
          if (lane > 0) {
            tv.node_a[s] = a0 + a;
            tv.node_n[s] = b - a;
            tv.node_parent[s] = (nd.y >> 8) & 255;
            tv.node_D[s] = __int_as_float(nd.z);
            tv.node_R[s] = __int_as_float(nd.w);
          }
          tv.node_nch[s] = (uint8_t)nk;
          tv.node_kind[s] = (uint8_t)kind;
          tv.node_cut[s] = nk ? a0 + (nd.y & 255) : -1;
        }
      }
      wave_lds_order();
    }
  }
}

// ---------------------------------------------------------------------------
// Breadth-first order of every unit that has more nodes than its root, one wave
// per unit, in place: (depth, start) ranks from one 128-bit mask of starts per
// depth.  The parent of a node is the last node of the depth above that starts
// at or before it, its first child the node of the depth below that starts
// where it does.  Latency-bound: about 40 bytes per node each way.
constexpr int NB_DEPTH = NMAX + 1;        // depths 0 .. 127, and none below
__global__ __launch_bounds__(256) void k_number(const Dims* __restrict__ dmp, const TreeView* __restrict__ tvp) {
  const Dims& dm = *dmp;
  const TreeView& tv = *tvp;
  __shared__ uint4 masks[4][NB_DEPTH];
  __shared__ int first[4][NB_DEPTH + 3];
  const int wave = uni((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  uint4* mk = masks[wave];
  int* fs = first[wave];
  const int J = min(uni(*tv.nslots), dm.J_cap);
  const int total = dm.L * dm.G * J;
  for (int x = uni((int)blockIdx.x * 4 + wave); x < total; x += (int)gridDim.x * 4) {
    const int lg = x / J, j = x - lg * J;
    const int64_t unit = (int64_t)lg * dm.J_cap + j;
    const int nn = uni(tv.unit_nn[unit]);
    if (nn < 2) continue;
    const int a0 = uni(tv.slots[j]), nslot = uni(tv.slots[j + 1]) - a0;
    if (nn > 2 * nslot - 1 || nslot > NMAX) continue;     // latched where the nodes were appended
    const int64_t base = (int64_t)lg * 2 * dm.N_c + 2 * (int64_t)a0;
    int a[4], n[4], dp[4], cut[4], nk[4];
    float D[4], R[4];
    int md = 0;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      const int i = lane + 64 * h;
      a[h] = 0; n[h] = 0; dp[h] = 0; cut[h] = -1; nk[h] = 0; D[h] = 0.f; R[h] = 0.f;
      if (i < nn) {
        const int64_t s = base + i;
        a[h] = (tv.node_a[s] - a0) & (NMAX - 1);
        n[h] = tv.node_n[s];
        dp[h] = i == 0 ? 0 : tv.node_parent[s] & (NMAX - 1);
        cut[h] = tv.node_cut[s];
        D[h] = tv.node_D[s];
        R[h] = tv.node_R[s];
        nk[h] = tv.node_nch[s] | (tv.node_kind[s] << 8);
        md = max(md, dp[h]);
      }
    }
    wait_vm();                                            // every node is read before one is written
#pragma unroll
    for (int sh = 8; sh > 0; sh >>= 1) md = max(md, dpp_ror_i(md, sh));
    md = max(max(__builtin_amdgcn_readlane(md, 0), __builtin_amdgcn_readlane(md, 16)),
             max(__builtin_amdgcn_readlane(md, 32), __builtin_amdgcn_readlane(md, 48)));
    for (int d = lane; d <= md + 1; d += 64) mk[d] = make_uint4(0u, 0u, 0u, 0u);
    wave_lds_order();
#pragma unroll
    for (int h = 0; h < 4; ++h)
      if (lane + 64 * h < nn) atomicOr((uint32_t*)&mk[dp[h]] + (a[h] >> 5), 1u << (a[h] & 31));
    wave_lds_order();
    // first index of each depth
    int run = 0;
    for (int d0 = 0; d0 <= md + 1; d0 += 64) {
      const int d = d0 + lane;
      int c = 0;
      if (d <= md + 1) {
        const uint4 m = mk[d];
        c = __popc(m.x) + __popc(m.y) + __popc(m.z) + __popc(m.w);
      }
      int inc = c;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
      }
      if (d <= md + 1) fs[d] = run + inc - c;
      run += __builtin_amdgcn_readlane(inc, 63);
    }
    wave_lds_order();
    // starts of depth d below position p
    auto below = [&](int d, int p) {
      const uint4 m = mk[d];
      const uint32_t wds[4] = {m.x, m.y, m.z, m.w};
      int c = 0;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int r = p - 32 * k;
        const uint32_t keep = r <= 0 ? 0u : (r >= 32 ? ~0u : (1u << r) - 1u);
        c += __popc(wds[k] & keep);
      }
      return c;
    };
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      if (lane + 64 * h >= nn) continue;
      const int i = fs[dp[h]] + below(dp[h], a[h]);
      const int64_t s = base + i;
      tv.node_a[s] = a0 + a[h];
      tv.node_n[s] = n[h];
      tv.node_child[s] = (nk[h] & 255) ? fs[dp[h] + 1] + below(dp[h] + 1, a[h]) : -1;
      tv.node_parent[s] = dp[h] == 0 ? -1 : fs[dp[h] - 1] + below(dp[h] - 1, a[h] + 1) - 1;
      tv.node_nch[s] = (uint8_t)(nk[h] & 255);
      tv.node_kind[s] = (uint8_t)(nk[h] >> 8);
      tv.node_cut[s] = cut[h];
      tv.node_D[s] = D[h];
      tv.node_R[s] = R[h];
    }
    wave_lds_order();
  }
}

hipError_t launch_below_roots(const Dims& dm, bool full, const void* K, const void* V, const void* Q,
                              const float* cosT, const float* sinT, const int32_t* n_slots, const float* kappa,
                              const TreeView& tv, int cus, hipStream_t st) {
  const Dims* dmp = (const Dims*)tv.kargs;
  const TreeView* tvp = (const TreeView*)((const char*)tv.kargs + 512);
  const int f = full ? 1 : 0;
  hipLaunchKernelGGL(k_sub_reset, dim3(1), dim3(256), 0, st, dmp, tvp);
  hipLaunchKernelGGL(k_sub_first, dim3((unsigned)(2 * cus)), dim3(256), 0, st, dmp, tvp, f);
  const hipError_t e = launch_split_long(dm, full, K, V, Q, cosT, sinT, n_slots, kappa, tv, cus, st);
  if (e != hipSuccess) return e;
  // a wave takes a share of one (l, g)'s subtrees at a time (the probe rows stay
  // in registers): about eight shares per wave, dealt round the grid
  const int grid = 2 * cus, LG = dm.L * dm.G;
  const int chunks = (8 * grid * (ST_T / 64) + LG - 1) / LG;
#define GKV_ST(DD)                                                                                              \
  do {                                                                                                          \
    const hipError_t e0 = hipFuncSetAttribute((const void*)k_subtree<DD>,                                       \
                                              hipFuncAttributeMaxDynamicSharedMemorySize, StLds<DD>::bytes);    \
    if (e0 != hipSuccess) return e0;                                                                            \
    hipLaunchKernelGGL((k_subtree<DD>), dim3((unsigned)grid), dim3(ST_T), StLds<DD>::bytes, st, dmp, tvp, f,    \
                       chunks, (const uint16_t*)K, (const uint16_t*)V, (const uint16_t*)Q, cosT, sinT, kappa);  \
  } while (0)
  if (dm.d == 128) GKV_ST(128); else if (dm.d == 64) GKV_ST(64); else return hipErrorInvalidValue;
#undef GKV_ST
  hipLaunchKernelGGL(k_number, dim3((unsigned)(8 * cus)), dim3(256), 0, st, dmp, tvp);
  return hipGetLastError();
}

}  // namespace gkv
