// Refinement of the long nodes of the prototype trees (bf16 caches): the root of
// every unit the build needs, then the nodes of more than ST_N tokens below the
// roots (App. A.3 "Recursive refinement rule": eq:app_binary_split,
// eq:app_extract_split, eq:app_split_choice; App. B.4
// eq:app_tree_split_candidates), with the child prototypes of
// eq:app_rope_prototype, eq:app_value_prototype, eq:app_effective_multiplicity
// and their distortions eq:app_original_attention_stats ..
// eq:app_node_and_drop_distortion.
//
// One workgroup of four waves per node, one kernel per size class (at most 32,
// 64 or 128 tokens: NT = 2, 4, 8 tiles of 16), so that a short node holds little
// LDS and few registers and more workgroups share a CU.  Of a node's children
// at most one is in its own class; the workgroup goes on with that one (a chain
// that peels one token at a time ends in one launch) and lists the others.
//
// The candidate children are prefixes [0, x) and suffixes [x, n) of the node, at
// most 18 each.  ||M_q||^2, <M_q, v~> and ||v~||^2 of a child are quadratic forms
// in the Gram matrix G = V V^T over its token pairs, i.e. sums over the child of
// per-token increments built from Y_t = sum G_tt' e_t' over t' < t (prefixes) or
// t' > t (suffixes).  Per node:
//   * each wave owns a token tile (two for NT = 8, one direction of one for
//     NT = 2): probe exponentials (matrix cores), then exchanged into lane =
//     probe, where prefix and suffix sums simply run down the tokens;
//   * Y of the wave's tile from the Gram tiles, computed where they are used: the
//     bf16 product's output is the fp32 product's operand, lane for lane, and so
//     is a tile of exponentials, so neither G nor Y passes through LDS.  Two
//     more columns, R and 1, give the sums of G against them;
//   * keys: lane = rotation pair, running sums of k° = RoPE^{-1}(k) (turned back
//     to the node's start) read off at the cuts, turned to the child's
//     representative position, in three bf16 parts (exact products) against the
//     probe rows on the matrix cores; the child key's norm is the diagonal of
//     its tile with itself;
//   * the sums of a tile, its running sums again with the tiles before it added,
//     and D_q of every child at its cut, lane = probe;
//   * the fp32 scores decide (binary form wins ties, smaller cut wins ties).
// The value term ||M - z v~||^2 = ||M||^2 - 2 z <M, v~> + z^2 ||v~||^2 (clamped at
// 0) carries a rounding error of a few fp32 ulps of ||M||^2, about 1e-6 of the
// node's attention mass in D, far below the distortions compared.
#include "common.h"

namespace gkv {

constexpr int SP_WGS = 3;
constexpr int SP_T = 256;               // threads: four waves
constexpr int SP_CM = CAND_MAX;         // children per direction
constexpr int SP_CC = 2 * SP_CM;        // prefix side [0, SP_CM), suffix side [SP_CM, SP_CC)

template <int D, int NT>
struct SpLds {
  static constexpr int NM = 16 * NT;                      // longest node
  static constexpr int KTS = D + 4;                       // row of a child's key sums (fp32)
  static constexpr int EB = NT * 4 * 64 * 16;             // exponentials: tile, probe tile, lane, four tokens
  static constexpr int TB = 2 * NT * 4 * 64 * 4;          // later, over them: sums of each tile and direction
  static constexpr int ZB = SP_CC * 64 * 4;               // ... and exp(k~ . q / sqrt(d) - m_q) of every child
  static constexpr int oE = 0;
  static constexpr int oZ = TB;
  static constexpr int oK = EB > TB + ZB ? EB : TB + ZB;  // [SP_CC][KTS] key sums of the children
  static constexpr int oT = oK + SP_CC * KTS * 4;            // [NT][2][64] key sums of each tile
  static constexpr int oCs = oT + NT * 2 * 64 * 4;        // [3][SP_CC] length, sum R, D
  static constexpr int oC4 = oCs + 3 * SP_CC * 4;         // [SP_CC] (beta, 1/den, ||v~||^2, mean ||k||)
  static constexpr int oSS = oC4 + SP_CC * 16;            // [SP_CC] ||mean k°||^2
  static constexpr int oAG = oSS + SP_CC * 4;             // [2][2][NM] sums of G against R and 1
  static constexpr int oGd = oAG + 4 * NM * 4;            // [NM] G_tt
  static constexpr int oR = oGd + NM * 4;                 // [NM] R_t
  static constexpr int oA = oR + NM * 4;                  // [NM] probe mass A_t
  static constexpr int oKap = oA + NM * 4;                // [NM] kappa_t
  static constexpr int oKn = oKap + NM * 4;               // [NM] ||k_t||
  static constexpr int oFlag = oKn + NM * 4;              // [NM] candidate cut flags
  static constexpr int oMap = oFlag + NM * 4;             // [NM + 16] cut x: prefix child | suffix child << 8
  static constexpr int oL = oMap + (NM + 16) * 4;         // lists and metadata (int)
  static constexpr int oFl = oL + 192 * 4;                // [NM] singleton-floor candidate flags
  static constexpr int bytes = oFl + NM;
  static_assert(oK % 16 == 0 && oC4 % 16 == 0 && oAG % 16 == 0, "16-byte rows");
};
static_assert(SpLds<128, 8>::bytes <= 80 * 1024, "two workgroups per CU");
static_assert(NMAX == 128 && SpLds<128, 4>::bytes <= 160 * 1024 / 3, "three workgroups per CU");

int split_lds_bytes(int d) { return d == 128 ? SpLds<128, 8>::bytes : SpLds<64, 8>::bytes; }

static __device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }

// inclusive prefix sums over the wave
__device__ __forceinline__ float wave_scan(float v) {
  v = row_scan16(v);
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x142, 0xa, 0xf, false));   // row_bcast:15
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x143, 0xc, 0xf, false));   // row_bcast:31
  return v;
}

// LV: the long nodes below the roots (mode BUILD_LONG or BUILD_LONG_FULL, list
// `cls`), else the roots (mode BUILD_ROOT_SPLIT or BUILD_ROOT_FULL, items [first
// of the class, its end) of the work list)
template <int D, int NT, bool LV>
__global__ __launch_bounds__(SP_T, NT == 8 ? 2 : SP_WGS) void k_split(const Dims* __restrict__ dmp, int mode, int cls,
                                                                const uint16_t* __restrict__ K,
                                                                const uint16_t* __restrict__ V,
                                                                const uint16_t* __restrict__ Q,
                                                                const float* __restrict__ cosT,
                                                                const float* __restrict__ sinT,
                                                                const int32_t* __restrict__ n_slots,
                                                                const float* __restrict__ kappa,
                                                                const TreeView* __restrict__ tvp) {
  const Dims& dm = *dmp;
  const TreeView& tv = *tvp;
  using Lay = SpLds<D, NT>;
  constexpr int NM = Lay::NM, H2 = D / 2, KS = D / 32, KTS = Lay::KTS;
  constexpr int TPW = NT == 8 ? 2 : 1;     // token tiles per wave
  constexpr int ND = NT == 2 ? 1 : 2;      // directions per wave
  constexpr float LOG2E = 1.44269504088896341f;
  extern __shared__ __align__(16) char smem[];
  float4* sE = (float4*)(smem + Lay::oE);
  float* sTot = (float*)(smem + Lay::oE);
  float* sZ = (float*)(smem + Lay::oZ);
  float* sK = (float*)(smem + Lay::oK);
  float* sT = (float*)(smem + Lay::oT);
  float* cN = (float*)(smem + Lay::oCs);
  float* cRr = cN + SP_CC;
  float* cD = cN + 2 * SP_CC;
  float4* sC4 = (float4*)(smem + Lay::oC4);
  float* sSS = (float*)(smem + Lay::oSS);
  float* sAG = (float*)(smem + Lay::oAG);
  float* sGd = (float*)(smem + Lay::oGd);
  float* sR = (float*)(smem + Lay::oR);
  float* sA = (float*)(smem + Lay::oA);
  float* sKap = (float*)(smem + Lay::oKap);
  float* sKn = (float*)(smem + Lay::oKn);
  int* sFlag = (int*)(smem + Lay::oFlag);
  int* sMap = (int*)(smem + Lay::oMap);
  uint8_t* sFl = (uint8_t*)(smem + Lay::oFl);
  int* XL = (int*)(smem + Lay::oL);        // [0, 32)   prefix cuts (child [0, x))
  int* XR = XL + 32;                       // [32, 64)  suffix cuts (child [x, n))
  int* XB = XL + 64;                       // [64, 96)  binary cuts
  int* posL = XL + 96;                     // index of XB[k] in XL
  int* posR = XL + 128;                    // index of XB[k] in XR
  int* meta = XL + 160;                    // nl, nr, nb, p, kmin, kmax, index of p in XL, of p+1 in XR,
                                           // forced extraction (singleton floor), work item, then (LV)
                                           // whether a node follows in this workgroup, and that node:
                                           // start, length | depth << 8 | node slot << 16, D, R, bound

  const int J = *n_slots;
  const int32_t* items = LV ? tv.long_items[cls] : tv.work;
  int32_t* next_ctr = LV ? tv.lv_ctr + 8 + cls : tv.wctr + 4 + cls;
  // the class's items: its list, or its part of the work list (the ends of the
  // classes, 0 for an empty one)
  const int e0 = LV ? 0 : tv.wctr[0], e1 = LV ? 0 : max(e0, tv.wctr[1]), e2 = LV ? 0 : max(e1, tv.wctr[2]);
  const int first = LV || cls == 0 ? 0 : (cls == 1 ? e0 : e1);
  const int nwork = LV ? (int)min((int64_t)tv.lv_ctr[cls], tv.long_cap) : (cls == 0 ? e0 : (cls == 1 ? e1 : e2));
  const uint32_t thi = LV && mode == BUILD_LONG ? (uint32_t)(tv.theta[0] >> 32) : 0u;
  const float sc2 = LOG2E / sqrtf((float)D);
  if (threadIdx.x == 0) {
    meta[9] = first + atomicAdd(next_ctr, 1);
    meta[10] = 0;
  }
  int64_t unit = 0;
  float w = 0.f;
  for (;;) {
    // per-lane indices are formed inside the loop: what the compiler derives from
    // them would else be held across items, past the register budget
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave = uni(tid >> 6), lane = tid & 63, i16 = lane & 15, g4 = lane >> 4;
    const int pi = lane & (H2 - 1);          // rotation pair of the lane
    const int rs = i16 & 3;
    // the wave's tiles and directions
    const int tile0 = NT == 2 ? (wave & 1) : wave;
    const int dir0 = NT == 2 ? (wave >> 1) : 0;
    sync_after_lds_stores();                 // meta[9] was stored at the end of the last pass
    const int wi = uni(meta[9]);
    // a node of the same unit that the last pass left for this workgroup
    const bool follows = LV && uni(meta[10]) != 0;
    int a0 = 0, word = 0;
    float Dv = 0.f, Rroot = 0.f;
    uint32_t bound = 0u;
    uint64_t Eadd = 0ull;
    if (follows) {
      a0 = uni(meta[11]);
      word = uni(meta[12]);
      Dv = __int_as_float(uni(meta[13]));
      Rroot = __int_as_float(uni(meta[14]));
      bound = (uint32_t)uni(meta[15]);
    }
    __syncthreads();
    if (!follows && wi >= nwork) break;
    // the next item, in flight while this one is processed (stored before the
    // barrier at the top of the next pass)
    int wnext = wi;
    if (!follows && tid == 0) wnext = first + atomicAdd(next_ctr, 1);
    if (LV && tid == 0) meta[10] = 0;
    auto publish_next = [&]() { if (tid == 0) meta[9] = wnext; };
    do {
    if (!follows) {
      // the work item: unit, the node's start, length, D and R, w and the key (LV:
      // the utility bound) of the op that creates it (one load)
      const int4 d0 = *(const int4*)(items + 8 * (int64_t)wi);
      const int4 d1 = *(const int4*)(items + 8 * (int64_t)wi + 4);
      unit = uni(d0.x);
      a0 = uni(d0.y);
      word = uni(d0.z);
      Dv = __int_as_float(uni(d0.w));
      Rroot = __int_as_float(uni(d1.x));
      w = __int_as_float(uni(d1.y));
      bound = (uint32_t)uni(d1.z);
      Eadd = mode == BUILD_ROOT_FULL ? 0ull : ((uint64_t)(uint32_t)uni(d1.w) << 32) | bound;
    }
    const int lg = (int)(unit / dm.J_cap), j = (int)(unit % dm.J_cap);
    const int l = lg / dm.G, g = lg % dm.G;
    const int n = word & 255;
    if (n < 2 || n > NM || j >= J) break;
    const int64_t base = (int64_t)lg * 2 * dm.N_c + 2 * (int64_t)a0;
    const uint32_t ord = (uint32_t)lg * (uint32_t)J + (uint32_t)j;
    const uint16_t* Kp = K + ((int64_t)lg * dm.T + a0) * D;
    const uint16_t* Vp = V + ((int64_t)lg * dm.T + a0) * D;
    const float* tokR = tv.tok_R + (int64_t)lg * dm.N_c + a0;
    // ---- writes the root and its children (local positions; LV: the node's
    // own choice, its children appended to the unit's nodes) ----
    auto write_tree = [&](int kind, int cut, int nkid, const int* ka, const int* kn, const float* kD,
                          const float* kR) {
      if constexpr (LV) {
        const int pos = atomicAdd(&tv.unit_nn[unit], nkid);
        float sd = 0.f;
        for (int k = 0; k < nkid; ++k) sd += kD[k];
        const float Us = utility(split_gain(w, Rroot, Dv, sd), nkid - 1);
        const uint32_t ub = min(bound, __float_as_uint(Us));
        const bool pass = mode == BUILD_LONG_FULL || ub >= thi;
        const int depth = (word >> 8) & 255;
        const int sl = tv.slots[j], nslot = tv.slots[j + 1] - sl;
        const int64_t ubase = (int64_t)lg * 2 * dm.N_c + 2 * (int64_t)sl;
        int keep = -1;                       // the child of the node's own class stays here (at most one)
        for (int k = 0; k < nkid; ++k)
          if (pass && kn[k] > NM / 2) keep = k;
        if (pos + nkid > 2 * nslot - 1) {    // a tree over n tokens has at most 2n - 1 nodes
          atomicOr(tv.status, STATUS_CAPACITY);
          return;
        }
        const int64_t s = ubase + ((word >> 16) & 255);
        tv.node_nch[s] = (uint8_t)nkid;
        tv.node_kind[s] = (uint8_t)kind;
        tv.node_cut[s] = a0 + cut;
        for (int k = 0; k < nkid; ++k) {
          const int64_t c = ubase + pos + k;
          tv.node_a[c] = a0 + ka[k];
          tv.node_n[c] = kn[k];
          tv.node_parent[c] = depth + 1;
          tv.node_nch[c] = 0;
          tv.node_kind[c] = 0;
          tv.node_cut[c] = -1;
          tv.node_D[c] = kD[k];
          tv.node_R[c] = kR[k];
          const int cw = kn[k] | ((depth + 1) << 8) | ((pos + k) << 16);
          if (k == keep) {
            meta[10] = 1;
            meta[11] = a0 + ka[k];
            meta[12] = cw;
            meta[13] = __float_as_int(kD[k]);
            meta[14] = __float_as_int(kR[k]);
            meta[15] = (int)ub;
          } else if (pass && kn[k] >= 2) {
            push_node(tv, dm, lg, make_int4((int)unit, a0 + ka[k], cw, __float_as_int(kD[k])),
                      make_int4(__float_as_int(kR[k]), __float_as_int(w), (int)ub, 0));
          }
        }
        return;
      }
      tv.node_child[base] = 1;
      tv.node_nch[base] = (uint8_t)nkid;
      tv.node_kind[base] = (uint8_t)kind;
      tv.node_cut[base] = a0 + cut;
      float sd = 0.f;
      for (int k = 0; k < nkid; ++k) {
        const int64_t s = base + 1 + k;
        tv.node_a[s] = a0 + ka[k];
        tv.node_n[s] = kn[k];
        tv.node_child[s] = -1;
        tv.node_parent[s] = 1;              // the depth: numbered at the end
        tv.node_nch[s] = 0;
        tv.node_kind[s] = 0;
        tv.node_cut[s] = -1;
        tv.node_D[s] = kD[k];
        tv.node_R[s] = kR[k];
        tv.sp_U[s] = 0.f;
        tv.sp_E[s] = 0;
        tv.sp_cost[s] = 0;
        tv.sp_exec[s] = 0;
        sd += kD[k];
      }
      if (mode != BUILD_ROOT_FULL) {        // the root's Split key, known now
        const float Us = utility(split_gain(w, Rroot, Dv, sd), nkid - 1);
        const uint64_t k = op_key(Us, ord * 256u + 1u);
        tv.sp_U[base] = Us;
        tv.sp_E[base] = k < Eadd ? k : Eadd;
        tv.sp_cost[base] = (uint8_t)(nkid - 1);
        tv.sp_exec[base] = 0;
      }
      tv.unit_nn[unit] = 1 + nkid;
    };
    if (n == 2) {                            // one cut, two singletons
      if (tid == 0) {
        const int ka[2] = {0, 1}, kn[2] = {1, 1};
        const float kD[2] = {0.f, 0.f}, kR[2] = {tokR[0], tokR[1]};
        write_tree(1, 1, 2, ka, kn, kD, kR);
      }
      break;
    }
    const int nt = (n + 15) >> 4;            // 16-token tiles

    // ---- loads: the tile's keys as rows of a product, token scalars, probe rows ----
    uint4 kf[TPW][KS];
#pragma unroll
    for (int m = 0; m < TPW; ++m) {
      const int t = min(16 * (tile0 + 4 * m) + i16, n - 1);
#pragma unroll
      for (int s = 0; s < KS; ++s) kf[m][s] = *(const uint4*)(Kp + (int64_t)t * D + 32 * s + 8 * g4);
    }
    float rv = 0.f, av = 0.f, kv = 0.f;
    uint8_t fl = 0;
    if (tid < n) {
      rv = tokR[tid];
      av = tv.tok_A[(int64_t)lg * dm.N_c + a0 + tid];
      kv = kappa[a0 + tid];
      if (tv.fl_flag) fl = tv.fl_flag[(int64_t)lg * dm.N_c + a0 + tid];
    }
    const float izc = lane < dm.W ? 1.0f / tv.probe_ZC[(int64_t)lg * dm.W + lane] : 0.f;
    const uint16_t* Qp = Q + ((int64_t)l * dm.H + (int64_t)g * dm.hpg) * dm.W * D;
    auto load_probes = [&](int pt, uint4* dst) {
      const int q0 = 16 * pt + i16, q = q0 < dm.W ? q0 : 0;
      const uint16_t* row = Qp + ((int64_t)(q % dm.hpg) * dm.W + q) * D + 8 * g4;
#pragma unroll
      for (int s = 0; s < KS; ++s) dst[s] = *(const uint4*)(row + 32 * s);
    };
    uint4 qf[4][KS];
    float mq4[4];                            // probe shift of probe 16 pt + i16; no such probe: e = 0
#pragma unroll
    for (int pt = 0; pt < 4; ++pt) {
      load_probes(pt, qf[pt]);
      const int q = 16 * pt + i16;
      mq4[pt] = q < dm.W ? tv.probe_m[(int64_t)lg * dm.W + q] * LOG2E : INFINITY;
    }
    if (tid < NM) {
      sR[tid] = rv;
      sA[tid] = av;
      sKap[tid] = kv;
      sFl[tid] = fl;
      sFlag[tid] = 0;
    }
    for (int t = tid; t < NM + 16; t += SP_T) sMap[t] = 0xffff;
    __syncthreads();
    // curvature position t proposes the cut t + 1: top k_curv by kappa over
    // [0, n-2], ties to the smaller t; midpoint floor(n/2)
    {
      constexpr int PP = NM >= 128 ? 2 : 4, PL = NM / PP;   // threads per position, positions each compares
      const int t = tid / PP, k0 = (tid % PP) * PL;
      if (dm.k_curv > 0 && t < n - 1) {
        const float kt = sKap[t];
        int rank = 0;
        for (int k = k0; k < min(k0 + PL, n - 1); k += 8) {
          const float4 a4 = *(const float4*)(sKap + k), b4 = *(const float4*)(sKap + k + 4);
          const float kk[8] = {a4.x, a4.y, a4.z, a4.w, b4.x, b4.y, b4.z, b4.w};
#pragma unroll
          for (int i = 0; i < 8; ++i) rank += (int)((k + i < n - 1) & ((kk[i] > kt) | ((kk[i] == kt) & (k + i < t))));
        }
        rank += __builtin_amdgcn_update_dpp(0, rank, 0xB1, 0xf, 0xf, false);
        if (PP == 4) rank += __builtin_amdgcn_update_dpp(0, rank, 0x4E, 0xf, 0xf, false);
        if (k0 == 0 && rank < dm.k_curv) sFlag[t + 1] = 1;
      }
      if (tid == SP_T - 1) sFlag[n / 2] = 1;
    }
    if (wave == 3) {                         // curvature range and extraction token
      float kmn = INFINITY, kmx = -INFINITY, best = -INFINITY, bestf = -INFINITY;
      int bi = 0x7fffffff, bf = 0x7fffffff;
      for (int t = lane; t < n; t += 64) {
        const float k = sKap[t];
        kmn = fminf(kmn, k);
        kmx = fmaxf(kmx, k);
        const float am = sA[t];
        if (am > best || (am == best && t < bi)) { best = am; bi = t; }
        // singleton floor: the candidate of largest token value (App. A.3 split choice)
        if (sFl[t] && (sR[t] > bestf || (sR[t] == bestf && t < bf))) { bestf = sR[t]; bf = t; }
      }
      wave_minmax(kmn, kmx);
      wave_argmax(best, bi);
      wave_argmax(bestf, bf);
      if (lane == 0) {
        // a node of three or more tokens holding a floor candidate is extracted
        // there, with no choice
        const bool forced = bf != 0x7fffffff;
        const int p = forced ? bf : bi;
        meta[3] = p < n ? p : 0;
        meta[4] = __float_as_int(kmn);
        meta[5] = __float_as_int(kmx);
        meta[8] = forced ? 1 : 0;
      }
    }
    __syncthreads();
    // binary cuts XB ascending (by ballot over the flags), then XL = XB + {p}
    // (p > 0) and XR = XB + {p+1} (p+1 < n)
    if (wave == 0) {
      const bool forced = meta[8] != 0;        // extraction only: no binary cut
      const bool f0 = !forced && lane >= 1 && lane < n && sFlag[lane < NM ? lane : 0];
      const bool f1 = NM > 64 && !forced && 64 + lane < n && sFlag[(64 + lane) & (NM - 1)];
      const uint64_t m0 = __ballot(f0), m1 = __ballot(f1);
      const uint64_t below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
      const int c0 = __popcll(m0);
      if (f0) XB[__popcll(m0 & below)] = lane;
      if (f1) XB[c0 + __popcll(m1 & below)] = 64 + lane;
      wave_lds_order();
      const int nb = c0 + __popcll(m1), p = meta[3];
      const bool on = lane < nb;
      const int xb = on ? XB[lane] : 0x7fffffff;
      const bool useP = p > 0, useQ = p + 1 < n;
      const uint64_t lessP = __ballot(on && xb < p), eqP = __ballot(on && xb == p);
      const uint64_t lessQ = __ballot(on && xb < p + 1), eqQ = __ballot(on && xb == p + 1);
      const bool insL = useP && eqP == 0ull, insR = useQ && eqQ == 0ull;
      const int cp = __popcll(lessP), cq = __popcll(lessQ);
      int pl = 0xff, pr = 0xff;
      if (on) {
        pl = lane + ((insL && xb > p) ? 1 : 0);
        pr = lane + ((insR && xb > p + 1) ? 1 : 0);
        XL[pl] = xb; posL[lane] = pl;
        XR[pr] = xb; posR[lane] = pr;
        ((uint8_t*)(sMap + xb))[0] = (uint8_t)pl;
        ((uint8_t*)(sMap + xb))[1] = (uint8_t)pr;
      }
      if (lane == 0) {
        if (insL) { XL[cp] = p; ((uint8_t*)(sMap + p))[0] = (uint8_t)cp; }
        if (insR) { XR[cq] = p + 1; ((uint8_t*)(sMap + p + 1))[1] = (uint8_t)cq; }
        meta[0] = nb + (insL ? 1 : 0);
        meta[1] = nb + (insR ? 1 : 0);
        meta[2] = nb;
        meta[6] = useP ? cp : -1;
        meta[7] = useQ ? cq : -1;
      }
    }

    // ---- the wave's tiles: probe exponentials, ||k||, k° and its tile sums ----
    float e[TPW][16];                        // lane = probe
    float k1[TPW][16], k2[TPW][16];          // lane = rotation pair
#pragma unroll
    for (int m = 0; m < TPW; ++m) {
      const int i = tile0 + 4 * m;
      if (i < nt) {
        f32x4 acc[4], kk = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) {
          acc[pt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int s = 0; s < KS; ++s) acc[pt] = mfma_bf16_16x16x32(pk8(kf[m][s]), pk8(qf[pt][s]), acc[pt]);
        }
#pragma unroll
        for (int s = 0; s < KS; ++s) kk = mfma_bf16_16x16x32(pk8(kf[m][s]), pk8(kf[m][s]), kk);
        mfma_done(kk);
        mfma_done(acc);
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) {
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc[pt][r] = 16 * i + 4 * g4 + r < n ? __builtin_amdgcn_exp2f(acc[pt][r] * sc2 - mq4[pt]) : 0.f;
          if (NT != 2 || dir0 == 0) sE[(i * 4 + pt) * 64 + lane] = make_float4(acc[pt][0], acc[pt][1], acc[pt][2], acc[pt][3]);
        }
        tiles_to_columns(acc, e[m]);
        // the diagonal of a tile sits at lane (i, i / 4), element i % 4
        if (g4 == (i16 >> 2) && (NT != 2 || dir0 == 0))
          sKn[16 * i + i16] = sqrtf(rs == 0 ? kk[0] : (rs == 1 ? kk[1] : (rs == 2 ? kk[2] : kk[3])));
        __builtin_amdgcn_sched_barrier(0);   // the products' operands are done with: their registers hold the rows below
        // k° turned back to the node's start a0: the table row of the offset
        // (R_{p~} R_{a0 + t}^{-1} = R_{p~ - a0} R_t^{-1}; rows below NMAX stay cached)
        uint16_t r1[16], r2[16];
        float cs[16], sn[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          const int tt = min(16 * i + t, n - 1);
          r1[t] = Kp[(int64_t)tt * D + pi];
          r2[t] = Kp[(int64_t)tt * D + pi + H2];
          cs[t] = cosT[tt * H2 + pi];
          sn[t] = sinT[tt * H2 + pi];
        }
        float t1 = 0.f, t2 = 0.f;
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          const float x = __uint_as_float((uint32_t)r1[t] << 16), y = __uint_as_float((uint32_t)r2[t] << 16);
          const bool on = 16 * i + t < n;
          k1[m][t] = on ? x * cs[t] + y * sn[t] : 0.f;
          k2[m][t] = on ? y * cs[t] - x * sn[t] : 0.f;
          t1 += k1[m][t];
          t2 += k2[m][t];
        }
        if (NT != 2 || dir0 == 0) {
          sT[(i * 2 + 0) * 64 + lane] = t1;
          sT[(i * 2 + 1) * 64 + lane] = t2;
        }
      } else {
#pragma unroll
        for (int t = 0; t < 16; ++t) { e[m][t] = 0.f; k1[m][t] = 0.f; k2[m][t] = 0.f; }
      }
    }
    __syncthreads();
    const int nl = uni(meta[0]), nr = uni(meta[1]), nb = uni(meta[2]), p = uni(meta[3]);

    // ---- key sums of the children, read off at the cuts (fp32, in the child's row).
    // The tile's running sum and the tiles before it are added at the cut only: an
    // outlier channel's rounding moves a logit by its full size, and sixteen additions
    // at the size of the whole sum cost a fifth of the gains' precision (rms error of
    // the gains above 16 tokens at 8B-128K 2.17e-9, so 1.83e-9) ----
#pragma unroll
    for (int m = 0; m < TPW; ++m) {
      const int i = tile0 + 4 * m;
      if (i < nt) {
#pragma unroll
        for (int d2 = 0; d2 < ND; ++d2) {
          const int dir = NT == 2 ? dir0 : d2;
          // the child that ends with token 16 i + i16 (prefix) or starts there (suffix)
          const int mine = dir == 0 ? sMap[16 * i + i16 + 1] & 255 : (sMap[16 * i + i16] >> 8) & 255;
          float b1 = 0.f, b2 = 0.f, s1 = 0.f, s2 = 0.f;   // the tiles before, and the tile's tokens
          for (int k = dir == 0 ? 0 : i + 1; k < (dir == 0 ? i : nt); ++k) {
            b1 += sT[(k * 2 + 0) * 64 + lane];
            b2 += sT[(k * 2 + 1) * 64 + lane];
          }
          auto emit = [&](int t) {
            const int c = __builtin_amdgcn_readlane(mine, t);
            if (c != 0xff) {
              float* row = sK + (c + dir * SP_CM) * KTS;
              row[pi] = b1 + s1;
              row[pi + H2] = b2 + s2;
            }
          };
          if (dir == 0) {
#pragma unroll
            for (int t = 0; t < 16; ++t) { s1 += k1[m][t]; s2 += k2[m][t]; emit(t); }
          } else {
#pragma unroll
            for (int t = 15; t >= 0; --t) { s1 += k1[m][t]; s2 += k2[m][t]; emit(t); }
          }
        }
      }
    }

    // ---- Y of the wave's tiles: Gram tile by Gram tile ----
    float y[TPW][ND][16];                    // lane = probe
    {
      f32x4 Y[TPW][ND][4], Yx[TPW][ND];
      uint4 vi[TPW][KS];
#pragma unroll
      for (int m = 0; m < TPW; ++m) {
        const int t = min(16 * (tile0 + 4 * m) + i16, n - 1);
#pragma unroll
        for (int s = 0; s < KS; ++s) vi[m][s] = *(const uint4*)(Vp + (int64_t)t * D + 32 * s + 8 * g4);
#pragma unroll
        for (int d2 = 0; d2 < ND; ++d2) {
          Yx[m][d2] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int pt = 0; pt < 4; ++pt) Y[m][d2][pt] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
      uint4 vn[KS];
#pragma unroll
      for (int s = 0; s < KS; ++s) vn[s] = *(const uint4*)(Vp + (int64_t)min(i16, n - 1) * D + 32 * s + 8 * g4);
#pragma unroll 1
      for (int jt = 0; jt < nt; ++jt) {
        uint4 vj[KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) vj[s] = vn[s];
        if (jt + 1 < nt) {                   // the next tile's values, in flight
          const int t = min(16 * (jt + 1) + i16, n - 1);
#pragma unroll
          for (int s = 0; s < KS; ++s) vn[s] = *(const uint4*)(Vp + (int64_t)t * D + 32 * s + 8 * g4);
        }
        float4 ej[4];
#pragma unroll
        for (int pt = 0; pt < 4; ++pt) ej[pt] = sE[(jt * 4 + pt) * 64 + lane];
        const float4 rj = *(const float4*)(sR + 16 * jt + 4 * g4);
        const float rr[4] = {rj.x, rj.y, rj.z, rj.w};
        float xj[4];                         // columns 0 and 1: R and 1 of the tile's tokens
#pragma unroll
        for (int r = 0; r < 4; ++r)
          xj[r] = i16 == 0 ? rr[r] : (i16 == 1 && 16 * jt + 4 * g4 + r < n ? 1.f : 0.f);
#pragma unroll
        for (int m = 0; m < TPW; ++m) {
          const int i = tile0 + 4 * m;
          if (i < nt) {
            f32x4 G = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) G = mfma_bf16_16x16x32(pk8(vj[s]), pk8(vi[m][s]), G);
            mfma_done(G);
            // lane (i16, g4): G[16 i + i16][16 jt + 4 g4 + r]
            if (jt == i && g4 == (i16 >> 2)) sGd[16 * i + i16] = rs == 0 ? G[0] : (rs == 1 ? G[1] : (rs == 2 ? G[2] : G[3]));
#pragma unroll
            for (int d2 = 0; d2 < ND; ++d2) {
              const int dir = NT == 2 ? dir0 : d2;
              if (dir == 0 ? jt <= i : jt >= i) {
                // the diagonal tile counts only the tokens before (after) the row's
                const uint32_t all = jt != i ? ~0u : 0u;
                float ga[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  const uint32_t keep = (uint32_t)((dir == 0 ? 4 * g4 + r - i16 : i16 - 4 * g4 - r) >> 31);
                  ga[r] = __uint_as_float(__float_as_uint(G[r]) & (keep | all));
                }
#pragma unroll
                for (int pt = 0; pt < 4; ++pt) {
                  Y[m][d2][pt] = mfma_f32_16x16x4(ga[0], ej[pt].x, Y[m][d2][pt]);
                  Y[m][d2][pt] = mfma_f32_16x16x4(ga[1], ej[pt].y, Y[m][d2][pt]);
                  Y[m][d2][pt] = mfma_f32_16x16x4(ga[2], ej[pt].z, Y[m][d2][pt]);
                  Y[m][d2][pt] = mfma_f32_16x16x4(ga[3], ej[pt].w, Y[m][d2][pt]);
                }
#pragma unroll
                for (int r = 0; r < 4; ++r) Yx[m][d2] = mfma_f32_16x16x4(ga[r], xj[r], Yx[m][d2]);
              }
            }
          }
        }
      }
#pragma unroll
      for (int m = 0; m < TPW; ++m)
#pragma unroll
        for (int d2 = 0; d2 < ND; ++d2) {
          const int i = tile0 + 4 * m, dir = NT == 2 ? dir0 : d2;
          mfma_done(Yx[m][d2]);
          mfma_done(Y[m][d2]);
          tiles_to_columns(Y[m][d2], y[m][d2]);
          // lane (0 or 1, g4): the sums against R or 1 of tokens 4 g4 + r
          if (i < nt && i16 < 2)
            *(float4*)(sAG + (2 * dir + i16) * NM + 16 * i + 4 * g4) =
                make_float4(Yx[m][d2][0], Yx[m][d2][1], Yx[m][d2][2], Yx[m][d2][3]);
        }
    }
    __syncthreads();

    if (tid < SP_CC) {
      const int c = tid < SP_CM ? tid : tid - SP_CM;
      cN[tid] = tid < SP_CM ? (c < nl ? (float)XL[c] : 0.f) : (c < nr ? (float)(n - XR[c]) : 0.f);
      cD[tid] = 0.f;
    }
    // ---- waves 0-2, one tile of children each: k~ = RoPE(mean k°, p)
    // (eq:app_rope_prototype) as the product's row operand in three bf16 parts (lane:
    // child i16, both halves of its rotation pairs), its logits against every probe ----
    if (wave < 3) {
      const int gr0 = 16 * wave + i16, gr = gr0 < SP_CC ? gr0 : 0;
      const int c = gr < SP_CM ? gr : gr - SP_CM;
      const bool live = gr < SP_CM ? c < nl : c < nr;
      const int x0 = live && gr >= SP_CM ? XR[c] : 0, x1 = !live ? 0 : (gr < SP_CM ? XL[c] : n);
      const int len = x1 - x0;
      const int pp = len >= 2 ? round_half_even_mid(a0 + x0, a0 + x1) - a0 : 0;
      const float nd = (float)max(len, 1), inv = 1.0f / nd;
      const float* row = sK + gr * KTS + 8 * g4;
      const float* ct = cosT + pp * H2 + 8 * g4;
      const float* st = sinT + pp * H2 + 8 * g4;
      uint4 kp[KS][3];
      float ss = 0.f;
#pragma unroll
      for (int s = 0; s < KS / 2; ++s) {
        float o[2][8];
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
          const float4 a4 = *(const float4*)(row + 32 * s + h), b4 = *(const float4*)(row + 32 * s + H2 + h);
          const float4 c4 = *(const float4*)(ct + 32 * s + h), s4 = *(const float4*)(st + 32 * s + h);
          const float av[4] = {a4.x, a4.y, a4.z, a4.w}, bv[4] = {b4.x, b4.y, b4.z, b4.w};
          const float cv[4] = {c4.x, c4.y, c4.z, c4.w}, sv[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const float m1 = len >= 2 ? quotient(av[r], nd, inv) : 0.f, m2 = len >= 2 ? quotient(bv[r], nd, inv) : 0.f;
            ss += m1 * m1 + m2 * m2;
            o[0][h + r] = m1 * cv[r] - m2 * sv[r];
            o[1][h + r] = m2 * cv[r] + m1 * sv[r];
          }
        }
        split3x8(o[0], kp[s]);
        split3x8(o[1], kp[s + KS / 2]);
      }
      ss = col_sum4(ss);
      if (g4 == 0 && gr0 < SP_CC) sSS[gr0] = ss;
#pragma unroll
      for (int pt = 0; pt < 4; ++pt) {
        uint4 qz[KS];
        load_probes(pt, qz);
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        // the low parts first: the matrix cores truncate at the size of the sum so far
#pragma unroll
        for (int part = 2; part >= 0; --part)
#pragma unroll
          for (int s = 0; s < KS; ++s) acc = mfma_bf16_16x16x32(pk8(kp[s][part]), pk8(qz[s]), acc);
        mfma_done(acc);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int zr = 16 * wave + 4 * g4 + r;
          if (zr < SP_CC) sZ[zr * 64 + 16 * pt + i16] = __builtin_amdgcn_exp2f(acc[r] * sc2 - mq4[pt]);
        }
      }
    }
    // ---- sum R, mean ||k|| and ||v~||^2 of every child (eq:app_value_prototype): with
    // w_t = R_t + beta, ||sum w_t v_t||^2 = RR + 2 beta RG + beta^2 GG, each the sum over
    // the child of a per-token increment; wave 3, one direction after the other, the
    // tokens in the order of its scan, two per lane where there are 128 ----
    if (wave == 3) {
      constexpr int TPL = NM > 64 ? 2 : 1;
#pragma unroll 1
      for (int dir = 0; dir < 2; ++dir) {
      float x[TPL][5];
#pragma unroll
      for (int e2 = 0; e2 < TPL; ++e2) {
        const int o = TPL * lane + e2;
        const int t = dir == 0 ? o : NM - 1 - o;
#pragma unroll
        for (int k = 0; k < 5; ++k) x[e2][k] = 0.f;
        if (t >= 0 && t < n) {
          const float R = sR[t], gd = sGd[t], at = sAG[2 * dir * NM + t], gt = sAG[(2 * dir + 1) * NM + t];
          x[e2][0] = R * (2.f * at + gd * R);
          x[e2][1] = (R * gt + at) + R * gd;
          x[e2][2] = 2.f * gt + gd;
          x[e2][3] = R;
          x[e2][4] = sKn[t];
        }
      }
      float s[TPL][5];
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        if (TPL == 2) {
          const float in = wave_scan(x[0][k] + x[TPL - 1][k]);
          s[TPL - 1][k] = in;
          const float ex = __shfl_up(in, 1, 64);
          s[0][k] = (lane > 0 ? ex : 0.f) + x[0][k];
        } else {
          s[0][k] = wave_scan(x[0][k]);
        }
      }
      const int c = lane < SP_CM ? lane : 0;
      const int gc = dir * SP_CM + c;
      const bool live = lane < SP_CM && (dir == 0 ? c < nl : c < nr);
      const int xc = live ? (dir == 0 ? XL[c] : XR[c]) : 0;
      const int len = live ? (dir == 0 ? xc : n - xc) : 0;
      // the last token of the child in scan order
      const int o = live ? (dir == 0 ? xc - 1 : NM - 1 - xc) : 0;
      float v[5];
#pragma unroll
      for (int k = 0; k < 5; ++k) {
        const float va = __shfl(s[0][k], o / TPL, 64), vb = __shfl(s[TPL - 1][k], o / TPL, 64);
        v[k] = (o % TPL) ? vb : va;
      }
      if (live) {
        const float nch = (float)len, inv = 1.0f / nch;
        const float beta = dm.beta_frac * v[3] * inv;
        const float iden = 1.0f / (v[3] + nch * beta + dm.eps);
        cRr[gc] = v[3];
        sC4[gc] = make_float4(beta, iden, (v[0] + beta * (2.f * v[1] + beta * v[2])) * (iden * iden), v[4] * inv);
      }
      }
    }
    // ---- lane = probe: sums over each tile of the increments
    //   e_t (Z), e_t (Y_t + u_t) (||M||^2), R_t u_t + e_t a_t and u_t + e_t g_t
    //   (<M, sum R v> and <M, sum v>), u_t = Y_t + e_t G_tt ----
    auto step = [&](float et, float yt, float R, float gd, float at, float gt, float& Z, float& S, float& P, float& Qs) {
      const float u = yt + et * gd;
      Z += et;
      S += et * (yt + u);
      P += R * u + et * at;
      Qs += u + et * gt;
    };
#pragma unroll
    for (int m = 0; m < TPW; ++m) {
      const int i = tile0 + 4 * m;
      if (i < nt) {
#pragma unroll
        for (int d2 = 0; d2 < ND; ++d2) {
          const int dir = NT == 2 ? dir0 : d2;
          const float* ag = sAG + 2 * dir * NM + 16 * i;
          float Z = 0.f, S = 0.f, P = 0.f, Qs = 0.f;
#pragma unroll
          for (int b4 = 0; b4 < 4; ++b4) {
            const float4 R4 = *(const float4*)(sR + 16 * i + 4 * b4), G4 = *(const float4*)(sGd + 16 * i + 4 * b4);
            const float4 A4 = *(const float4*)(ag + 4 * b4), O4 = *(const float4*)(ag + NM + 4 * b4);
            // tokens past the node: e = 0 but Y is not; they count for nothing
            const int t0 = 16 * i + 4 * b4;
            if (t0 + 0 < n) step(e[m][4 * b4 + 0], y[m][d2][4 * b4 + 0], R4.x, G4.x, A4.x, O4.x, Z, S, P, Qs);
            if (t0 + 1 < n) step(e[m][4 * b4 + 1], y[m][d2][4 * b4 + 1], R4.y, G4.y, A4.y, O4.y, Z, S, P, Qs);
            if (t0 + 2 < n) step(e[m][4 * b4 + 2], y[m][d2][4 * b4 + 2], R4.z, G4.z, A4.z, O4.z, Z, S, P, Qs);
            if (t0 + 3 < n) step(e[m][4 * b4 + 3], y[m][d2][4 * b4 + 3], R4.w, G4.w, A4.w, O4.w, Z, S, P, Qs);
          }
          float* tot = sTot + ((dir * NT + i) * 4) * 64 + lane;
          tot[0] = Z;
          tot[64] = S;
          tot[128] = P;
          tot[192] = Qs;
        }
      }
    }
    __syncthreads();

    // ---- lane = probe: the running sums over each child and D_q at its cut
    // (eq:app_node_and_drop_distortion) ----
    {
      const float invW = 1.0f / (float)dm.W;
#pragma unroll
      for (int m = 0; m < TPW; ++m) {
        const int i = tile0 + 4 * m;
        if (i < nt) {
#pragma unroll
          for (int d2 = 0; d2 < ND; ++d2) {
            const int dir = NT == 2 ? dir0 : d2;
            const int mine = dir == 0 ? sMap[16 * i + i16 + 1] & 255 : (sMap[16 * i + i16] >> 8) & 255;
            // the tile's last cut in scan order: nothing is read after it
            const uint64_t has = __ballot(mine != 0xff) & 0xffffull;
            if (has == 0ull) continue;
            const int lastt = dir == 0 ? 63 - __builtin_clzll(has) : __builtin_ctzll(has);
            const float* ag = sAG + 2 * dir * NM + 16 * i;
            // the tiles before, and the tile's tokens (added at the cut only, as the keys)
            float Zb = 0.f, Sb = 0.f, Pb = 0.f, Qb = 0.f, Z = 0.f, S = 0.f, P = 0.f, Qs = 0.f;
            for (int k = dir == 0 ? 0 : i + 1; k < (dir == 0 ? i : nt); ++k) {
              const float* tot = sTot + ((dir * NT + k) * 4) * 64 + lane;
              Zb += tot[0];
              Sb += tot[64];
              Pb += tot[128];
              Qb += tot[192];
            }
            auto child = [&](int t) {
              const int c0 = __builtin_amdgcn_readlane(mine, t);
              const int x = 16 * i + t;
              if (c0 == 0xff || x == (dir == 0 ? 0 : n - 1)) return;     // a singleton has D = 0
              const int c = c0 + dir * SP_CM;
              const float4 c4 = sC4[c];
              // coherence and multiplicity (eq:app_effective_multiplicity)
              const float nch = (float)(dir == 0 ? x + 1 : n - x), km = c4.w + dm.eps;
              const float me = fminf(fmaxf(nch * (sSS[c] / (km * km)), 1.0f), nch);
              const float z = lane < dm.W ? sZ[c * 64 + lane] * me : 0.f;
              const float Zt = Zb + Z, St = Sb + S;
              const float xv = ((Pb + P) + c4.x * (Qb + Qs)) * c4.y;
              const float s1 = fmaxf(St + z * (z * c4.z - 2.f * xv), 0.f);
              const float dz = Zt - z;
              const float Dq = dm.lam_Z * dz * dz * __builtin_amdgcn_rcpf(Zt * Zt + dm.eps) +
                               dm.lam_M * s1 * __builtin_amdgcn_rcpf(St + dm.eps);
              const float con = wave_sum_dpp((Zt * izc) * Dq);
              if (lane == 0) cD[c] = con * invW;
            };
            auto token = [&](int t, float R, float gd, float at, float gt) {
              if ((dir == 0 ? t <= lastt : t >= lastt) && 16 * i + t < n) {
                step(e[m][t], y[m][d2][t], R, gd, at, gt, Z, S, P, Qs);
                child(t);
              }
            };
            if (dir == 0) {
#pragma unroll
              for (int b4 = 0; b4 < 4; ++b4) {
                const float4 R4 = *(const float4*)(sR + 16 * i + 4 * b4), G4 = *(const float4*)(sGd + 16 * i + 4 * b4);
                const float4 A4 = *(const float4*)(ag + 4 * b4), O4 = *(const float4*)(ag + NM + 4 * b4);
                token(4 * b4 + 0, R4.x, G4.x, A4.x, O4.x);
                token(4 * b4 + 1, R4.y, G4.y, A4.y, O4.y);
                token(4 * b4 + 2, R4.z, G4.z, A4.z, O4.z);
                token(4 * b4 + 3, R4.w, G4.w, A4.w, O4.w);
              }
            } else {
#pragma unroll
              for (int b4 = 3; b4 >= 0; --b4) {
                const float4 R4 = *(const float4*)(sR + 16 * i + 4 * b4), G4 = *(const float4*)(sGd + 16 * i + 4 * b4);
                const float4 A4 = *(const float4*)(ag + 4 * b4), O4 = *(const float4*)(ag + NM + 4 * b4);
                token(4 * b4 + 3, R4.w, G4.w, A4.w, O4.w);
                token(4 * b4 + 2, R4.z, G4.z, A4.z, O4.z);
                token(4 * b4 + 1, R4.y, G4.y, A4.y, O4.y);
                token(4 * b4 + 0, R4.x, G4.x, A4.x, O4.x);
              }
            }
          }
        }
      }
    }
    __syncthreads();
    // ---- decision (fp32): best binary cut (smaller cut wins ties), then extraction ----
    if (wave == 0) {
      const float kmn = __int_as_float(meta[4]), kmx = __int_as_float(meta[5]);
      const float kr = kmx - kmn;
      float best = -INFINITY;
      int bk = 0x7fffffff;
      if (lane < nb) {
        const int x = XB[lane];
        const float kh = kr > 0.f ? (sKap[x - 1] - kmn) / kr : 0.f;
        best = ((Dv - cD[posL[lane]]) - cD[SP_CM + posR[lane]]) + dm.lam_kappa * kh;
        bk = lane;
      }
      wave_argmax(best, bk);
      if (lane == 0) {
        const int iL = meta[6], iR = meta[7];
        float dsum = 0.f;
        int nkid = 1;
        if (p > 0) { dsum += cD[iL]; ++nkid; }
        if (p + 1 < n) { dsum += cD[SP_CM + iR]; ++nkid; }
        const float gext = (Dv - dsum) / (float)(nkid - 1);
        int ka[3], kn[3];
        float kD[3], kR[3];
        if (best >= gext && bk < nb) {
          const int bx = XB[bk];
          ka[0] = 0; kn[0] = bx; kD[0] = cD[posL[bk]]; kR[0] = cRr[posL[bk]];
          ka[1] = bx; kn[1] = n - bx; kD[1] = cD[SP_CM + posR[bk]]; kR[1] = cRr[SP_CM + posR[bk]];
          write_tree(1, bx, 2, ka, kn, kD, kR);
        } else {
          int c = 0;
          if (p > 0) { ka[c] = 0; kn[c] = p; kD[c] = cD[iL]; kR[c] = cRr[iL]; ++c; }
          ka[c] = p; kn[c] = 1; kD[c] = 0.f; kR[c] = sR[p]; ++c;
          if (p + 1 < n) { ka[c] = p + 1; kn[c] = n - p - 1; kD[c] = cD[SP_CM + iR]; kR[c] = cRr[SP_CM + iR]; ++c; }
          write_tree(2, p, c, ka, kn, kD, kR);
        }
      }
    }
    } while (0);
    publish_next();
  }
}

// one class of nodes: cls 0, 1, 2 -- up to 128, 64 and 32 tokens
static hipError_t launch_split(const Dims& dm, int mode, int cls, const void* K, const void* V, const void* Q,
                               const float* cosT, const float* sinT, const int32_t* n_slots, const float* kappa,
                               const TreeView& tv, int cus, hipStream_t st) {
  const Dims* dmp = (const Dims*)tv.kargs;
  const TreeView* tvp = (const TreeView*)((const char*)tv.kargs + 512);
#define GKV_SP1(DD, NN, LL)                                                                                   \
  do {                                                                                                        \
    auto fn = k_split<DD, NN, LL>;                                                                            \
    constexpr int lds = SpLds<DD, NN>::bytes;                                                                 \
    const hipError_t e0 = hipFuncSetAttribute((const void*)fn, hipFuncAttributeMaxDynamicSharedMemorySize, lds); \
    if (e0 != hipSuccess) return e0;                                                                          \
    hipLaunchKernelGGL(fn, dim3((unsigned)((NN == 8 ? 2 : 3) * cus)), dim3(SP_T), lds, st, dmp, mode, cls,    \
                       (const uint16_t*)K, (const uint16_t*)V, (const uint16_t*)Q, cosT, sinT, n_slots, kappa, tvp); \
  } while (0)
#define GKV_SP(DD, NN) do { if (lv) GKV_SP1(DD, NN, true); else GKV_SP1(DD, NN, false); } while (0)
  const bool lv = mode == BUILD_LONG || mode == BUILD_LONG_FULL;
  if (dm.d == 128) {
    if (cls == 0) GKV_SP(128, 8); else if (cls == 1) GKV_SP(128, 4); else GKV_SP(128, 2);
  } else if (dm.d == 64) {
    if (cls == 0) GKV_SP(64, 8); else if (cls == 1) GKV_SP(64, 4); else GKV_SP(64, 2);
  } else {
    return hipErrorInvalidValue;
  }
#undef GKV_SP
#undef GKV_SP1
  return hipGetLastError();
}

hipError_t launch_split_roots(const Dims& dm, int mode, const void* K, const void* V, const void* Q, const float* cosT,
                              const float* sinT, const int32_t* n_slots, const float* kappa, const TreeView& tv,
                              int cus, hipStream_t st) {
  for (int cls = 0; cls < LONG_CLASSES; ++cls) {
    const hipError_t e = launch_split(dm, mode, cls, K, V, Q, cosT, sinT, n_slots, kappa, tv, cus, st);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_split_long(const Dims& dm, bool full, const void* K, const void* V, const void* Q,
                             const float* cosT, const float* sinT, const int32_t* n_slots, const float* kappa,
                             const TreeView& tv, int cus, hipStream_t st) {
  return launch_split_roots(dm, full ? BUILD_LONG_FULL : BUILD_LONG, K, V, Q, cosT, sinT, n_slots, kappa, tv, cus, st);
}

}  // namespace gkv
