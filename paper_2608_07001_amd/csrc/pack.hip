// Ragged compressed cache (App. A.5 "Frontier updates and physical packing",
// eq:app_frontier_update).  A node is on its tree's frontier when the op that
// created it executed (Add for the root, the parent's Split otherwise) and its
// own Split did not.  Per (l, g) the output holds, in ascending position, each
// frontier node -- a singleton as its original K/V with its position and
// log-multiplicity 0, any other node as its prototype (k~, v~ rounded to the
// cache dtype, p_v, log m_eff; App. A.3) -- followed by the r recent-window
// tokens.  A root's prototype is the one the tree build stored; deeper nodes
// are recomputed from K and V.  Offsets are a CSR over (l, g).
#include "common.h"

namespace gkv {

struct PackWs {
  int32_t* ucount;   // [unit_cap] frontier nodes per unit
  int64_t* uoff;     // [unit_cap] offset of the unit inside its (l, g) range
};

size_t pack_ws_bytes(const Dims& dm) {
  const int64_t units = (int64_t)dm.L * dm.G * dm.J_cap;
  return (size_t)units * (4 + 8) + 64;
}

static PackWs pack_view(void* ws, const Dims& dm) {
  const int64_t units = (int64_t)dm.L * dm.G * dm.J_cap;
  PackWs p;
  p.uoff = (int64_t*)ws;
  p.ucount = (int32_t*)((char*)ws + units * 8);
  return p;
}

__device__ __forceinline__ bool on_frontier(const TreeView& tv, int64_t u, int64_t base, int i) {
  const int par = tv.node_parent[base + i];
  const bool created = par < 0 ? tv.add_exec[u] != 0 : tv.sp_exec[base + par] != 0;
  if (!created) return false;
  return tv.node_nch[base + i] == 0 || tv.sp_exec[base + i] == 0;
}

// a wave counts PC_U units, one after the other (nodes across the lanes: one
// thread per unit read a cache line for every node)
constexpr int PC_U = 8;
__global__ __launch_bounds__(256) void k_pack_count(Dims dm, TreeView tv, PackWs pw) {
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int64_t units = (int64_t)dm.L * dm.G * dm.J_cap;
  const int64_t u0 = ((int64_t)blockIdx.x * 4 + wave) * PC_U;
  const int J = *tv.nslots;
  // a unit whose Add was not executed has nothing on its frontier, one that is a lone root has it
  int nn = 0, c = 0;
  const int64_t u = u0 + lane;
  const bool mine = lane < PC_U && u < units;
  if (mine && (int)(u % dm.J_cap) < J && tv.add_exec[u] != 0) {
    nn = tv.unit_nn[u];
    c = nn == 1 ? 1 : 0;
  }
  uint64_t more = __ballot(nn > 1);
  while (more != 0ull) {
    const int q = __builtin_ctzll(more);
    more &= more - 1;
    const int n = __builtin_amdgcn_readlane(nn, q);
    const int64_t uq = u0 + q;
    const int64_t base = (uq / dm.J_cap) * 2 * dm.N_c + 2 * (int64_t)tv.slots[uq % dm.J_cap];
    int k = 0;
    for (int i0 = 0; i0 < n; i0 += 64) k += __popcll(__ballot(i0 + lane < n && on_frontier(tv, uq, base, i0 + lane)));
    if (lane == q) c = k;
  }
  if (mine) pw.ucount[u] = c;
}

// per (l, g): exclusive scan over its units, then the (l, g) entry count
__global__ __launch_bounds__(256) void k_pack_scan_units(Dims dm, TreeView tv, PackWs pw, int64_t* counts) {
  const int lg = blockIdx.x;
  const int J = *tv.nslots;
  __shared__ int64_t part[256];
  __shared__ int64_t carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  for (int j0 = 0; j0 < J; j0 += 256) {
    const int j = j0 + threadIdx.x;
    const int64_t v = j < J ? pw.ucount[(int64_t)lg * dm.J_cap + j] : 0;
    part[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < 256; o <<= 1) {          // inclusive Hillis-Steele scan
      const int64_t x = threadIdx.x >= o ? part[threadIdx.x - o] : 0;
      __syncthreads();
      part[threadIdx.x] += x;
      __syncthreads();
    }
    if (j < J) pw.uoff[(int64_t)lg * dm.J_cap + j] = carry + part[threadIdx.x] - v;
    __syncthreads();
    if (threadIdx.x == 0) carry += part[255];
    __syncthreads();
  }
  if (threadIdx.x == 0) counts[lg] = carry + dm.r;
}

__global__ void k_pack_scan_lg(Dims dm, const int64_t* __restrict__ counts, int64_t* offsets) {
  if (threadIdx.x != 0) return;
  int64_t acc = 0;
  offsets[0] = 0;
  for (int i = 0; i < dm.L * dm.G; ++i) {
    acc += counts[i];
    offsets[i + 1] = acc;
  }
}

// one wave per unit
template <typename T, int D>
__global__ __launch_bounds__(64) void k_pack_emit(Dims dm, const T* __restrict__ K, const T* __restrict__ V,
                                                  const float* __restrict__ cosT, const float* __restrict__ sinT,
                                                  TreeView tv, PackWs pw, const int64_t* __restrict__ offsets,
                                                  T* __restrict__ Ko, T* __restrict__ Vo, int32_t* __restrict__ po,
                                                  float* __restrict__ lo) {
  constexpr int H2 = D / 2;
  constexpr int DL = (D + 63) / 64;   // dims per lane
  const int64_t u = blockIdx.x;
  const int lg = (int)(u / dm.J_cap), j = (int)(u % dm.J_cap);
  const int J = *tv.nslots;
  if (j >= J) return;
  const int lane = threadIdx.x;
  const int64_t base = (int64_t)lg * 2 * dm.N_c + 2 * (int64_t)tv.slots[j];
  const int nn = tv.unit_nn[u];
  const int cnt = pw.ucount[u];
  if (cnt < 1) return;
  __shared__ uint32_t mask[NMAX / 32];      // starts of the frontier nodes, relative to the slot's
  __shared__ int at[NMAX];                  // by start: node index | length << 16
  __shared__ int list[NMAX];                // by rank: start | length << 8 | (the root) << 16
  __shared__ float mk[D];
  if (lane < NMAX / 32) mask[lane] = 0u;
  __syncthreads();
  // the output order is that of the starts: ranks are population counts
  const int s0 = tv.slots[j];
  for (int i = lane; i < nn; i += 64)
    if (on_frontier(tv, u, base, i)) {
      const int a = (tv.node_a[base + i] - s0) & (NMAX - 1);
      atomicOr(&mask[a >> 5], 1u << (a & 31));
      at[a] = i | (tv.node_n[base + i] << 16);
    }
  __syncthreads();
#pragma unroll
  for (int h = 0; h < NMAX / 64; ++h) {
    const int a = lane + 64 * h;
    if ((mask[a >> 5] >> (a & 31)) & 1u) {
      int rank = __popc(mask[a >> 5] & ((1u << (a & 31)) - 1u));
      for (int k = 0; k < (a >> 5); ++k) rank += __popc(mask[k]);
      list[rank] = a | ((at[a] >> 16) << 8) | ((at[a] & 0xffff) == 0 ? 1 << 16 : 0);
    }
  }
  __syncthreads();
  const int64_t out0 = offsets[lg] + pw.uoff[u];
  const T* Kp = K + (int64_t)lg * dm.T * D;
  const T* Vp = V + (int64_t)lg * dm.T * D;
  const float* Rt = tv.tok_R + (int64_t)lg * dm.N_c;
  // singletons: the original rows, 16 bytes a lane, several entries at a time
  constexpr int LPR = D * (int)sizeof(T) / 16, EPS = 64 / LPR;
  for (int r0 = 0; r0 < cnt; r0 += EPS) {
    const int r = r0 + lane / LPR, c = lane % LPR;
    const int it = r < cnt ? list[r] : 0;
    if (((it >> 8) & 255) != 1) continue;
    const int64_t o = out0 + r;
    if (o >= dm.B_total) { atomicOr(tv.status, STATUS_CAPACITY); continue; }
    const int a = s0 + (it & 255);
    ((uint4*)(Ko + o * D))[c] = ((const uint4*)(Kp + (int64_t)a * D))[c];
    ((uint4*)(Vo + o * D))[c] = ((const uint4*)(Vp + (int64_t)a * D))[c];
    if (c == 0) { po[o] = a; lo[o] = 0.f; }
  }
  for (int r = 0; r < cnt; ++r) {
    const int it = __builtin_amdgcn_readfirstlane(list[r]);
    const int a = s0 + (it & 255), n = (it >> 8) & 255;
    const int64_t o = out0 + r;
    if (n == 1) continue;
    if (o >= dm.B_total) { if (lane == 0) atomicOr(tv.status, STATUS_CAPACITY); break; }
    if (it >> 16) {                           // the root: the prototype the build stored
      const T* pr = (const T*)tv.proto + u * 2 * D;
      for (int c = lane; c < D; c += 64) {
        Ko[o * D + c] = pr[c];
        Vo[o * D + c] = pr[D + c];
      }
      if (lane == 0) { po[o] = round_half_even_mid(a, a + n); lo[o] = tv.proto_logm[u]; }
      continue;
    }
    float sk[DL], srv[DL], sv[DL];
#pragma unroll
    for (int k = 0; k < DL; ++k) { sk[k] = 0.f; srv[k] = 0.f; sv[k] = 0.f; }
    float sr = 0.f, skn = 0.f;
    constexpr int TU = 4;                     // tokens in flight
    for (int t0 = a; t0 < a + n; t0 += TU) {
      float x[TU][DL], y[TU][DL], v[TU][DL], c[TU][DL], s[TU][DL], rt[TU], kk[TU];
#pragma unroll
      for (int q = 0; q < TU; ++q) {
        const int t = t0 + q < a + n ? t0 + q : a + n - 1;
        rt[q] = Rt[t];
#pragma unroll
        for (int k = 0; k < DL; ++k) {
          const int i2 = lane + 64 * k < D ? lane + 64 * k : 0;
          const int ih = i2 < H2 ? i2 : i2 - H2;
          const int ip = i2 < H2 ? i2 + H2 : i2 - H2;
          c[q][k] = cosT[(int64_t)t * H2 + ih];
          s[q][k] = sinT[(int64_t)t * H2 + ih];
          x[q][k] = ldf(Kp, (int64_t)t * D + i2);
          y[q][k] = ldf(Kp, (int64_t)t * D + ip);
          v[q][k] = ldf(Vp, (int64_t)t * D + i2);
        }
      }
#pragma unroll
      for (int q = 0; q < TU; ++q) {
        kk[q] = 0.f;
#pragma unroll
        for (int k = 0; k < DL; ++k)
          if (lane + 64 * k < D) kk[q] += x[q][k] * x[q][k];
        kk[q] = wave_sum_dpp(kk[q]);
      }
#pragma unroll
      for (int q = 0; q < TU; ++q) {
        if (t0 + q >= a + n) break;
#pragma unroll
        for (int k = 0; k < DL; ++k) {
          const int i2 = lane + 64 * k;
          if (i2 < D) {
            sk[k] += i2 < H2 ? x[q][k] * c[q][k] + y[q][k] * s[q][k] : x[q][k] * c[q][k] - y[q][k] * s[q][k];
            srv[k] += rt[q] * v[q][k];
            sv[k] += v[q][k];
          }
        }
        skn += sqrtf(kk[q]);
        sr += rt[q];
      }
    }
    const float inv = 1.0f / (float)n;
    float ss = 0.f;
#pragma unroll
    for (int k = 0; k < DL; ++k) {
      const int i2 = lane + 64 * k;
      if (i2 < D) { mk[i2] = sk[k] * inv; ss += mk[i2] * mk[i2]; }
    }
    ss = wave_sum_dpp(ss);
    __syncthreads();
    const float coh = sqrtf(ss) / (skn * inv + dm.eps);
    const float me = fminf(fmaxf((float)n * coh * coh, 1.0f), (float)n);
    int s2 = 2 * a + n - 1;
    int p = (s2 & 1) == 0 ? (s2 >> 1) : (((s2 >> 1) & 1) ? (s2 >> 1) + 1 : (s2 >> 1));
    const float beta = dm.beta_frac * sr * inv;
    const float den = sr + (float)n * beta + dm.eps;
#pragma unroll
    for (int k = 0; k < DL; ++k) {
      const int i2 = lane + 64 * k;
      if (i2 < D) {
        const int ih = i2 < H2 ? i2 : i2 - H2;
        const float c = cosT[(int64_t)p * H2 + ih], s = sinT[(int64_t)p * H2 + ih];
        const float kt = i2 < H2 ? mk[i2] * c - mk[i2 + H2] * s : mk[i2] * c + mk[i2 - H2] * s;
        stf(Ko, o * D + i2, kt);
        stf(Vo, o * D + i2, (srv[k] + beta * sv[k]) / den);
      }
    }
    if (lane == 0) { po[o] = p; lo[o] = logf(me); }
    __syncthreads();
  }
}

// recent window: tokens [N_c, N_ctx) after the frontier entries of each (l, g)
template <typename T>
__global__ void k_pack_window(Dims dm, const T* __restrict__ K, const T* __restrict__ V,
                              const int64_t* __restrict__ offsets, T* Ko, T* Vo, int32_t* po, float* lo) {
  const int lg = blockIdx.y;
  const int k = blockIdx.x;
  const int64_t t = dm.N_c + k;
  const int64_t o = offsets[lg + 1] - dm.r + k;
  if (o < 0 || o >= dm.B_total) return;
  for (int c = threadIdx.x; c < dm.d; c += blockDim.x) {
    Ko[o * dm.d + c] = K[((int64_t)lg * dm.T + t) * dm.d + c];
    Vo[o * dm.d + c] = V[((int64_t)lg * dm.T + t) * dm.d + c];
  }
  if (threadIdx.x == 0) { po[o] = (int32_t)t; lo[o] = 0.f; }
}

hipError_t launch_pack(const Dims& dm, const void* K, const void* V, const float* cosT, const float* sinT,
                       const TreeView& tv, int64_t* offsets, int64_t* counts, void* K_out, void* V_out,
                       int32_t* pos_out, float* logm_out, void* ws, hipStream_t st) {
  PackWs pw = pack_view(ws, dm);
  const int64_t units = (int64_t)dm.L * dm.G * dm.J_cap;
  const int LG = dm.L * dm.G;
  hipLaunchKernelGGL(k_pack_count, dim3((unsigned)((units + 4 * PC_U - 1) / (4 * PC_U))), dim3(256), 0, st, dm, tv, pw);
  hipLaunchKernelGGL(k_pack_scan_units, dim3(LG), dim3(256), 0, st, dm, tv, pw, counts);
  hipLaunchKernelGGL(k_pack_scan_lg, dim3(1), dim3(64), 0, st, dm, (const int64_t*)counts, offsets);
  const int clk = clock_begin(dm, GRACEKV_STAGE_PACK, st);
#define GKV_EMIT(TT, DD)                                                                                     \
  hipLaunchKernelGGL((k_pack_emit<TT, DD>), dim3((unsigned)units), dim3(64), 0, st, dm, (const TT*)K,       \
                     (const TT*)V, cosT, sinT, tv, pw, (const int64_t*)offsets, (TT*)K_out, (TT*)V_out, pos_out, \
                     logm_out)
  if (dm.dtype == GRACEKV_BF16) {
    if (dm.d == 128) GKV_EMIT(uint16_t, 128); else GKV_EMIT(uint16_t, 64);
  } else {
    if (dm.d == 128) GKV_EMIT(float, 128); else GKV_EMIT(float, 64);
  }
#undef GKV_EMIT
  clock_end(clk, st);
  if (dm.r > 0) {
    if (dm.dtype == GRACEKV_BF16)
      hipLaunchKernelGGL(k_pack_window<uint16_t>, dim3(dm.r, LG), dim3(64), 0, st, dm, (const uint16_t*)K,
                         (const uint16_t*)V, (const int64_t*)offsets, (uint16_t*)K_out, (uint16_t*)V_out, pos_out,
                         logm_out);
    else
      hipLaunchKernelGGL(k_pack_window<float>, dim3(dm.r, LG), dim3(64), 0, st, dm, (const float*)K,
                         (const float*)V, (const int64_t*)offsets, (float*)K_out, (float*)V_out, pos_out, logm_out);
  }
  return hipGetLastError();
}

}  // namespace gkv
