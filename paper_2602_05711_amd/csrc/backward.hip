// Backward of the expert compute (Eq. 4, 7) for L = sum_t dy_t . y_t, the gradients a training
// step needs from this layer's experts and gates:
//   h_p = x_t . u_e,  a_p = g_p act(h_p),  da_p = dy_t . v_e,
//   dgates_p = da_p act(h_p),  dh_p = da_p g_p act'(h_p),
//   dx_t = sum over t's slots of dh_p u_e,
//   du_e = sum over e's tasks of dh_p x_t,  dv_e = sum over e's tasks of a_p dy_t,
//   dscores_p = g_p (dgates_p - sum over the (t, h) row of g dgates)   (softmax, Eq. 2).
// expert pass: one wavefront walks the segments of one or two active experts (task ids
//   ascending), forms h, da, a, dh and dgates of every task and sums du and dv in that order: the
//   expert-major order makes the per-expert gradients plain sequential sums, with no atomics, so
//   every run gives the same bits;
// dx: the forward's token-major routed sum with dh in the place of a and u in the place of v;
// score pass: one wavefront per (token, head) row.
// Router backward (selections fixed; S_p = s_r[i_p] + s_c[j_p]): tasks are sorted by sub-key
// row (h, i) with the schedule's radix sort, and one wavefront per selected sub-key sums
// dscores_p x_t over its segment in task order (the same expert-major pattern, applied to the
// sub-key tables); the input gradient adds dscores_p times the two sub-keys, token by token.
#include "device_common.hpp"
#include "internal.hpp"

namespace omnimoe {
namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct BwdArgs {
  const void* x;
  const void* u;
  const void* v;
  const int32_t* idx;
  const float* gates;
  const float* dy;
  const int32_t* perm;
  const int32_t* offsets;
  const int32_t* n_active;
  float* dx;
  float* du;
  float* dv;
  float* dgates;
  float* dscores;
  float* dh;   // dh_p per task (workspace)
  int64_t T;
  int64_t N;
  int64_t M;
  int64_t cap;  // min(M, N): rows of du / dv
  int d;
  int hk;
  int K;
  int act;
  int run;      // consecutive active experts per wave (at most 63)
};

__device__ __forceinline__ int clamp_id(int v, int64_t n) {
  return v < 0 ? 0 : (v >= n ? (int)(n - 1) : v);
}

// Element k (0 .. EPC-1) of a stored 16-byte chunk, as fp32.
template <bool BF16>
__device__ __forceinline__ float chunk_elem(const uint4& c, int k) {
  if constexpr (BF16) {
    const uint32_t w = k < 2 ? c.x : (k < 4 ? c.y : (k < 6 ? c.z : c.w));
    return (k & 1) ? bf16_hi(w) : bf16_lo(w);
  } else {
    const uint32_t w = k == 0 ? c.x : (k == 1 ? c.y : (k == 2 ? c.z : c.w));
    return __uint_as_float(w);
  }
}

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// A 64-position window of the schedule: lane l holds the task, expert and gate of position
// base + l (positions from end on repeat the last one).
struct TaskWindow {
  int64_t base;
  int p;
  int e;
  float g;
};

__device__ __forceinline__ void load_window(const BwdArgs& a, int64_t base, int64_t end,
                                            TaskWindow& w) {
  const int64_t pos = base + lane_id();
  w.base = base;
  w.p = clamp_id(a.perm[pos < end ? pos : end - 1], a.M);
  w.e = clamp_id(a.idx[w.p], a.N);
  w.g = a.gates[w.p];
}

// Four elements of a stored row: 8 bytes of bf16 or 16 bytes of fp32.
template <bool BF16>
struct Quad;
template <>
struct Quad<true> {
  typedef unsigned int raw __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ float at(const raw& v, int k) {
    const uint32_t w = k < 2 ? v.x : v.y;
    return (k & 1) ? bf16_hi(w) : bf16_lo(w);
  }
  static __device__ __forceinline__ float dot(const raw& p, const raw& q, float acc) {
    return dot2_bf16(p.y, q.y, dot2_bf16(p.x, q.x, acc));
  }
};
template <>
struct Quad<false> {
  typedef f32x4_t raw;
  static __device__ __forceinline__ float at(const raw& v, int k) { return v[k]; }
  static __device__ __forceinline__ float dot(const raw& p, const raw& q, float acc) {
#pragma unroll
    for (int k = 0; k < 4; ++k) acc = fmaf(p[k], q[k], acc);
    return acc;
  }
};

// Expert pass: a wave takes a.run consecutive active experts. It reads the run's segment bounds
// and then the segments' tasks, experts and gates 64 positions at a time with one load per lane.
// Per expert it loads u_e and v_e once and takes the tasks G at a time with all of their token and
// dy rows in flight: the dot products h = x . u and da = dy . v, one activation for the group (lane
// i finishes task i), then du += dh x and dv += a dy in task order.
//
// Bound by memory: at the training shape u, v and the fp32 rows du and dv are 22 GB once (4.7 ms
// at the rate of a large copy), the token and dy rows 26 GB from the caches. Forming the dots here
// and not in a token pass of their own saves that pass's v gather and its second read of x and dy; its
// dx = sum of dh u stays token-major (launch_accumulate with dh and u). Each XCD takes a contiguous
// share of the active experts, so that a token's experts in one grid row find its rows in that XCD's
// L2; du and dv leave with non-temporal stores, and u and v are read with the non-temporal hint when
// the tables do not stay in the MALL (NTL), so that neither pushes those rows out. A lane holds four
// neighbouring elements of every 256: fp32 rows move in whole lines (with the eight elements of a
// 16-byte bf16 load every store would write half lines, and the non-temporal stores cost 1.5 ms
// instead of saving 0.6). Measured at the training shape, token pass and expert pass 8.73 ms before, this pass
// and the routed sum 7.02 ms (two experts per wave; four 7.03, eight 7.32; two tasks in flight instead of
// one 7.49; four waves sharing an expert's columns 7.27); 4093 tokens, 2^16 experts of d = 512: 236 ->
// 156 us (G = 4; 161 with two in flight, 169 with six).
template <int CPL, bool BF16, bool FULL, int G, bool NTL>
__global__ __launch_bounds__(256) void bwd_expert_kernel(BwdArgs a) {
  typedef Quad<BF16> Q;
  typedef typename Q::raw raw;
  const int l = lane_id();
  const int64_t rc = a.d / 4;
  bool cv[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) cv[q] = FULL || (l + kWave * q) < rc;
  const int64_t na = *a.n_active < a.cap ? *a.n_active : a.cap;
  // the grid covers a.cap experts; the workgroups that the active ones need are shared out to the
  // XCDs (workgroup b runs on XCD b % 8) in contiguous parts
  const int64_t nblk = (na + 4 * a.run - 1) / (4 * a.run);
  if (blockIdx.x >= nblk) return;
  const int64_t per_xcd = nblk / 8, extra = nblk % 8, xcd = blockIdx.x % 8;
  const int64_t blk = xcd * per_xcd + (xcd < extra ? xcd : extra) + blockIdx.x / 8;
  const int64_t r0 = (blk * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * a.run;
  if (r0 >= na) return;
  const int n = (int)(na - r0 < a.run ? na - r0 : a.run);
  int off = a.offsets[r0 + (l < n ? l : n)];
  off = off < 0 ? 0 : (off > a.M ? (int)a.M : off);
  const int hk_shift = (a.hk & (a.hk - 1)) == 0 ? __builtin_ctz((unsigned)a.hk) : -1;
  auto token_of = [&](int p) { return hk_shift >= 0 ? p >> hk_shift : p / a.hk; };
  const int last = readlane_i32(off, n);  // end of the wave's positions
  TaskWindow w;
  w.base = -1;
  for (int i = 0; i < n; ++i) {
    const int b = readlane_i32(off, i), e = readlane_i32(off, i + 1);
    f32x4_t du[CPL], dv[CPL];
#pragma unroll
    for (int q = 0; q < CPL; ++q) du[q] = dv[q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    raw ur[CPL], vr[CPL];
    for (int64_t pos = b; pos < e;) {
      if (w.base < 0 || pos < w.base || pos >= w.base + kWave)
        load_window(a, pos, last > pos ? last : pos + 1, w);
      const int j0 = (int)(pos - w.base);
      int cnt = (int)(e - pos < G ? e - pos : G);
      if (cnt > kWave - j0) cnt = kWave - j0;
      if (pos == b) {
        const int64_t row = (int64_t)readlane_i32(w.e, j0) * rc + l;
        const raw* U = (const raw*)a.u + row;
        const raw* V = (const raw*)a.v + row;
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          ur[q] = vr[q] = raw{};
          if (cv[q]) {
            ur[q] = NTL ? __builtin_nontemporal_load(U + kWave * q) : U[kWave * q];
            vr[q] = NTL ? __builtin_nontemporal_load(V + kWave * q) : V[kWave * q];
          }
        }
      }
      raw xr[G][CPL];
      f32x4_t yr[G][CPL];
#pragma unroll
      for (int g = 0; g < G; ++g) {
        // past the group's last task its rows are loaded again (and not added)
        const int64_t t = token_of(readlane_i32(w.p, j0 + (g < cnt ? g : cnt - 1)));
        const raw* X = (const raw*)a.x + t * rc + l;
        const f32x4_t* Y = (const f32x4_t*)a.dy + t * rc + l;
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          xr[g][q] = raw{};
          yr[g][q] = f32x4_t{0.f, 0.f, 0.f, 0.f};
          if (cv[q]) {
            xr[g][q] = X[kWave * q];
            yr[g][q] = Y[kWave * q];
          }
        }
      }
      // every load above is issued before the first product (left alone, the scheduler interleaves
      // them with the products and waits for each row in turn)
      __builtin_amdgcn_sched_barrier(0);
      float hv = 0.0f, dav = 0.0f, gv = 0.0f;
      int pv = 0;
#pragma unroll
      for (int g = 0; g < G; ++g) {
        float hs = 0.0f, ds = 0.0f;
#pragma unroll
        for (int q = 0; q < CPL; ++q) {
          hs = Q::dot(ur[q], xr[g][q], hs);
#pragma unroll
          for (int k = 0; k < 4; ++k) ds = fmaf(yr[g][q][k], Q::at(vr[q], k), ds);
        }
        if (g < cnt) {
          const float h = wave_sum_uniform(hs), da = wave_sum_uniform(ds);
          const float gt = readlane_f32(w.g, j0 + g);
          const int p = readlane_i32(w.p, j0 + g);
          if (l == g) {
            hv = h;
            dav = da;
            gv = gt;
            pv = p;
          }
        }
      }
      const float act = activation(a.act, hv);
      const float av = gv * act, dhv = dav * gv * activation_grad(a.act, hv);
      if (l < cnt) {
        a.dh[pv] = dhv;
        a.dgates[pv] = dav * act;
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        if (g < cnt) {
          const float ap = readlane_f32(av, g), dhp = readlane_f32(dhv, g);
#pragma unroll
          for (int q = 0; q < CPL; ++q)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
              dv[q][k] = fmaf(ap, yr[g][q][k], dv[q][k]);
              du[q][k] = fmaf(dhp, Q::at(xr[g][q], k), du[q][k]);
            }
        }
      }
      pos += cnt;
    }
    f32x4_t* ou = (f32x4_t*)a.du + (r0 + i) * rc + l;
    f32x4_t* ov = (f32x4_t*)a.dv + (r0 + i) * rc + l;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!cv[q]) continue;
      __builtin_nontemporal_store(du[q], ou + kWave * q);
      __builtin_nontemporal_store(dv[q], ov + kWave * q);
    }
  }
}

__global__ __launch_bounds__(256) void bwd_score_kernel(BwdArgs a) {
  const int l = lane_id();
  const int64_t rows = a.T * (a.hk / a.K);
  const int64_t stride = (int64_t)gridDim.x * 4;
  for (int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); row < rows; row += stride) {
    const int64_t base = row * a.K;
    float part = 0.0f;
    for (int k = l; k < a.K; k += kWave) part = fmaf(a.gates[base + k], a.dgates[base + k], part);
    const float sgd = wave_sum_f32(part);
    for (int k = l; k < a.K; k += kWave)
      a.dscores[base + k] = a.gates[base + k] * (a.dgates[base + k] - sgd);
  }
}

// Sub-key of every task for one half: key = h * n_half + (row or column of the expert id).
__global__ __launch_bounds__(256) void subkey_kernel(const int32_t* idx, int32_t* key, int64_t m,
                                                     int hk, int K, int nc, int n_half, int col,
                                                     int64_t n_experts) {
  const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (p >= m) return;
  const int e = clamp_id(idx[p], n_experts);
  const int h = (int)((p % hk) / K);
  key[p] = h * n_half + (col ? e % nc : e / nc);
}

struct KeySumArgs {
  const void* x;
  const float* ds;
  const int32_t* perm;
  const int32_t* active;
  const int32_t* offsets;
  const int32_t* n_active;
  float* dk;         // [H * n_half, d_key]
  int64_t M;
  int64_t cap;
  int64_t n_keys;
  int d;             // row length of x
  int dkey;
  int c0;            // first x column of this half's query
  int hk;
  int nchunks;       // 16-byte chunks of a d_key slice
};

// Tasks j0 .. j0 + GG - 1 of a keysum batch (slot pl, weight wl on lane j): their x slices are
// loaded together, then acc += ds_p x_t in task order.
template <int GG, int CPL, bool BF16>
__device__ __forceinline__ void keysum_group(const KeySumArgs& a, const uint4* X, int64_t xrc,
                                             int64_t c0, const bool (&cv)[CPL], int pl, float wl,
                                             int j0, float (&acc)[CPL][BF16 ? 8 : 4]) {
  constexpr int EPC = BF16 ? 8 : 4;
  const int l = lane_id();
  uint4 xr[GG][CPL];
#pragma unroll
  for (int i = 0; i < GG; ++i) {
    const int64_t t = readlane_i32(pl, j0 + i) / a.hk;
#pragma unroll
    for (int q = 0; q < CPL; ++q)
      xr[i][q] = cv[q] ? X[t * xrc + c0 + l + kWave * q] : make_uint4(0, 0, 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);  // all of the group's loads before its first product
#pragma unroll
  for (int i = 0; i < GG; ++i) {
    const float w = readlane_f32(wl, j0 + i);
#pragma unroll
    for (int q = 0; q < CPL; ++q)
#pragma unroll
      for (int k = 0; k < EPC; ++k) acc[q][k] = fmaf(w, chunk_elem<BF16>(xr[i][q], k), acc[q][k]);
  }
}

// One wavefront per selected sub-key: dk[key] = sum over its tasks (task order) of ds_p x_t.
// The segment's tasks are taken 64 at a time (slot and ds with one load per lane), then eight
// (or, with wide rows, fewer) at a time with their x slices in flight together; whole groups
// first and the rest singly, so that every product of a group is unconditional.
template <int CPL, bool BF16, bool FULL>
__global__ __launch_bounds__(256) void keysum_kernel(KeySumArgs a) {
  constexpr int EPC = BF16 ? 8 : 4;
  constexpr int G = CPL >= 8 ? 2 : (CPL >= 4 ? 4 : 8);
  const int l = lane_id();
  const int64_t xrc = a.d / EPC;   // chunks per x row
  const int64_t c0 = a.c0 / EPC;
  const uint4* X = (const uint4*)a.x;
  bool cv[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) cv[q] = FULL || (l + kWave * q) < a.nchunks;
  const int64_t na = *a.n_active < a.cap ? *a.n_active : a.cap;
  const int64_t stride = (int64_t)gridDim.x * 4;
  for (int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); r < na; r += stride) {
    float acc[CPL][EPC];
#pragma unroll
    for (int q = 0; q < CPL; ++q)
#pragma unroll
      for (int k = 0; k < EPC; ++k) acc[q][k] = 0.0f;
    int64_t b = a.offsets[r], e = a.offsets[r + 1];
    b = b < 0 ? 0 : (b > a.M ? a.M : b);
    e = e < b ? b : (e > a.M ? a.M : e);
    for (int64_t base = b; base < e; base += kWave) {
      const int n = (int)(e - base < kWave ? e - base : kWave);
      const int pl = clamp_id(a.perm[base + (l < n ? l : n - 1)], a.M);
      const float wl = a.ds[pl];
      int j0 = 0;
      for (; j0 + G <= n; j0 += G) keysum_group<G, CPL, BF16>(a, X, xrc, c0, cv, pl, wl, j0, acc);
      for (; j0 < n; ++j0) keysum_group<1, CPL, BF16>(a, X, xrc, c0, cv, pl, wl, j0, acc);
    }
    const int key = clamp_id(a.active[r], a.n_keys);
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!cv[q]) continue;
      float4* o = (float4*)(a.dk + (int64_t)key * a.dkey + (int64_t)(l + kWave * q) * EPC);
#pragma unroll
      for (int k = 0; k < EPC; k += 4) o[k / 4] = make_float4(acc[q][k], acc[q][k + 1], acc[q][k + 2], acc[q][k + 3]);
    }
  }
}

struct RouteDxArgs {
  const void* kr;
  const void* kc;
  const int32_t* idx;
  const float* ds;
  float* dx;
  int64_t T;
  int64_t N;
  int d;
  int dkey;
  int c0;
  int hk;
  int K;
  int nr, nc;
  int nchunks;   // 16-byte chunks of a d_key row
};

// Slots s0 .. s0 + GG - 1 of token t (expert on lane s - sb of ev, weight of wv): both sub-key
// rows of each are loaded together, then ar += ds_p keys_row[h, i_p] and ac += ds_p
// keys_col[h, j_p] in slot order.
template <int GG, int CPL, bool BF16>
__device__ __forceinline__ void route_dx_group(const RouteDxArgs& a, const bool (&cv)[CPL], int s0,
                                               int sb, int ev, float wv,
                                               float (&ar)[CPL][BF16 ? 8 : 4],
                                               float (&ac)[CPL][BF16 ? 8 : 4]) {
  constexpr int EPC = BF16 ? 8 : 4;
  const int l = lane_id();
  const uint4* KR = (const uint4*)a.kr;
  const uint4* KC = (const uint4*)a.kc;
  const int64_t rc = a.nchunks;
  uint4 rr[GG][CPL], cr[GG][CPL];
#pragma unroll
  for (int i = 0; i < GG; ++i) {
    const int s = s0 + i;
    const int e = clamp_id(readlane_i32(ev, s - sb), a.N);
    const int h = s / a.K;
    const int64_t ri = (int64_t)h * a.nr + e / a.nc;
    const int64_t cj = (int64_t)h * a.nc + e % a.nc;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      rr[i][q] = cv[q] ? KR[ri * rc + l + kWave * q] : make_uint4(0, 0, 0, 0);
      cr[i][q] = cv[q] ? KC[cj * rc + l + kWave * q] : make_uint4(0, 0, 0, 0);
    }
  }
  __builtin_amdgcn_sched_barrier(0);  // all of the group's loads before its first product
#pragma unroll
  for (int i = 0; i < GG; ++i) {
    const float w = readlane_f32(wv, s0 + i - sb);
#pragma unroll
    for (int q = 0; q < CPL; ++q)
#pragma unroll
      for (int k = 0; k < EPC; ++k) {
        ar[q][k] = fmaf(w, chunk_elem<BF16>(rr[i][q], k), ar[q][k]);
        ac[q][k] = fmaf(w, chunk_elem<BF16>(cr[i][q], k), ac[q][k]);
      }
  }
}

// dx_t[0 : d_key] += sum of ds_p keys_row[h, i_p]; dx_t[c0 : c0 + d_key] += sum of ds_p
// keys_col[h, j_p]; one wavefront per token, slots in order: experts and weights read 64 slots
// at a time, then groups of slots with all of their sub-key rows in flight.
template <int CPL, bool BF16, bool FULL>
__global__ __launch_bounds__(256) void route_dx_kernel(RouteDxArgs a) {
  constexpr int EPC = BF16 ? 8 : 4;
  constexpr int G = CPL >= 8 ? 1 : (CPL >= 4 ? 2 : 4);
  const int l = lane_id();
  bool cv[CPL];
#pragma unroll
  for (int q = 0; q < CPL; ++q) cv[q] = FULL || (l + kWave * q) < a.nchunks;
  const int64_t stride = (int64_t)gridDim.x * 4;
  for (int64_t t = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); t < a.T; t += stride) {
    float ar[CPL][EPC], ac[CPL][EPC];
#pragma unroll
    for (int q = 0; q < CPL; ++q)
#pragma unroll
      for (int k = 0; k < EPC; ++k) ar[q][k] = ac[q][k] = 0.0f;
    for (int sb = 0; sb < a.hk; sb += kWave) {
      const int n = a.hk - sb < kWave ? a.hk - sb : kWave;
      const int64_t pl = t * a.hk + sb + (l < n ? l : n - 1);
      const int ev = a.idx[pl];
      const float wv = a.ds[pl];
      int s0 = sb;
      for (; s0 + G <= sb + n; s0 += G) route_dx_group<G, CPL, BF16>(a, cv, s0, sb, ev, wv, ar, ac);
      for (; s0 < sb + n; ++s0) route_dx_group<1, CPL, BF16>(a, cv, s0, sb, ev, wv, ar, ac);
    }
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!cv[q]) continue;
      float* o1 = a.dx + t * a.d + (int64_t)(l + kWave * q) * EPC;
      float* o2 = a.dx + t * a.d + a.c0 + (int64_t)(l + kWave * q) * EPC;
      if (a.c0 == 0) {
#pragma unroll
        for (int k = 0; k < EPC; ++k) o1[k] += ar[q][k] + ac[q][k];
      } else {
#pragma unroll
        for (int k = 0; k < EPC; ++k) {
          o1[k] += ar[q][k];
          o2[k] += ac[q][k];
        }
      }
    }
  }
}

template <int CPL, bool BF16>
void launch_router_bwd_kernels(const KeySumArgs& kr, const KeySumArgs& kc, const RouteDxArgs& rd,
                               int pass, hipStream_t st) {
  if (pass < 2) {
    const KeySumArgs& a = pass == 0 ? kr : kc;
    int64_t blocks = (a.cap + 3) / 4;
    if (blocks > 65536) blocks = 65536;
    if (a.nchunks == CPL * kWave)
      hipLaunchKernelGGL((keysum_kernel<CPL, BF16, true>), dim3((unsigned)blocks), dim3(256), 0,
                         st, a);
    else
      hipLaunchKernelGGL((keysum_kernel<CPL, BF16, false>), dim3((unsigned)blocks), dim3(256), 0,
                         st, a);
  } else {
    int64_t blocks = (rd.T + 3) / 4;
    if (blocks > 16384) blocks = 16384;
    if (rd.nchunks == CPL * kWave)
      hipLaunchKernelGGL((route_dx_kernel<CPL, BF16, true>), dim3((unsigned)blocks), dim3(256), 0,
                         st, rd);
    else
      hipLaunchKernelGGL((route_dx_kernel<CPL, BF16, false>), dim3((unsigned)blocks), dim3(256),
                         0, st, rd);
  }
}

template <bool BF16>
hipError_t dispatch_router_bwd(int cpl, const KeySumArgs& kr, const KeySumArgs& kc,
                               const RouteDxArgs& rd, int pass, hipStream_t st) {
  switch (cpl) {
    case 1: launch_router_bwd_kernels<1, BF16>(kr, kc, rd, pass, st); break;
    case 2: launch_router_bwd_kernels<2, BF16>(kr, kc, rd, pass, st); break;
    case 4: launch_router_bwd_kernels<4, BF16>(kr, kc, rd, pass, st); break;
    case 8: launch_router_bwd_kernels<8, BF16>(kr, kc, rd, pass, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

int cpl_of(int nchunks) {
  int c = 1;
  while (c * kWave < nchunks) c <<= 1;
  return c;
}

// Tables up to this size stay in the MALL (256 MB) between the passes that read them.
constexpr int64_t kMallTableBytes = 128ll << 20;

template <bool BF16, int CPL, int G>
void launch_bwd(hipStream_t st, const BwdArgs& a) {
  const dim3 grid((unsigned)((a.cap + 4 * a.run - 1) / (4 * a.run)));
  const bool full = a.d == CPL * 4 * kWave;
  const bool ntl = a.N * (int64_t)a.d * (BF16 ? 2 : 4) > kMallTableBytes;
#define OMNIMOE_BWD(F_, N_) \
  hipLaunchKernelGGL((bwd_expert_kernel<CPL, BF16, F_, G, N_>), grid, dim3(256), 0, st, a)
  if (full && ntl) OMNIMOE_BWD(true, true);
  else if (full) OMNIMOE_BWD(true, false);
  else if (ntl) OMNIMOE_BWD(false, true);
  else OMNIMOE_BWD(false, false);
#undef OMNIMOE_BWD
}

// cpl: 256-element pieces of a row, rounded up to a power of two (at most 16: d <= 4096).
template <bool BF16>
hipError_t dispatch_bwd(int cpl, hipStream_t st, const BwdArgs& a) {
  switch (cpl) {
    case 1: launch_bwd<BF16, 1, 4>(st, a); break;
    case 2: launch_bwd<BF16, 2, 4>(st, a); break;
    case 4: launch_bwd<BF16, 4, 2>(st, a); break;
    case 8: launch_bwd<BF16, 8, 1>(st, a); break;
    case 16: launch_bwd<BF16, 16, 1>(st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

size_t backward_ws_bytes(int64_t M) { return ((size_t)M * 4 + 255) & ~(size_t)255; }

hipError_t launch_expert_backward(const Shape& s, const void* x, const void* u, const void* v,
                                  const int32_t* idx, const float* gates, const int32_t* perm,
                                  const int32_t* offsets, const int32_t* n_active,
                                  const float* dy, float* dx, float* du, float* dv,
                                  float* dgates, float* dscores, void* ws, hipStream_t st) {
  if (s.T == 0) return hipSuccess;
  BwdArgs a;
  a.x = x;
  a.u = u;
  a.v = v;
  a.idx = idx;
  a.gates = gates;
  a.dy = dy;
  a.perm = perm;
  a.offsets = offsets;
  a.n_active = n_active;
  a.dx = dx;
  a.du = du;
  a.dv = dv;
  a.dgates = dgates;
  a.dscores = dscores;
  a.dh = (float*)ws;
  a.T = s.T;
  a.N = s.N;
  a.M = s.M;
  a.cap = s.M < s.N ? s.M : s.N;
  a.d = s.d;
  a.hk = s.hk;
  a.K = s.K;
  a.act = s.act;
  // Two experts per wave share its window loads (training shape 7.08 -> 7.02 ms); one below 32768,
  // where halving the waves costs more (10^4 experts of d = 256: 83 us with one, 92 with two).
  a.run = a.cap >= 32768 ? 2 : 1;
  hipError_t e = s.bf16 ? dispatch_bwd<true>(cpl_of(s.d / 4), st, a)
                        : dispatch_bwd<false>(cpl_of(s.d / 4), st, a);
  // dx_t = sum of dh_p u_e over t's slots: the token-major routed sum with dh and u
  if (e == hipSuccess) e = launch_accumulate(s, u, idx, a.dh, dx, st);
  if (e != hipSuccess) return e;
  int64_t sb = (s.rows + 3) / 4;
  if (sb > 16384) sb = 16384;
  hipLaunchKernelGGL(bwd_score_kernel, dim3((unsigned)sb), dim3(256), 0, st, a);
  return hipGetLastError();
}

size_t route_backward_ws_bytes(const Shape& s) {
  const int64_t nkeys = (int64_t)s.H * (s.nr > s.nc ? s.nr : s.nc);
  const int64_t cap = s.M < nkeys ? s.M : nkeys;
  auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
  return 2 * al((size_t)s.M * 4) + al((size_t)s.M * 4) + 2 * al((size_t)(cap + 1) * 4) + 256 +
         schedule_ws_bytes(s.M, nkeys);
}

hipError_t launch_route_backward(const Shape& s, const void* x, const void* keys_row,
                                 const void* keys_col, const int32_t* idx, const float* dscores,
                                 float* dx, float* dkeys_row, float* dkeys_col, void* ws,
                                 hipStream_t st) {
  if (s.T == 0) return hipSuccess;
  auto al = [](size_t v) { return (v + 255) & ~(size_t)255; };
  const int64_t nkeys = (int64_t)s.H * (s.nr > s.nc ? s.nr : s.nc);
  const int64_t cap = s.M < nkeys ? s.M : nkeys;
  char* w = (char*)ws;
  int32_t* rkey = (int32_t*)w; w += al((size_t)s.M * 4);
  int32_t* ckey = (int32_t*)w; w += al((size_t)s.M * 4);
  int32_t* perm = (int32_t*)w; w += al((size_t)s.M * 4);
  int32_t* active = (int32_t*)w; w += al((size_t)(cap + 1) * 4);
  int32_t* offsets = (int32_t*)w; w += al((size_t)(cap + 1) * 4);
  int32_t* n_active = (int32_t*)w; w += 256;
  void* sws = w;
  const int64_t mb = (s.M + 255) / 256;
  hipLaunchKernelGGL(subkey_kernel, dim3((unsigned)mb), dim3(256), 0, st, idx, rkey, s.M, s.hk,
                     s.K, s.nc, s.nr, 0, s.N);
  hipLaunchKernelGGL(subkey_kernel, dim3((unsigned)mb), dim3(256), 0, st, idx, ckey, s.M, s.hk,
                     s.K, s.nc, s.nc, 1, s.N);
  hipError_t e = launch_fill_i32((int32_t*)dkeys_row, (int64_t)s.H * s.nr * s.dk, 0, st);
  if (e == hipSuccess) e = launch_fill_i32((int32_t*)dkeys_col, (int64_t)s.H * s.nc * s.dk, 0, st);
  if (e != hipSuccess) return e;
  const int epc = s.bf16 ? 8 : 4;
  const int nchunks = s.dk / epc;
  const int cpl = cpl_of(nchunks);
  KeySumArgs ka;
  ka.x = x;
  ka.ds = dscores;
  ka.perm = perm;
  ka.active = active;
  ka.offsets = offsets;
  ka.n_active = n_active;
  ka.M = s.M;
  ka.d = s.d;
  ka.dkey = s.dk;
  ka.hk = s.hk;
  ka.nchunks = nchunks;
  RouteDxArgs rd;
  rd.kr = keys_row;
  rd.kc = keys_col;
  rd.idx = idx;
  rd.ds = dscores;
  rd.dx = dx;
  rd.T = s.T;
  rd.N = s.N;
  rd.d = s.d;
  rd.dkey = s.dk;
  rd.c0 = s.col0;
  rd.hk = s.hk;
  rd.K = s.K;
  rd.nr = s.nr;
  rd.nc = s.nc;
  rd.nchunks = nchunks;
  for (int half = 0; half < 2; ++half) {
    // the tasks sorted by this half's sub-key, then one wavefront per selected sub-key
    Shape ss = s;
    ss.N = (int64_t)s.H * (half ? s.nc : s.nr);
    ss.B = 1;
    const int32_t* sk = nullptr;
    e = launch_schedule(ss, half ? ckey : rkey, perm, active, offsets, n_active, nullptr, sws, &sk,
                        st);
    if (e != hipSuccess) return e;
    ka.cap = s.M < ss.N ? s.M : ss.N;
    ka.n_keys = ss.N;
    ka.c0 = half ? s.col0 : 0;
    ka.dk = half ? dkeys_col : dkeys_row;
    e = s.bf16 ? dispatch_router_bwd<true>(cpl, ka, ka, rd, 0, st)
               : dispatch_router_bwd<false>(cpl, ka, ka, rd, 0, st);
    if (e != hipSuccess) return e;
  }
  return s.bf16 ? dispatch_router_bwd<true>(cpl, ka, ka, rd, 2, st)
                : dispatch_router_bwd<false>(cpl, ka, ka, rd, 2, st);
}

}  // namespace omnimoe
