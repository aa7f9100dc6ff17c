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
//   every run gives the same bits; a segment of more than piece_tasks(M) tasks is cut at the
//   multiples of that number, its pieces go to waves of their own, and their sums are added in order;
// dx: the forward's token-major routed sum with dh in the place of a and u in the place of v;
// score pass: one wavefront per (token, head) row; the same launch adds the pieces' sums to du and dv.
// Router backward (selections fixed; S_p = s_r[i_p] + s_c[j_p]): the tasks of a (token, head) row
// that share a sub-key are merged into one pick, the picks of both halves are put in sub-key order
// by one counting pass, and one wavefront per sub-key sums its picks' w x_t, tokens ascending; the input
// gradient adds w times the picks' sub-keys, token by token.
#include <algorithm>

#include "device_common.hpp"
#include "internal.hpp"

namespace omnimoe {
namespace {

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
  int32_t* piece_row;  // [blocks] du / dv row that the piece from position j << piece_bits on belongs to, or -1
  float* piece_sum;    // [blocks][2][d] its du and dv
  int64_t T;
  int64_t N;
  int64_t M;
  int64_t cap;  // min(M, N): rows of du / dv
  int d;
  int hk;
  int K;
  int act;
  int run;      // consecutive active experts per wave (at most 63)
  int piece_bits;  // log2 of the tasks of a piece
  int blocks;      // ceil(M / piece): positions where a piece may begin
  int piece_wgs;   // workgroups of the expert pass that look for pieces (a multiple of 8)
  int score_wgs;   // workgroups of the score pass that take rows
};

__device__ __forceinline__ int clamp_id(int v, int64_t n) {
  return v < 0 ? 0 : (v >= n ? (int)(n - 1) : v);
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

__device__ __forceinline__ int clamp_pos(int v, int64_t m) {
  return v < 0 ? 0 : (v > m ? (int)m : v);
}

// The last of n ascending segment starts that is at most pos (the first where none is): the wave
// probes 64 of them at a time.
__device__ __forceinline__ int64_t segment_of(const int32_t* offsets, int64_t n, int pos) {
  int64_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const int64_t step = (hi - lo + kWave - 1) / kWave;
    const int64_t q = lo + lane_id() * step;
    const uint64_t m = __ballot(q < hi && offsets[q < hi ? q : lo] <= pos);
    const int c = __popcll(m);
    lo += (c > 0 ? c - 1 : 0) * step;
    hi = lo + step < hi ? lo + step : hi;
  }
  return lo;
}

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
// 156 us (G = 4; 161 with two in flight, 169 with six). 2048 tokens of 32 tasks, 2^14 experts of d = 4096: 461 -> 428. With
// about one task per active expert the sum over dx reads most u rows a second time (2048 tokens at the training
// shape, 231k experts of 1.1 tasks: 1354 -> 1409 us, 5.7 GB and 1.07 GB at 4.8 and 5.5 TB/s); with fewer tokens the
// former pass by tokens had too few waves (512 tokens 441 -> 350, 64 tokens 168 -> 52).
//
// A wave forms about one task a microsecond, so an expert that many tokens pick would be walked by one wave
// while the chip idles. A segment of more than one piece of tasks (16, or M / 2048 where that is more: at most
// about 2048 pieces, the waves that the chip holds at d = 2048, and as many rows of workspace) is cut at the
// multiples of a piece: its expert's wave takes the tasks up to the first cut, and the first a.piece_wgs
// workgroups the other pieces, one a wave, with sums of their own that bwd_score_kernel's launch adds in order.
// Zipf-distributed picks (exponent, tasks of the most picked expert), before and after: training shape, 0.6
// (3278) 8990 -> 8200 us, 0.8 (27473) 36310 -> 7756, 1.0 (145305) 159.1 -> 6.6 ms; 4096 tokens, 2^16 experts of d =
// 512, 0.6 (1248) 674 -> 231 us, 1.0 (22585) 8979 -> 205; 300 tokens of 8 tasks, 900 experts of d = 64, 0.6 (63)
// 33 -> 17. Looking for pieces where there is none costs up to 1 us (uniform picks: 198 and 198 us, 16.0 and 16.6).
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
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int piece = 1 << a.piece_bits;
  int n, off;
  f32x4_t *ou, *ov;  // the first segment's du and dv
  if ((int)blockIdx.x < a.piece_wgs) {
    // the piece that begins at position j * piece, if a segment of more tasks runs across it
    const int j = (int)blockIdx.x * 4 + wv;
    if (j >= a.blocks) return;
    const int pos = j << a.piece_bits;
    const int64_t r = na > 0 ? segment_of(a.offsets, na, pos) : 0;
    const int b = clamp_pos(a.offsets[r], a.M), e = clamp_pos(a.offsets[r + 1], a.M);
    const bool mine = na > 0 && b < pos && pos < e && e - b > piece;
    if (l == 0) a.piece_row[j] = mine ? (int)r : -1;
    if (!mine) return;
    n = 1;
    off = l == 0 ? pos : (e - pos < piece ? e : pos + piece);
    ou = (f32x4_t*)a.piece_sum + (int64_t)j * 2 * rc;
    ov = ou + rc;
  } else {
    // the grid covers a.cap experts; the workgroups that the active ones need are shared out to the
    // XCDs (workgroup b runs on XCD b % 8) in contiguous parts
    const int64_t wg = blockIdx.x - a.piece_wgs;
    const int64_t nblk = (na + 4 * a.run - 1) / (4 * a.run);
    if (wg >= nblk) return;
    const int64_t per_xcd = nblk / 8, extra = nblk % 8, xcd = wg % 8;
    const int64_t blk = xcd * per_xcd + (xcd < extra ? xcd : extra) + wg / 8;
    const int64_t r0 = (blk * 4 + wv) * a.run;
    if (r0 >= na) return;
    n = (int)(na - r0 < a.run ? na - r0 : a.run);
    off = clamp_pos(a.offsets[r0 + (l < n ? l : n)], a.M);
    ou = (f32x4_t*)a.du + r0 * rc;
    ov = (f32x4_t*)a.dv + r0 * rc;
  }
  const int hk_shift = (a.hk & (a.hk - 1)) == 0 ? __builtin_ctz((unsigned)a.hk) : -1;
  auto token_of = [&](int p) { return hk_shift >= 0 ? p >> hk_shift : p / a.hk; };
  const int last = readlane_i32(off, n);  // end of the wave's positions
  TaskWindow w;
  w.base = -1;
  for (int i = 0; i < n; ++i) {
    const int b = readlane_i32(off, i);
    int e = readlane_i32(off, i + 1);
    if (e - b > piece) e = ((b >> a.piece_bits) + 1) << a.piece_bits;  // its first piece
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
    f32x4_t* const pu = ou + i * rc + l;
    f32x4_t* const pv = ov + i * rc + l;
#pragma unroll
    for (int q = 0; q < CPL; ++q) {
      if (!cv[q]) continue;
      __builtin_nontemporal_store(du[q], pu + kWave * q);
      __builtin_nontemporal_store(dv[q], pv + kWave * q);
    }
  }
}

// Piece positions per workgroup of add_pieces.
constexpr int kPieceGroup = 16;

// du and dv of the rows whose segments were cut: the first piece's sum (in place) plus the others', in
// order. Workgroup g takes 1024 columns of du or dv for the rows whose second piece is among kPieceGroup
// positions.
__device__ __forceinline__ void add_pieces(const BwdArgs& a, int g) {
  const int slices = (a.d + 1023) / 1024;
  const int64_t rc = a.d / 4;
  const int which = g % 2, c = (g / 2) % slices * 256 + (int)threadIdx.x, j0 = g / (2 * slices) * kPieceGroup;
  // lane i holds position j0 - 1 + i: a second piece is one whose predecessor belongs to another row
  const int l = lane_id(), jl = j0 - 1 + l;
  const int mine = l <= kPieceGroup && jl >= 0 && jl < a.blocks ? a.piece_row[jl] : -1;
  const int before = __shfl_up(mine, 1, kWave);
  for (uint64_t m = __ballot(l > 0 && mine >= 0 && mine != before); m; m &= m - 1) {
    const int i = __builtin_ctzll(m), j = j0 - 1 + i;
    const int64_t r = readlane_i32(mine, i);
    if (c >= rc) continue;
    const int e = clamp_pos(a.offsets[r + 1], a.M);
    const int jend = (int)(((int64_t)e + (1 << a.piece_bits) - 1) >> a.piece_bits);
    f32x4_t* const row = (f32x4_t*)(which ? a.dv : a.du) + r * rc + c;
    const f32x4_t* const part = (const f32x4_t*)a.piece_sum + which * rc + c;
    f32x4_t acc = *row;
    constexpr int G = 8;
    for (int k0 = j; k0 < jend; k0 += G) {
      f32x4_t p[G];
#pragma unroll
      for (int k = 0; k < G; ++k)
        p[k] = part[(int64_t)(k0 + k < jend ? k0 + k : jend - 1) * 2 * rc];
#pragma unroll
      for (int k = 0; k < G; ++k)
        if (k0 + k < jend) acc += p[k];
    }
    *row = acc;
  }
}

__global__ __launch_bounds__(256) void bwd_score_kernel(BwdArgs a) {
  if ((int)blockIdx.x >= a.score_wgs) {
    add_pieces(a, (int)blockIdx.x - a.score_wgs);
    return;
  }
  const int l = lane_id();
  const int64_t rows = a.T * (a.hk / a.K);
  const int64_t stride = (int64_t)a.score_wgs * 4;
  for (int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); row < rows; row += stride) {
    const int64_t base = row * a.K;
    float part = 0.0f;
    for (int k = l; k < a.K; k += kWave) part = fmaf(a.gates[base + k], a.dgates[base + k], part);
    const float sgd = wave_sum_f32(part);
    for (int k = l; k < a.K; k += kWave)
      a.dscores[base + k] = a.gates[base + k] * (a.dgates[base + k] - sgd);
  }
}

// ------------------------------------------------------------------ router backward
// Buckets are the sub-keys of both halves: row i of head h is bucket h nr + i, column j of head h
// bucket H nr + h nc + j. A pick is a task that leads its block: of the tasks of one (token, head)
// row and one block of up to sixteen slots that share a sub-key, the first carries the sum of their
// weights and the others carry none (a row's K cells lie in few grid rows and columns, so the K
// picks of one half are about a third as many sub-keys; the key and token rows are then read once
// for each of those). The picks of a head are ordered by one counting pass over its own sub-keys:
// per-tile counts, a scan, and the places, both halves in the same launches. Measured, the router backward
// at the training shape 1.29 -> 0.68 ms (keys and sums 600 + 2 x 262 us before, 282 + 274 now; the
// rest 190 -> 110) and with 4093 tokens, 2^16 experts of d = 512, 290 -> 66 us, against a
// radix sort of all tasks per half.
struct RouteArgs {
  const int32_t* idx;
  const float* ds;
  const void* x;
  const void* keys[2];
  float* dkeys[2];
  float* dx;
  int32_t* key;    // [halves][M] sub-key index within its head, -1 where the task leads no block
  float* w;        // [halves][M] summed weight of a pick
  int32_t* hist;   // [buckets][tiles] picks, then their exclusive scan; one more entry: the total
  int2* picks;     // (token, weight bits) of every pick, by bucket, tokens ascending
  int64_t T;
  int64_t N;
  int64_t M;
  int half0;       // first half of this round (0, or 1 where the halves take a round each)
  int d;
  int dkey;
  int col0;        // first x column of the column half
  int H;
  int K;
  int nh[2];       // nr, nc
  int tpt;         // tokens per tile
  int tiles;       // tiles per head
  int halves;      // halves of this round
  int slices;      // 256-element pieces of a d_key row
};

// Bucket of sub-key 0 of head h, counted from the round's first half.
__device__ __forceinline__ int64_t bucket0(const RouteArgs& a, int half, int h) {
  return (half > a.half0 ? (int64_t)a.H * a.nh[0] : 0) + (int64_t)h * a.nh[half];
}

// One workgroup per (tile of a.tpt tokens, head, half): finds the picks and counts them by
// sub-key. P: slots per block, a power of two of at most 16 (lanes of one block exchange keys and
// weights; weights are added in slot order). LDS: a counter per sub-key of the head.
__global__ __launch_bounds__(256) void route_count_kernel(RouteArgs a, int P) {
  extern __shared__ int cnt[];
  const int h = (int)(blockIdx.x / (unsigned)a.tiles), tile = (int)(blockIdx.x - (unsigned)h * a.tiles);
  const int half = a.half0 + (int)blockIdx.z, n = a.nh[half], nc = a.nh[1];
  for (int i = threadIdx.x; i < n; i += 256) cnt[i] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)tile * a.tpt;
  const int ntok = (int)(a.T - t0 < a.tpt ? a.T - t0 : a.tpt);
  const int nb = (a.K + P - 1) / P;
  const int items = ntok * nb * P;
  const int l = lane_id();
  int32_t* const key = a.key + (int64_t)blockIdx.z * a.M;
  float* const wout = a.w + (int64_t)blockIdx.z * a.M;
  for (int i0 = 0; i0 < items; i0 += 256) {
    const int it = i0 + threadIdx.x;
    const int bl = it / P, tok = bl / nb, slot = (bl - tok * nb) * P + (it & (P - 1));
    const bool valid = it < items && slot < a.K;
    const int64_t p = ((t0 + tok) * a.H + h) * a.K + slot;
    const int e = valid ? clamp_id(a.idx[p], a.N) : 0;
    float w = valid ? a.ds[p] : 0.0f;
    const int k = valid ? (half ? e % nc : e / nc) : -1;
    bool lead = valid;
    const float own = w;
    for (int r = 1; r < P; ++r) {
      const int src = (l & ~(P - 1)) | ((l + r) & (P - 1));
      const int ko = __shfl(k, src, kWave);
      const float wo = __shfl(own, src, kWave);
      if (ko == k) {
        if (src < l) lead = false;
        else w += wo;
      }
    }
    if (valid) {
      key[p] = lead ? k : -1;
      wout[p] = w;
      if (lead) atomicAdd(&cnt[k], 1);
    }
  }
  __syncthreads();
  int32_t* const hist = a.hist + bucket0(a, half, h) * a.tiles + tile;
  for (int i = threadIdx.x; i < n; i += 256) hist[(int64_t)i * a.tiles] = cnt[i];
  if (blockIdx.x == 0 && blockIdx.z == 0 && threadIdx.x == 0) {
    const int64_t nbk = (int64_t)a.H * (a.nh[a.half0] + (a.halves > 1 ? a.nh[1] : 0));
    a.hist[nbk * a.tiles] = 0;
  }
}

// Puts the tile's picks at their places: each wave takes a quarter of the tile's tasks in order, and
// ranks its picks stably (ballot-matched peers in lane order on a running place per sub-key). LDS:
// a place per sub-key and wave.
__global__ __launch_bounds__(256) void route_place_kernel(RouteArgs a, int bits) {
  extern __shared__ int place[];  // [4][n]
  const int h = (int)(blockIdx.x / (unsigned)a.tiles), tile = (int)(blockIdx.x - (unsigned)h * a.tiles);
  const int half = a.half0 + (int)blockIdx.z, n = a.nh[half];
  for (int i = threadIdx.x; i < 4 * n; i += 256) place[i] = 0;
  __syncthreads();
  const int64_t t0 = (int64_t)tile * a.tpt;
  const int ntok = (int)(a.T - t0 < a.tpt ? a.T - t0 : a.tpt);
  const int items = ntok * a.K;
  const int l = lane_id(), wv = threadIdx.x >> 6;
  const int per = ((items + 3) / 4 + kWave - 1) / kWave * kWave;
  const int lo = wv * per, hi = lo + per < items ? lo + per : items;
  int* const mine = place + wv * n;
  const int32_t* const key = a.key + (int64_t)blockIdx.z * a.M;
  const float* const win = a.w + (int64_t)blockIdx.z * a.M;
  for (int q = lo + l; q < hi; q += kWave) {
    const int tok = q / a.K;
    const int k = key[((t0 + tok) * a.H + h) * a.K + (q - tok * a.K)];
    if (k >= 0) atomicAdd(&mine[k], 1);
  }
  __syncthreads();
  const int32_t* const hist = a.hist + bucket0(a, half, h) * a.tiles + tile;
  for (int i = threadIdx.x; i < n; i += 256) {
    int at = hist[(int64_t)i * a.tiles];
#pragma unroll
    for (int ww = 0; ww < 4; ++ww) {
      const int c = place[ww * n + i];
      place[ww * n + i] = at;
      at += c;
    }
  }
  __syncthreads();
  const uint64_t lt = lanemask_lt();
  for (int q0 = lo; q0 < hi; q0 += kWave) {
    const int q = q0 + l;
    const bool in = q < hi;
    const int tok = in ? q / a.K : 0;
    const int64_t p = ((t0 + tok) * a.H + h) * a.K + (in ? q - tok * a.K : 0);
    const int k = in ? key[p] : -1;
    const float w = in ? win[p] : 0.0f;
    const bool pick = k >= 0;
    uint64_t peers = __ballot(pick);
    for (int b = 0; b < bits; ++b) {
      const bool bit = (k >> b) & 1;
      const uint64_t bal = __ballot(bit);
      peers &= bit ? bal : ~bal;
    }
    const int before = __popcll(peers & lt);
    const int at = pick ? mine[k] : 0;
    wave_lds_sync();
    if (pick && before == 0) mine[k] = at + __popcll(peers);
    wave_lds_sync();
    if (pick) a.picks[at + before] = make_int2((int)(t0 + tok), __float_as_int(w));
  }
}

// Workgroups of the sum kernels are dealt to (half, slice) combinations c: workgroup b runs on XCD
// b % 8, so with c = b % 8 each XCD reads one half's 256-column slice of the rows it gathers
// (4 MB of key rows and 8 MB of token rows at the training shape, against a 4 MB L2) instead of all
// of them. More than eight combinations go in rounds of eight, unit by unit otherwise.
__device__ __forceinline__ void combo_of(int64_t b, int combos, int64_t per_combo, int* c,
                                         int64_t* unit) {
  if (combos % 8 == 0) {
    const int64_t round = b / (8 * per_combo), in = b - round * 8 * per_combo;
    *c = (int)(round * 8 + in % 8);
    *unit = in / 8;
  } else {
    *c = (int)(b % combos);
    *unit = b / combos;
  }
}

// dkeys[bucket] = sum over its picks (tokens ascending) of w x_t; one wave per bucket and
// 256-column slice, four elements a lane, sixteen token rows in flight. Every sub-key's row is
// written (zeros where it has no pick).
template <bool BF16>
__global__ __launch_bounds__(256) void route_keysum_kernel(RouteArgs a, int64_t per_combo) {
  typedef Quad<BF16> Q;
  typedef typename Q::raw raw;
  constexpr int G = 16;
  const int l = lane_id();
  const int combos = a.halves * a.slices;
  for (int64_t blk = blockIdx.x; blk < combos * per_combo; blk += gridDim.x) {
    int c;
    int64_t unit;
    combo_of(blk, combos, per_combo, &c, &unit);
    const int half = a.half0 + c / a.slices, q = (c % a.slices) * kWave + l;
    const int64_t r = unit * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (r >= (int64_t)a.H * a.nh[half]) continue;
    const int64_t bucket = bucket0(a, half, 0) + r;
    const int b = a.hist[bucket * a.tiles], e = a.hist[(bucket + 1) * a.tiles];
    const int rq = a.dkey / 4;
    const bool cv = q < rq;
    const int qc = cv ? q : rq - 1;
    const raw* const X = (const raw*)a.x + (half ? a.col0 / 4 : 0) + qc;
    const int64_t xq = a.d / 4;
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int64_t base = b; base < e; base += kWave) {  // (the step past the last pick may leave 32 bits)
      const int n = (int)(e - base < kWave ? e - base : kWave);
      const int2 pk = a.picks[base + (l < n ? l : n - 1)];
      const int tl = clamp_id(pk.x, a.T);
      for (int j0 = 0; j0 < n; j0 += G) {
        raw xr[G];
#pragma unroll
        for (int g = 0; g < G; ++g)
          xr[g] = X[(int64_t)readlane_i32(tl, j0 + g < n ? j0 + g : n - 1) * xq];
        __builtin_amdgcn_sched_barrier(0);  // all of the group's loads before its first product
#pragma unroll
        for (int g = 0; g < G; ++g) {
          if (j0 + g < n) {
            const float w = __int_as_float(readlane_i32(pk.y, j0 + g));
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[k] = fmaf(w, Q::at(xr[g], k), acc[k]);
          }
        }
      }
    }
    if (cv) *((f32x4_t*)a.dkeys[half] + r * rq + q) = acc;
  }
}

// dx_t += sum over t's picks of w keys[h, i]: one wave per token and slice of the round's halves
// (both halves of a shared query write the same columns, so one wave takes both). A batch of 64
// slots' picks is packed to the front lanes by a ballot, then eight key rows are in flight.
template <bool BF16>
__global__ __launch_bounds__(256) void route_dx_kernel(RouteArgs a, int64_t per_combo) {
  typedef Quad<BF16> Q;
  typedef typename Q::raw raw;
  constexpr int G = 8;
  const int l = lane_id();
  const bool both = a.col0 == 0 && a.halves > 1;
  const int combos = both ? a.slices : a.halves * a.slices;
  for (int64_t blk = blockIdx.x; blk < combos * per_combo; blk += gridDim.x) {
    int c;
    int64_t unit;
    combo_of(blk, combos, per_combo, &c, &unit);
    const int64_t t = unit * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (t >= a.T) continue;
    const int hk = a.H * a.K;
    const int q = (c % a.slices) * kWave + l, rq = a.dkey / 4;
    const bool cv = q < rq;
    const int qc = cv ? q : rq - 1;
    const int first = a.half0 + (both ? 0 : c / a.slices);
    f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
    for (int half = first; half <= first + (both ? 1 : 0); ++half) {
      const raw* const R = (const raw*)a.keys[half] + qc;
      const int n_half = a.nh[half];
      const int64_t o = (int64_t)(half - a.half0) * a.M + t * hk;
      for (int sb = 0; sb < hk; sb += kWave) {
        const int s = sb + l;
        const bool in = s < hk;
        const int k = in ? a.key[o + s] : -1;
        const float w = in ? a.w[o + s] : 0.0f;
        const int row = (in ? s / a.K : 0) * n_half + k;
        const uint64_t m = __ballot(k >= 0);
        const int n = __popcll(m);
        // lane j takes the j-th pick of the batch (slot order)
        const int dst = __popcll(m & lanemask_lt());
        const int rowp = __builtin_amdgcn_ds_permute((k >= 0 ? dst : 63) << 2, row);
        const int wp = __builtin_amdgcn_ds_permute((k >= 0 ? dst : 63) << 2, __float_as_int(w));
        for (int j0 = 0; j0 < n; j0 += G) {
          raw kr[G];
#pragma unroll
          for (int g = 0; g < G; ++g)
            kr[g] = R[(int64_t)readlane_i32(rowp, j0 + g < n ? j0 + g : n - 1) * rq];
          __builtin_amdgcn_sched_barrier(0);  // all of the group's loads before its first product
#pragma unroll
          for (int g = 0; g < G; ++g) {
            if (j0 + g < n) {
              const float wg = __int_as_float(readlane_i32(wp, j0 + g));
#pragma unroll
              for (int i = 0; i < 4; ++i) acc[i] = fmaf(wg, Q::at(kr[g], i), acc[i]);
            }
          }
        }
      }
    }
    if (cv) {
      f32x4_t* const out = (f32x4_t*)(a.dx + t * a.d + (first ? a.col0 : 0)) + q;
      *out += acc;
    }
  }
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
  const dim3 grid((unsigned)(a.piece_wgs + (a.cap + 4 * a.run - 1) / (4 * a.run)));
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

// cpl: 256-element pieces of a row, rounded up to a power of two (at most 16: d <= 4096; 8 in fp32: d <= 2048).
template <bool BF16>
hipError_t dispatch_bwd(int cpl, hipStream_t st, const BwdArgs& a) {
  switch (cpl) {
    case 1: launch_bwd<BF16, 1, 4>(st, a); break;
    case 2: launch_bwd<BF16, 2, 4>(st, a); break;
    case 4: launch_bwd<BF16, 4, 2>(st, a); break;
    case 8: launch_bwd<BF16, 8, 1>(st, a); break;
    case 16:
      if constexpr (BF16) {
        launch_bwd<BF16, 16, 1>(st, a);
        break;
      }
      [[fallthrough]];
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

namespace {

size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

// log2 of the tasks of a piece (see bwd_expert_kernel): at least 16, and at most 2048 pieces, the waves that
// the chip holds at the longest rows.
int piece_bits(int64_t M) {
  int b = 4;
  while ((M >> b) > 2048) ++b;
  return b;
}
int64_t piece_blocks(int64_t M) { return (M + (1ll << piece_bits(M)) - 1) >> piece_bits(M); }

}  // namespace

size_t backward_ws_bytes(const Shape& s) {
  const size_t n = (size_t)piece_blocks(s.M);
  return al256((size_t)s.M * 4) + al256(n * 4) + al256(n * 2 * s.d * 4);
}

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
  a.piece_bits = piece_bits(s.M);
  a.blocks = (int)piece_blocks(s.M);
  a.piece_row = (int32_t*)((char*)ws + al256((size_t)s.M * 4));
  a.piece_sum = (float*)((char*)a.piece_row + al256((size_t)a.blocks * 4));
  a.piece_wgs = (a.blocks + 31) / 32 * 8;
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
  a.score_wgs = (int)sb;
  const int64_t adds = (int64_t)(a.blocks + kPieceGroup - 1) / kPieceGroup * 2 * ((s.d + 1023) / 1024);
  hipLaunchKernelGGL(bwd_score_kernel, dim3((unsigned)(sb + adds)), dim3(256), 0, st, a);
  return hipGetLastError();
}

namespace {

constexpr int64_t kMaxBlocks = 1 << 22;  // past it the sum kernels walk the rest (a multiple of 8)

// Tokens per tile of the picks: about 4096 tasks, or 1024 where that leaves fewer than 512
// workgroups.
int route_tile_tokens(const Shape& s) {
  const int64_t tasks = 2 * s.M / 4096 < 512 ? 1024 : 4096;
  const int64_t t = (tasks + s.K - 1) / s.K;
  return (int)(t < s.T ? t : (s.T > 0 ? s.T : 1));
}

// Both halves go in one round while their picks can be numbered in 32 bits.
int route_halves(const Shape& s) { return 2 * s.M < (1ll << 31) - 1 ? 2 : 1; }

int64_t route_hist_len(const Shape& s) {
  const int64_t tpt = route_tile_tokens(s), tiles = (s.T + tpt - 1) / tpt;
  const int64_t keys = route_halves(s) == 2 ? s.nr + s.nc : (s.nr > s.nc ? s.nr : s.nc);
  return (int64_t)s.H * keys * tiles + 1;
}

}  // namespace

size_t route_backward_ws_bytes(const Shape& s) {
  const int64_t m = route_halves(s) * s.M, n = route_hist_len(s);
  return 2 * al256((size_t)m * 4) + al256((size_t)m * 8) + al256((size_t)n * 4) +
         al256((size_t)exclusive_scan_partials(n) * 4);
}

hipError_t launch_route_backward(const Shape& s, const void* x, const void* keys_row,
                                 const void* keys_col, const int32_t* idx, const float* dscores,
                                 float* dx, float* dkeys_row, float* dkeys_col, void* ws,
                                 hipStream_t st) {
  if (s.T == 0) return hipSuccess;
  const int halves = route_halves(s);
  const int64_t m = halves * s.M;
  RouteArgs a;
  char* w = (char*)ws;
  a.key = (int32_t*)w; w += al256((size_t)m * 4);
  a.w = (float*)w; w += al256((size_t)m * 4);
  a.picks = (int2*)w; w += al256((size_t)m * 8);
  a.hist = (int32_t*)w; w += al256((size_t)route_hist_len(s) * 4);
  int32_t* const partial = (int32_t*)w;
  a.idx = idx;
  a.ds = dscores;
  a.x = x;
  a.keys[0] = keys_row;
  a.keys[1] = keys_col;
  a.dkeys[0] = dkeys_row;
  a.dkeys[1] = dkeys_col;
  a.dx = dx;
  a.T = s.T;
  a.N = s.N;
  a.M = s.M;
  a.d = s.d;
  a.dkey = s.dk;
  a.col0 = s.col0;
  a.H = s.H;
  a.K = s.K;
  a.nh[0] = s.nr;
  a.nh[1] = s.nc;
  a.tpt = route_tile_tokens(s);
  a.tiles = (int)((s.T + a.tpt - 1) / a.tpt);
  a.halves = halves;
  a.slices = (s.dk / 4 + kWave - 1) / kWave;
  int P = 1;
  while (P < s.K && P < 16) P <<= 1;
  const int nmax = s.nr > s.nc ? s.nr : s.nc;
  int bits = 0;
  while ((1 << bits) < nmax) ++bits;
  for (a.half0 = 0; a.half0 < 2; a.half0 += halves) {
    const dim3 grid((unsigned)(a.tiles * s.H), 1, (unsigned)halves);
    const int64_t keys = halves == 2 ? s.nr + s.nc : a.nh[a.half0];
    hipLaunchKernelGGL(route_count_kernel, grid, dim3(256), (size_t)nmax * 4, st, a, P);
    hipError_t e = launch_exclusive_scan(a.hist, (int64_t)s.H * keys * a.tiles + 1, partial, st);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(route_place_kernel, grid, dim3(256), (size_t)nmax * 16, st, a, bits);
    const int64_t kper = ((int64_t)s.H * nmax + 3) / 4, tper = (s.T + 3) / 4;
    const int64_t kblocks = halves * a.slices * kper;
    const int64_t tblocks = (s.col0 == 0 && halves == 2 ? 1 : halves) * a.slices * tper;
    const dim3 kgrid((unsigned)std::min(kblocks, kMaxBlocks));
    const dim3 tgrid((unsigned)std::min(tblocks, kMaxBlocks));
    if (s.bf16) {
      hipLaunchKernelGGL(route_keysum_kernel<true>, kgrid, dim3(256), 0, st, a, kper);
      hipLaunchKernelGGL(route_dx_kernel<true>, tgrid, dim3(256), 0, st, a, tper);
    } else {
      hipLaunchKernelGGL(route_keysum_kernel<false>, kgrid, dim3(256), 0, st, a, kper);
      hipLaunchKernelGGL(route_dx_kernel<false>, tgrid, dim3(256), 0, st, a, tper);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace omnimoe
