// The expert stage in sweeps, for tables that the MALL holds and experts with several tasks each.
//
// Gathering a u or v row per task moves M rows past L2: at 20 tasks per expert that is 20 times the
// table, at the MALL's rate (7.3 TB/s). Here every XCD takes one eighth of the columns of all rows,
// every token's tasks are put in one pseudo-random order of the experts (64 buckets of a
// multiplicative hash), and all tokens walk through the buckets at the same time, so that the row
// eighths that they share are still in that XCD's 4 MB L2:
//   sweep_order  one wave per token: its tasks by bucket, stable;
//   sweep_dot    x . u over the XCD's columns for every task: eight partial sums per task;
//   sweep_act    a = g act(sum of the eight partial sums, in slice order);
//   sweep_sum    y = sum of a v in the sorted order, for the XCD's columns.
// The hash matters: a token's experts crowd into a few grid rows, so tokens that walked through the
// ids themselves would be at different places after as many tasks (sum of 4096 tokens, K = 512, on
// 320^2 experts of d = 1024: 501 us by id, 376 by hash). So does the pace: older waves are served
// first and run ahead, and a barrier of sixteen waves every 32 tasks holds them together (376 -> 270
// us, 16 TB/s; the slot-order sum takes 570). Every sum has a fixed order (no atomics), so y is the
// same on every run.
#include <type_traits>

#include "device_common.hpp"
#include "internal.hpp"

namespace omnimoe {
namespace {

constexpr int64_t kSweepMaxTableBytes = 256ll << 20;  // the MALL
constexpr int kSlices = 8;    // XCDs
constexpr int kBuckets = 64;  // one per lane
constexpr int kPace = 32;     // tasks between the barriers of a sixteen-wave workgroup

struct SweepArgs {
  const uint4* x;      // [T, chunks]
  const uint4* table;  // u or v [N, chunks], 16-byte chunks
  const int32_t* idx;
  const float* gates;
  const float* a;      // per task (sweep_order of a given a[]), or NULL
  int2* list;          // [T, hk] (expert, slot) or (expert, a), in bucket order
  float* part;         // [slice][T, hk]
  float* y;
  int64_t T;
  int64_t N;
  int64_t M;
  int hk;
  int chunks;          // 16-byte chunks of a row: kSlices LG
  int act;
};

__device__ __forceinline__ int clamp_e(int v, int64_t n) {
  return v < 0 ? 0 : (v >= n ? (int)(n - 1) : v);
}

// Stable counting sort of a token's tasks by bucket: counts, an exclusive scan over the lanes, and
// the places (peers of a bucket matched by ballots, in lane order on a running place).
__global__ __launch_bounds__(256) void sweep_order_kernel(SweepArgs a) {
  __shared__ int places[4][kBuckets];
  const int l = lane_id(), wv = threadIdx.x >> 6;
  int* const place = places[wv];
  const uint64_t lt = lanemask_lt();
  for (int64_t t = (int64_t)blockIdx.x * 4 + wv; t < a.T; t += (int64_t)gridDim.x * 4) {
    const int64_t p0 = t * a.hk;
    auto peers_of = [&](int s, int* e, int* b) {
      const bool in = s < a.hk;
      *e = in ? clamp_e(a.idx[p0 + s], a.N) : 0;
      *b = (int)(((uint32_t)*e * 0x9E3779B1u) >> 26);
      uint64_t peers = __ballot(in);
#pragma unroll
      for (int k = 0; k < 6; ++k) {
        const bool bit = (*b >> k) & 1;
        const uint64_t bal = __ballot(bit);
        peers &= bit ? bal : ~bal;
      }
      return in ? peers : 0ull;
    };
    place[l] = 0;
    wave_lds_sync();
    for (int sb = 0; sb < a.hk; sb += kWave) {
      int e, b;
      const uint64_t peers = peers_of(sb + l, &e, &b);
      if (peers && !(peers & lt)) place[b] += __popcll(peers);
      wave_lds_sync();
    }
    const int c = place[l];
    const int at = wave_excl_scan_i32(c);
    wave_lds_sync();
    place[l] = at;
    wave_lds_sync();
    for (int sb = 0; sb < a.hk; sb += kWave) {
      int e, b;
      const uint64_t peers = peers_of(sb + l, &e, &b);
      const int pos = peers ? place[b] + __popcll(peers & lt) : 0;
      wave_lds_sync();
      if (peers && !(peers & lt)) place[b] = pos + __popcll(peers);
      wave_lds_sync();
      if (peers)
        a.list[p0 + pos] = make_int2(e, a.a ? __float_as_int(a.a[p0 + sb + l]) : sb + l);
    }
    wave_lds_sync();
  }
}

// Lane j of every 16-lane row, broadcast within the row.
template <int J>
__device__ __forceinline__ int row_bcast(int v) {
  return __builtin_amdgcn_update_dpp(v, v, 0x150 + J, 0xF, 0xF, false);
}
template <int J0, int G, class F>
__device__ __forceinline__ void row_each(F&& f) {
  if constexpr (G > 0) {
    f(std::integral_constant<int, J0>());
    row_each<J0 + 1, G - 1>(f);
  }
}

// The next 16 entries' rows G at a time: every load of a group before the first use.
template <int G, class L, class U>
__device__ __forceinline__ void sixteen(L&& load, U&& use) {
  row_each<0, G>(load);
  __builtin_amdgcn_sched_barrier(0);
  row_each<0, G>(use);
  row_each<G, G>(load);
  __builtin_amdgcn_sched_barrier(0);
  row_each<G, G>(use);
  static_assert(2 * G == 16, "two groups");
}

// LG lanes hold a token's slice of columns (64 / LG tokens per wave); every 16-lane row reads the
// next 16 entries of its token's list, one per lane, and takes them eight at a time with their row
// slices in flight. Workgroup b runs on XCD b % 8 and takes slice b % 8. NW waves: four, or sixteen
// in step where the launch fills the chip. Row offsets fit in 32 bits (sweepable tables).
template <int LG, bool BF16, int NW>
__global__ __launch_bounds__(64 * NW, 8) void sweep_sum_kernel(SweepArgs a) {
  constexpr int EPC = BF16 ? 8 : 4, G = 8;
  constexpr int TPB = NW * (kWave / LG);  // tokens per workgroup
  const int l = lane_id();
  const int slice = blockIdx.x % kSlices;
  const int col = slice * LG + (l & (LG - 1));
  const uint32_t c0 = (uint32_t)col * 16u, rb = (uint32_t)a.chunks * 16u;
  const char* const V = (const char*)a.table;
  for (int64_t unit = blockIdx.x / kSlices; unit * TPB < a.T; unit += gridDim.x / kSlices) {
    const int64_t tt = unit * TPB + (threadIdx.x / LG);
    const int64_t t = tt < a.T ? tt : a.T - 1;
    const int2* const L = a.list + t * a.hk;
    float acc[EPC];
#pragma unroll
    for (int k = 0; k < EPC; ++k) acc[k] = 0.0f;
    int2 ent = L[(l & 15) < a.hk ? (l & 15) : a.hk - 1];
    for (int base = 0; base < a.hk; base += 16) {
      if (NW > 4 && base % kPace == 0) __builtin_amdgcn_s_barrier();
      const int2 cur = ent;
      const int nx = base + 16 + (l & 15);
      ent = L[nx < a.hk ? nx : a.hk - 1];
      const int left = a.hk - base;
      uint4 r[G];
      sixteen<G>(
          [&](auto J) {
            constexpr int j = decltype(J)::value;
            r[j % G] = *(const uint4*)(V + ((uint32_t)row_bcast<j>(cur.x) * rb + c0));
          },
          [&](auto J) {
            constexpr int j = decltype(J)::value;
            if (j >= left) return;  // past the end: loaded again, not added
            const float w = __int_as_float(row_bcast<j>(cur.y));
            const uint4 c = r[j % G];
            if constexpr (BF16) {
              acc[0] = fmaf(w, bf16_lo(c.x), acc[0]);
              acc[1] = fmaf(w, bf16_hi(c.x), acc[1]);
              acc[2] = fmaf(w, bf16_lo(c.y), acc[2]);
              acc[3] = fmaf(w, bf16_hi(c.y), acc[3]);
              acc[4] = fmaf(w, bf16_lo(c.z), acc[4]);
              acc[5] = fmaf(w, bf16_hi(c.z), acc[5]);
              acc[6] = fmaf(w, bf16_lo(c.w), acc[6]);
              acc[7] = fmaf(w, bf16_hi(c.w), acc[7]);
            } else {
              acc[0] = fmaf(w, __uint_as_float(c.x), acc[0]);
              acc[1] = fmaf(w, __uint_as_float(c.y), acc[1]);
              acc[2] = fmaf(w, __uint_as_float(c.z), acc[2]);
              acc[3] = fmaf(w, __uint_as_float(c.w), acc[3]);
            }
          });
    }
    if (tt < a.T) {
      float4* const yt = (float4*)a.y + (t * a.chunks + col) * (EPC / 4);
#pragma unroll
      for (int k = 0; k < EPC; k += 4)
        yt[k / 4] = make_float4(acc[k], acc[k + 1], acc[k + 2], acc[k + 3]);
    }
  }
}

template <int LG, bool BF16, int NW>
__global__ __launch_bounds__(64 * NW, 8) void sweep_dot_kernel(SweepArgs a) {
  constexpr int G = 8, TPB = NW * (kWave / LG);
  const int l = lane_id();
  const int slice = blockIdx.x % kSlices;
  const int col = slice * LG + (l & (LG - 1));
  const uint32_t c0 = (uint32_t)col * 16u, rb = (uint32_t)a.chunks * 16u;
  const char* const U = (const char*)a.table;
  float* const part = a.part + slice * a.M;
  for (int64_t unit = blockIdx.x / kSlices; unit * TPB < a.T; unit += gridDim.x / kSlices) {
    const int64_t tt = unit * TPB + (threadIdx.x / LG);
    const int64_t t = tt < a.T ? tt : a.T - 1;
    const int2* const L = a.list + t * a.hk;
    const uint4 xr = a.x[t * a.chunks + col];
    int ent = L[(l & 15) < a.hk ? (l & 15) : a.hk - 1].x;
    for (int base = 0; base < a.hk; base += 16) {
      if (NW > 4 && base % kPace == 0) __builtin_amdgcn_s_barrier();
      const int cur = ent;
      const int nx = base + 16 + (l & 15);
      ent = L[nx < a.hk ? nx : a.hk - 1].x;
      float mine = 0.0f;
      uint4 r[G];
      sixteen<G>(
          [&](auto J) {
            constexpr int j = decltype(J)::value;
            r[j % G] = *(const uint4*)(U + ((uint32_t)row_bcast<j>(cur) * rb + c0));
          },
          [&](auto J) {
            constexpr int j = decltype(J)::value;
            float v = chunk_dot<BF16>(r[j % G], xr, 0.0f);
            int x = __float_as_int(v);  // sum over the 16-lane row
            v += __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0xB1, 0xF, 0xF, false));
            x = __float_as_int(v);
            v += __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x4E, 0xF, 0xF, false));
            x = __float_as_int(v);
            v += __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x124, 0xF, 0xF, false));
            x = __float_as_int(v);
            v += __int_as_float(__builtin_amdgcn_update_dpp(x, x, 0x128, 0xF, 0xF, false));
            if ((l & 15) == j) mine = v;
          });
      // the group's rows of sixteen lanes hold their own sums of the same sixteen tasks
      if constexpr (LG >= 32) mine += __shfl_xor(mine, 16, kWave);
      if constexpr (LG >= 64) mine += __shfl_xor(mine, 32, kWave);
      const int i = base + (l & 15);
      if ((l & (LG - 1)) < 16 && tt < a.T && i < a.hk) part[t * a.hk + i] = mine;
    }
  }
}

// (expert, slot) becomes (expert, a): a = g act(x . u), the eight slices' sums added in order.
__global__ __launch_bounds__(256) void sweep_act_kernel(SweepArgs a) {
  const int64_t stride = (int64_t)gridDim.x * 256;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < a.M; i += stride) {
    float h = a.part[i];
#pragma unroll
    for (int s = 1; s < kSlices; ++s) h += a.part[s * a.M + i];
    const int2 e = a.list[i];
    const int64_t p = i / a.hk * a.hk + e.y;
    a.list[i] = make_int2(e.x, __float_as_int(a.gates[p] * activation(a.act, h)));
  }
}

SweepArgs sweep_args(const Shape& s) {
  SweepArgs a = {};
  a.T = s.T;
  a.N = s.N;
  a.M = s.M;
  a.hk = s.hk;
  a.chunks = s.bf16 ? s.d / 8 : s.d / 4;
  a.act = s.act;
  return a;
}

// Sixteen waves in step from here on (tokens times lanes per token): fewer leave compute units
// without a workgroup of that size. Sum, and dots and sum, of K = 512 on 320^2 experts of d = 1024: 1024 tokens
// 97 and 200 us with four waves, 169 and 355 with sixteen; 2048 tokens 178 and 362, 159 and 338.
constexpr int64_t kPacedLanes = 2048 * 16;

template <bool BF16, int LG>
void run_kernels(const SweepArgs& a, bool dot, hipStream_t st) {
  const bool paced = a.T * LG >= kPacedLanes;
  // as many workgroups as stay resident (32 waves per compute unit): every token's walk then starts
  // at the same time
  const int tpb = (paced ? 16 : 4) * (kWave / LG), cap = paced ? 64 : 256;
  const int64_t units = (a.T + tpb - 1) / tpb;
  const dim3 grid((unsigned)(kSlices * (units < cap ? units : cap)));
  if (dot && paced) hipLaunchKernelGGL((sweep_dot_kernel<LG, BF16, 16>), grid, dim3(1024), 0, st, a);
  else if (dot) hipLaunchKernelGGL((sweep_dot_kernel<LG, BF16, 4>), grid, dim3(256), 0, st, a);
  else if (paced) hipLaunchKernelGGL((sweep_sum_kernel<LG, BF16, 16>), grid, dim3(1024), 0, st, a);
  else hipLaunchKernelGGL((sweep_sum_kernel<LG, BF16, 4>), grid, dim3(256), 0, st, a);
}

template <bool BF16>
hipError_t run_sweep(const SweepArgs& a, bool dot, hipStream_t st) {
  switch (a.chunks / kSlices) {
    case 16: run_kernels<BF16, 16>(a, dot, st); break;
    case 32: run_kernels<BF16, 32>(a, dot, st); break;
    case 64: run_kernels<BF16, 64>(a, dot, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}
hipError_t run_sweep(const SweepArgs& a, bool bf16, bool dot, hipStream_t st) {
  return bf16 ? run_sweep<true>(a, dot, st) : run_sweep<false>(a, dot, st);
}

void run_order(const SweepArgs& a, hipStream_t st) {
  const int64_t blocks = (a.T + 3) / 4;
  hipLaunchKernelGGL(sweep_order_kernel, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256),
                     0, st, a);
}

size_t al256(size_t v) { return (v + 255) & ~(size_t)255; }

}  // namespace

bool sweepable(const Shape& s) {
  const int64_t chunks = s.bf16 ? s.d / 8 : s.d / 4;
  return s.T > 0 && (chunks == 128 || chunks == 256 || chunks == 512) &&
         s.N * chunks * 16 <= kSweepMaxTableBytes;
}

size_t sweep_stage_ws_bytes(const Shape& s, int64_t tokens) {
  return al256((size_t)s.M * 8) + al256((size_t)tokens * s.hk * 4 * kSlices);
}

hipError_t launch_sweep_sum(const Shape& s, const void* v, const int32_t* idx, const float* abuf,
                            float* y, void* ws, hipStream_t st) {
  if (s.T == 0) return hipSuccess;
  SweepArgs a = sweep_args(s);
  a.idx = idx;
  a.a = abuf;
  a.list = (int2*)ws;
  run_order(a, st);
  a.table = (const uint4*)v;
  a.y = y;
  return run_sweep(a, s.bf16, false, st);
}

hipError_t launch_sweep_order(const Shape& s, const int32_t* idx, void* ws, hipStream_t st) {
  SweepArgs a = sweep_args(s);
  a.idx = idx;
  a.list = (int2*)ws;
  run_order(a, st);
  return hipGetLastError();
}

hipError_t launch_sweep_dot(const Shape& s, int64_t tokens, const void* x, const void* u,
                            const float* gates, void* ws, hipStream_t st) {
  SweepArgs a = sweep_args(s);
  a.part = (float*)((char*)ws + al256((size_t)s.M * 8));
  a.table = (const uint4*)u;
  for (int64_t t0 = 0; t0 < s.T; t0 += tokens) {
    a.T = s.T - t0 < tokens ? s.T - t0 : tokens;
    a.M = a.T * s.hk;
    a.x = (const uint4*)x + t0 * a.chunks;
    a.gates = gates + t0 * s.hk;
    a.list = (int2*)ws + t0 * s.hk;
    hipError_t e = run_sweep(a, s.bf16, true, st);
    if (e != hipSuccess) return e;
    const int64_t blocks = (a.M + 255) / 256;
    hipLaunchKernelGGL(sweep_act_kernel, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0,
                       st, a);
  }
  return hipGetLastError();
}

hipError_t launch_sweep_sorted_sum(const Shape& s, const void* v, float* y, void* ws,
                                   hipStream_t st) {
  SweepArgs a = sweep_args(s);
  a.list = (int2*)ws;
  a.table = (const uint4*)v;
  a.y = y;
  return run_sweep(a, s.bf16, false, st);
}

}  // namespace omnimoe
