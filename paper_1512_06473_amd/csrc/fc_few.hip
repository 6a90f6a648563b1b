// PQ fully-connected layer straight from the caller's code stream, a lane per
// output channel; the layers' dispatch.
//
// Paper: Sec. 3.1, Eq. (5): T(c_t) = sum_m L[m][ k_m(c_t) ].
//
// With many images a code serves a whole wave and is re-laid for that
// (fc_tiled).  With a few the codes are the work (fc6: 9.4 million, one table
// read each), and re-laying them costs more than the layer.  Here a lane owns
// an output channel and up to four images: it reads its row of the stream
// (bytes or packed, 32 codes at a time, shifted to the row's first bit so that
// every code's place is a constant), and the lanes of a wave look up the same
// subspace's table row at once.  A row of K <= 64 fp32 entries spans at most
// 64 banks and equal codes share an address, so one image's lookups are free
// of bank conflicts.
//
// A workgroup of 256 lanes owns 256 channels and some groups of 32 subspaces,
// whose tables [subspace][2^bits][images] it builds in LDS (entries past K
// repeat the last one, subspaces past M are 0, so only a byte code needs a
// check).  The groups are split over workgroups to fill the chip; a second
// kernel adds the splits in order.
//
// Bound by the chain codeword loads -> table -> code loads -> lookups with 4 to
// 8 waves per CU and by the two launches, not by bytes (fc6 for one image: 5.9
// MB of packed codes, 1 us).  fc6, one image, packed codes per call: 64 us with
// fc_tiled and its re-layout, 16 us here, of which the kernel is 12 (23 with
// one table entry per lane in flight) and the sum of the splits 3.  The kernel
// that took K > 64 and C's > 8 before read each code for 64 lanes: 1024 to
// 1024, C's = 16, one image 221 -> 12 us, 128 images 240 -> 17 us; 25088 to
// 4096, K = 256, one image 6200 -> 102 us, 128 images 12000 -> 7200 us.
#include <type_traits>

#include "qcnn_internal.h"

namespace qcnn {
namespace {

constexpr int kThreads = 256;
constexpr int kGroup = 32;      // subspaces per group
constexpr int kBuild = 8;       // table entries a lane builds at once
constexpr size_t kTableBytes = 64 * 1024;  // of a workgroup's tables, where one group takes less: two workgroups per CU

struct FewParams {
  int N, Cs, M, K, Csp, Ct;
  int ni, tblocks;   // images per workgroup; blocks of 256 channels
  long long blocks;  // channel blocks x image blocks
  int lb;            // log2 of a table row's entries
  int groups;        // groups of 32 subspaces per workgroup
  int fit;           // of them in LDS at a time
  int splits;
  long long dwords;  // of the code stream
  int relu;
  int vec;  // 4: sub-codewords and inputs are whole 16-byte loads, else 1
};

template <int V>
__device__ inline void load_vec(const float* __restrict__ at, float (&v)[V]) {
  if constexpr (V == 4) {
    const float4 f = *reinterpret_cast<const float4*>(at);
    v[0] = f.x, v[1] = f.y, v[2] = f.z, v[3] = f.w;
  } else {
    v[0] = at[0];
  }
}

// BITS: of the code stream (0: K = 1, every code 0); NI: images per workgroup (1, 2 or 4).
template <int BITS, int NI>
__global__ __launch_bounds__(kThreads) void fc_few_kernel(const float* __restrict__ x, const float* __restrict__ D,
                                                        CodeStream codes, const float* __restrict__ bias,
                                                        float* __restrict__ y, float* __restrict__ partial,
                                                        FewParams p) {
  extern __shared__ float lut[];  // [32 groups][2^lb][NI]
  const int tid = threadIdx.x, t = (blockIdx.x % p.tblocks) * kThreads + tid;
  const int split = blockIdx.y, n0 = (blockIdx.x / p.tblocks) * NI;
  const int m0 = split * p.groups * kGroup;
  const int ng = min(p.groups, (p.M - m0 + kGroup - 1) / kGroup);
  const int row = 1 << p.lb;

  // this lane's first codes on their way while the tables are built
  constexpr int WORDS = kGroup * BITS / 32;  // dwords of a group
  const uint32_t* w = reinterpret_cast<const uint32_t*>(codes.p);
  const long long bit0 = ((long long)(t < p.Ct ? t : 0) * p.M + m0) * BITS;
  const uint32_t sh = (uint32_t)(bit0 & 31);
  uint32_t cur[WORDS + 1], nxt[WORDS + 1];
  auto load = [&](int g, uint32_t (&v)[WORDS + 1]) {
    if (BITS == 0) return;  // K = 1: no stream
    const long long at = (bit0 >> 5) + (long long)g * WORDS;
#pragma unroll
    for (int i = 0; i <= WORDS; ++i) v[i] = w[min(at + i, p.dwords - 1)];
  };
  load(0, cur);

  // kBuild entries in flight per lane: their codewords and inputs arrive in one
  // wait (one at a time, the build took more than the layer).
  auto build = [&](auto vec, int mb, int total) {
    constexpr int V = decltype(vec)::value;  // elements per load
    for (int b0 = 0; b0 < total; b0 += kThreads * kBuild) {
      const int e0 = b0 + tid;
      float s[kBuild][NI];
#pragma unroll
      for (int u = 0; u < kBuild; ++u)
#pragma unroll
        for (int i = 0; i < NI; ++i) s[u][i] = 0.f;
      const int csp = mb + (b0 >> p.lb) < p.M ? p.Csp : 0;  // nothing to load past the last subspace
      for (int j = 0; j < csp; j += V) {
        float dv[kBuild][V], xv[kBuild][NI][V];
#pragma unroll
        for (int u = 0; u < kBuild; ++u) {
          const int e = min(e0 + u * kThreads, total - 1);
          const int m = min(mb + (e >> p.lb), p.M - 1), k = min(e & (row - 1), p.K - 1);
          load_vec<V>(D + ((size_t)m * p.K + k) * p.Csp + j, dv[u]);
#pragma unroll
          for (int i = 0; i < NI; ++i)
            load_vec<V>(x + (size_t)min(n0 + i, p.N - 1) * p.Cs + (size_t)m * p.Csp + j, xv[u][i]);
        }
#pragma unroll
        for (int u = 0; u < kBuild; ++u)
#pragma unroll
          for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int v = 0; v < V; ++v) s[u][i] = fmaf(dv[u][v], xv[u][i][v], s[u][i]);
      }
#pragma unroll
      for (int u = 0; u < kBuild; ++u) {
        const int e = e0 + u * kThreads;
        if (e >= total) break;
#pragma unroll
        for (int i = 0; i < NI; ++i) lut[e * NI + i] = mb + (e >> p.lb) < p.M ? s[u][i] : 0.f;
      }
    }
  };
  // four sums per image, subspaces 4 q + r into sum r: short chains
  float acc[NI][4];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[i][r] = 0.f;
  const uint32_t kmax = (uint32_t)(p.K - 1);
  for (int g = 0; g < ng; ++g) {
    const int at = g % p.fit;
    if (at == 0) {  // the next groups' tables
      if (g) __syncthreads();
      const int mb = m0 + g * kGroup, total = min(p.fit, ng - g) * kGroup * row;
      if (p.vec == 4)
        build(std::integral_constant<int, 4>{}, mb, total);
      else
        build(std::integral_constant<int, 1>{}, mb, total);
      __syncthreads();
    }
    if (g + 1 < ng) load(g + 1, nxt);
    uint32_t a[WORDS + 1];
#pragma unroll
    for (int i = 0; i < WORDS; ++i) a[i] = __builtin_amdgcn_alignbit(cur[i + 1], cur[i], sh);
    a[WORDS] = 0;
    const float* base = lut + (size_t)at * kGroup * row * NI;
#pragma unroll
    for (int c = 0; c < kGroup; ++c) {
      constexpr uint32_t mask = (1u << BITS) - 1u;
      const int bit = c * BITS, lo = bit >> 5, off = bit & 31;
      uint32_t code = BITS ? a[lo] >> off : 0u;
      if (off + BITS > 32) code = __builtin_amdgcn_alignbit(a[lo + 1], a[lo], off);
      code &= mask;
      if (BITS == 8) code = min(code, kmax);
      const float* entry = base + ((c << p.lb) + (int)code) * NI;
      if constexpr (NI == 1) {
        acc[0][c & 3] += entry[0];
      } else if constexpr (NI == 2) {
        const float2 v = *reinterpret_cast<const float2*>(entry);
        acc[0][c & 3] += v.x;
        acc[1][c & 3] += v.y;
      } else {
        const float4 v = *reinterpret_cast<const float4*>(entry);
        acc[0][c & 3] += v.x;
        acc[1][c & 3] += v.y;
        acc[2][c & 3] += v.z;
        acc[3][c & 3] += v.w;
      }
    }
#pragma unroll
    for (int i = 0; i <= WORDS; ++i) cur[i] = nxt[i];
  }
  if (t >= p.Ct) return;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    if (n0 + i >= p.N) break;
    float v = (acc[i][0] + acc[i][1]) + (acc[i][2] + acc[i][3]);
    if (partial) {
      partial[((size_t)split * p.N + n0 + i) * p.Ct + t] = v;
    } else {
      v += bias ? bias[t] : 0.f;
      if (p.relu) v = fmaxf(v, 0.f);
      y[(size_t)(n0 + i) * p.Ct + t] = v;
    }
  }
}

// y = sum over splits (in split order, sixteen loads in flight) + bias, then ReLU.
__global__ __launch_bounds__(64) void fc_few_reduce_kernel(const float* __restrict__ partial, FewParams p,
                                                         const float* __restrict__ bias, float* __restrict__ y) {
  const int i = blockIdx.x * 64 + threadIdx.x, total = p.N * p.Ct;
  if (i >= total) return;
  const float b = bias ? bias[i % p.Ct] : 0.f;
  float s = 0.f;
  for (int k0 = 0; k0 < p.splits; k0 += 16) {
    float v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = k0 + u < p.splits ? partial[(size_t)(k0 + u) * total + i] : 0.f;
#pragma unroll
    for (int u = 0; u < 16; ++u) s += v[u];
  }
  s += b;
  if (p.relu) s = fmaxf(s, 0.f);
  y[i] = s;
}

size_t few_group_bytes(const FewParams& p) { return ((size_t)kGroup << p.lb) * p.ni * sizeof(float); }

template <int BITS>
void (*few_kernel(int ni))(const float*, const float*, CodeStream, const float*, float*, float*, FewParams) {
  return ni == 1 ? fc_few_kernel<BITS, 1> : ni == 2 ? fc_few_kernel<BITS, 2> : fc_few_kernel<BITS, 4>;
}

}  // namespace

namespace {

// A workgroup for every CU where that leaves each a group, and no more: a
// workgroup with more groups than its table holds takes them in turns, so the
// partial sums stay near 1 MB whatever the layer.
FewParams few_plan(int N, int Cs, int M, int K, int Csp, int Ct) {
  FewParams p{};
  p.N = N, p.Cs = Cs, p.M = M, p.K = K, p.Csp = Csp, p.Ct = Ct;
  p.lb = code_bits(K);
  p.ni = N == 1 ? 1 : N == 2 ? 2 : 4;
  p.tblocks = ceil_div(Ct, kThreads);
  p.blocks = (long long)p.tblocks * ceil_div(N, p.ni);
  const int all = ceil_div(M, kGroup);
  p.groups = ceil_div(all, (int)std::max<long long>(1, 256 / p.blocks));
  // a layer that fc_tiled computes without scratch needs none here either
  if (fc_tiled_splits(N, Cs, M, K, Csp, Ct) == 1) p.groups = all;
  p.splits = ceil_div(all, p.groups);
  p.fit = std::min(p.groups, (int)std::max<size_t>(1, kTableBytes / few_group_bytes(p)));
  return p;
}

}  // namespace

// A group of 32 subspaces costs a workgroup 3 us at K = 32, C's = 4 and four
// images (5 us with its codes and codebooks not in the caches, as between the
// layers of a network), of which the table is a third, on top of 10 us;
// fc_tiled takes 28 us and 1 us more per 75 subspaces however few its images
// are.  The line lies where the dearer of the two figures meets it.  us, plan
// call, fc_tiled -> this kernel: fc6 (9216 to 4096) with 8 images, 9 groups in a
// row, 60 -> 36; 12 images, 15 groups, 60 -> 58.  4096 to 1000: 32 images, 4
// groups, 39 -> 21; 64, 8 groups, 40 -> 33 when repeated but 40 -> 50 in a
// network, so fc_tiled's.  2048 to 512, C's = 8, K = 64, 128 images: 2 groups,
// 29 -> 21.  Where fc_tiled does not go (K > 64 or C's > 8) this is the only
// kernel.
bool fc_few_better(int N, int Cs, int M, int K, int Csp, int Ct) {
  if (!fc_tiled_supported(N, Cs, M, K, Csp, Ct)) return true;
  const FewParams p = few_plan(N, Cs, M, K, Csp, Ct);
  const double rounds = (double)((p.blocks * p.splits + 255) / 256);
  return rounds * p.groups * (2.0 + (double)(Csp << p.lb) / 128.0) / 3.0 <= 3.5 + M / 400.0;
}

hipError_t launch_fc_few(int N, int Cs, int M, int K, int Csp, int Ct, const float* x, const float* D,
                         CodeStream codes, const float* bias, int relu, float* y, hipStream_t stream) {
  FewParams p = few_plan(N, Cs, M, K, Csp, Ct);
  p.relu = relu;
  p.dwords = ((long long)Ct * M * codes.bits + 31) / 32;
  p.vec = Csp % 4 == 0 && Cs % 4 == 0 && (((uintptr_t)x | (uintptr_t)D) & 15) == 0 ? 4 : 1;
  const int ni = p.ni;
  if (p.blocks > (1LL << 31) - 1 || few_group_bytes(p) > kLdsBytes) return hipErrorInvalidConfiguration;
  void (*kern)(const float*, const float*, CodeStream, const float*, float*, float*, FewParams) = nullptr;
  switch (codes.bits) {
    case 0: kern = few_kernel<0>(ni); break;
    case 1: kern = few_kernel<1>(ni); break;
    case 2: kern = few_kernel<2>(ni); break;
    case 3: kern = few_kernel<3>(ni); break;
    case 4: kern = few_kernel<4>(ni); break;
    case 5: kern = few_kernel<5>(ni); break;
    case 6: kern = few_kernel<6>(ni); break;
    case 7: kern = few_kernel<7>(ni); break;
    default: kern = few_kernel<8>(ni); break;
  }
  hipError_t e = allow_max_lds((const void*)kern);
  if (e != hipSuccess) return e;
  float* partial = nullptr;
  Scratch scratch;
  if (p.splits > 1) {
    if ((e = scratch.acquire(stream, (size_t)p.splits * N * Ct * sizeof(float))) != hipSuccess) return e;
    partial = reinterpret_cast<float*>(scratch.get());
  }
  {
    LaunchTimer timer;
    e = timed_launch(&timer, kern, dim3((unsigned)p.blocks, p.splits), dim3(kThreads),
                     (uint32_t)(p.fit * few_group_bytes(p)), stream, x, D, codes, bias, y, partial, p);
  }
  if (e == hipSuccess && partial) {
    hipLaunchKernelGGL(fc_few_reduce_kernel, dim3((unsigned)ceil_div(N * Ct, 64)), dim3(64), 0, stream,
                       (const float*)partial, p, bias, y);
    e = hipGetLastError();
  }
  return e;
}

bool fc_relays(int N, int Cs, int M, int K, int Csp, int Ct) { return !fc_few_better(N, Cs, M, K, Csp, Ct); }

hipError_t launch_fc_forward(int N, int Cs, int M, int K, int Csp, int Ct, const float* x, const float* D,
                             CodeStream codes, const float* bias, int relu, float* y, hipStream_t stream) {
  auto launch = fc_relays(N, Cs, M, K, Csp, Ct) ? launch_fc_tiled
                : !fc_tiled_supported(N, Cs, M, K, Csp, Ct) && fc_pq_better(N, M, K, Csp, Ct) ? launch_fc_pq
                                                                                              : launch_fc_few;
  return launch(N, Cs, M, K, Csp, Ct, x, D, codes, bias, relu, y, stream);
}

}  // namespace qcnn
