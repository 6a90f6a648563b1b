// Error-corrected quantization of a convolutional layer.
//
// Paper: Sec. 3.3.2 (Eq. (13)) and App. B (Eq. (14)-(21)).  With the input
// maps S_n and desired responses T_n of N images, the sub-codebooks D^(m)
// (shared by every kernel position p) and the assignments k(c, p) minimise
// the response error by block coordinate descent over the subspaces; for
// subspace m, with R the residual of the other subspaces (Eq. (15)):
//   * sub-codewords k = 0 .. K-1 in order (Eq. (17)-(19)): D_k becomes the
//     least-squares fit, over images, output positions and channels, of the
//     residual without the other sub-codewords' terms;
//   * kernel positions p = 0 .. d_k^2 - 1 in order (Eq. (20)-(21)): each
//     channel takes the sub-codeword of least error for the residual without
//     the other positions' terms, tried exhaustively.
// Readings: Q_k of Eq. (18) takes out, per channel, the positions whose
// sub-codeword is not k, and Eq. (19) sums over the channels with a position
// on k; P of Eq. (20) takes out every other position p' (paired with its own
// input position); p_s = p_t s - pad + p (no flip), S = 0 outside the input;
// normal equations with the pivot rule of the FC case; ties to the lowest k.
//
// Both updates see the large arrays only through two small summaries of
// subspace m, with s_p(n, o) the input sub-vector that position p meets at
// output o of image n:
//   G[p][p'] = sum_{n,o} s_p s_p'^T          ([d_k^2][d_k^2][C'_s][C'_s], once)
//   H[c][p]  = sum_{n,o} s_p R(c)             ([C_t][d_k^2][C'_s], per step)
// Eq. (19) for k is then sum_{(c,p) on k} (sum_{p' on k} G[p][p']) D_k =
// sum_{(c,p) on k} (H[c][p] - sum_{p' not on k} G[p][p'] D_{k(c,p')}), and the
// error of Eq. (21) for (c, p) and candidate k is, up to a constant,
// D_k^T G[p][p] D_k - 2 D_k^T (H[c][p] - sum_{p' != p} G[p][p'] D_{k(c,p')}).
//
// State, float64: the residual of the whole layer E = T - Y [N][C_t][O]
// (O = H_o W_o), D64, G, and the codes as [M][C_t][d_k^2].  Per subspace:
//   ecc_pass_kernel   E -= the change of the subspace fitted before (from
//                     its delta[c][p] = D_new[k_new] - D_old[k_old]); block
//                     sums of E^2 (the objective after that step); and, while
//                     E is in registers, partial sum_{n,o} s_p E(c) of this
//                     subspace per chunk of outputs (ecc_apply_kernel and
//                     ecc_corr_kernel where a map does not fit);
//   ecc_reduce_kernel H = the partials in chunk order + sum_p' G[p][p'] W(c, p')
//                     (so H is taken against R = E + this subspace's terms);
//   ecc_rows_kernel   one workgroup per sub-codeword k: its row of the linear
//                     system below;
//   ecc_solve_kernel  one workgroup: Eq. (17)-(19), the sub-codewords in
//                     order, by substitution in those rows;
//   ecc_bupdate_kernel one wave per channel: Eq. (20)-(21), the positions in
//                     order; after the last of `inner` rounds, delta for the
//                     next apply.
#include "qcnn_internal.h"

namespace qcnn {
namespace {

constexpr int kCThreads = 256;

struct EccParams {
  int N, Cs, H, W, Ct, Ho, Wo, dk, stride, pad, M, K, Csp, P, O;
  int chunk, nchunks;  // images per correlation chunk, number of chunks
};

// Fixed-order sum of one value per thread into opart[block].
__device__ __forceinline__ void ecc_block_sum(double v, double* red, double* __restrict__ opart) {
  for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_down(v, off, kWave);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kCThreads / kWave; ++w) s += red[w];
    opart[blockIdx.x] = s;
  }
}

// D64 = codebooks; ct[m][c][p] = codes[c][p][m] (codes >= K read as K - 1).
__global__ __launch_bounds__(kCThreads) void ecc_init_kernel(const float* __restrict__ D,
                                                           const uint8_t* __restrict__ codes, EccParams q,
                                                           double* __restrict__ D64, uint8_t* __restrict__ ct) {
  const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
  const size_t nd = (size_t)q.M * q.K * q.Csp, nc = (size_t)q.M * q.Ct * q.P;
  for (size_t i = tid; i < nd; i += stride) D64[i] = (double)D[i];
  for (size_t i = tid; i < nc; i += stride) {
    const size_t m = i / ((size_t)q.Ct * q.P), cp = i % ((size_t)q.Ct * q.P);
    const uint8_t k = codes[cp * q.M + m];
    ct[i] = k < q.K ? k : (uint8_t)(q.K - 1);
  }
}

// G[m][p][p'][i][j] = sum over n, o (in order) of s_p[i] s_p'[j].
__global__ __launch_bounds__(kCThreads) void ecc_gram_kernel(const float* __restrict__ S, EccParams q,
                                                           double* __restrict__ G) {
  const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  const size_t per_m = (size_t)q.P * q.P * q.Csp * q.Csp;
  if (i0 >= (size_t)q.M * per_m) return;
  const int m = (int)(i0 / per_m);
  size_t r = i0 % per_m;
  const int j = (int)(r % q.Csp);
  r /= q.Csp;
  const int i = (int)(r % q.Csp);
  r /= q.Csp;
  const int p2 = (int)(r % q.P), p = (int)(r / q.P);
  // output positions whose two input positions both lie inside the input
  // (the others add exact zeros)
  const int ky = p / q.dk, kx = p - ky * q.dk, ky2 = p2 / q.dk, kx2 = p2 - ky2 * q.dk;
  const size_t HW = (size_t)q.H * q.W;
  double s = 0.0;
  for (int n = 0; n < q.N; ++n) {
    const float* si = S + ((size_t)n * q.Cs + (size_t)m * q.Csp + i) * HW;
    const float* sj = S + ((size_t)n * q.Cs + (size_t)m * q.Csp + j) * HW;
    for (int yo = 0; yo < q.Ho; ++yo) {
      const int y = yo * q.stride - q.pad + ky, y2 = yo * q.stride - q.pad + ky2;
      if ((unsigned)y >= (unsigned)q.H || (unsigned)y2 >= (unsigned)q.H) continue;
      for (int xo0 = 0; xo0 < q.Wo; xo0 += 8) {  // eight positions' loads in flight, added in order
        float a[8], b[8];
        bool ok[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int xo = xo0 + u;
          const int x = xo * q.stride - q.pad + kx, x2 = xo * q.stride - q.pad + kx2;
          ok[u] = xo < q.Wo && (unsigned)x < (unsigned)q.W && (unsigned)x2 < (unsigned)q.W;
          const float va = si[ok[u] ? y * q.W + x : 0], vb = sj[ok[u] ? y2 * q.W + x2 : 0];
          a[u] = va;
          b[u] = vb;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
          if (ok[u]) s += (double)a[u] * (double)b[u];
      }
    }
  }
  G[i0] = s;
}

// The same blocks on v_mfma_f64_16x16x4_f64, for (p, j) up to 64: G_m = X X^T
// with X [(p, j)][(n, o)], one lane value serving as A operand of its row tile
// and as B operand of its column tile.  A workgroup (m, chunk) takes the chunk's
// images with their maps in LDS, wave w every fourth 16-position tile; the
// waves' sums are added in order into gpart[chunk][m][(p, j)][(p', i)], the
// chunks by ecc_gram_sum_kernel.  660 us as one thread per entry at 256
// channels, 32 x 13 x 13, 3x3, C's = 4.
typedef double d4v __attribute__((ext_vector_type(4)));
constexpr int kMaxGramTiles = 4;
constexpr int kGramChunks = 8;

template <int NT>
__global__ __launch_bounds__(kCThreads) void ecc_gram_mfma_kernel(const float* __restrict__ S, EccParams q, int pw,
                                                                int plane, double* __restrict__ gpart) {
  extern __shared__ float smf[];
  constexpr int NW = kCThreads / kWave;
  const int QN = q.P * q.Csp, size = q.Csp * plane, tiles = (q.O + 15) / 16;
  double* sums = reinterpret_cast<double*>(smf);           // [16 NT][16 NT]
  float* map = smf + 2 * (16 * NT) * (16 * NT);            // one image's maps, zero halos, then one zero
  int* ooff = reinterpret_cast<int*>(map + size + 1);      // [16 tiles]
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int m = blockIdx.x, chunk = blockIdx.y;
  const int n0 = (int)((long long)q.N * chunk / kGramChunks), n1 = (int)((long long)q.N * (chunk + 1) / kGramChunks);
  const size_t HW = (size_t)q.H * q.W;
  const int col = lane & 15, quad = lane >> 4;
  int qoff[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int i = 16 * t + col, p = i / q.Csp, j = i - p * q.Csp;
    qoff[t] = i < QN ? j * plane + (p / q.dk) * pw + p % q.dk : -1;
  }
  for (int i = tid; i < 16 * tiles; i += kCThreads)
    ooff[i] = i < q.O ? (i / q.Wo) * q.stride * pw + (i % q.Wo) * q.stride : -1;
  d4v g[NT][NT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < NT; ++b) g[a][b] = d4v{0.0, 0.0, 0.0, 0.0};
  for (int n = n0; n < n1; ++n) {
    __syncthreads();
    for (int i = tid; i <= size; i += kCThreads) {
      const int j = min(i, size - 1) / plane, r = i - j * plane;
      const int y = r / pw - q.pad, x = r % pw - q.pad;
      const bool in = i < size && (unsigned)y < (unsigned)q.H && (unsigned)x < (unsigned)q.W;
      map[i] = in ? S[((size_t)n * q.Cs + (size_t)m * q.Csp + j) * HW + (size_t)y * q.W + x] : 0.f;
    }
    __syncthreads();
    for (int t = wave; t < tiles; t += NW)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) {
        const int o = ooff[16 * t + 4 * kk + quad];
        double v[NT];
#pragma unroll
        for (int a = 0; a < NT; ++a) v[a] = (double)map[o >= 0 && qoff[a] >= 0 ? o + qoff[a] : size];
#pragma unroll
        for (int a = 0; a < NT; ++a)
#pragma unroll
          for (int b = 0; b < NT; ++b) g[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(v[a], v[b], g[a][b], 0, 0, 0);
      }
  }
  for (int w = 0; w < NW; ++w) {
    if (wave == w)
#pragma unroll
      for (int a = 0; a < NT; ++a)
#pragma unroll
        for (int b = 0; b < NT; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            double* at = sums + (16 * a + 4 * i + quad) * 16 * NT + 16 * b + col;
            *at = w == 0 ? g[a][b][i] : *at + g[a][b][i];
          }
    __syncthreads();
  }
  for (int i = tid; i < QN * QN; i += kCThreads)
    gpart[((size_t)chunk * q.M + m) * QN * QN + i] = sums[i / QN * 16 * NT + i % QN];
}

// G[m][p][p'][i][j] = the chunks' sums in order.
__global__ __launch_bounds__(kCThreads) void ecc_gram_sum_kernel(const double* __restrict__ gpart, EccParams q,
                                                               double* __restrict__ G) {
  const size_t i0 = (size_t)blockIdx.x * kCThreads + threadIdx.x, QN = (size_t)q.P * q.Csp, total = q.M * QN * QN;
  if (i0 >= total) return;
  double s = 0.0;
#pragma unroll
  for (int c = 0; c < kGramChunks; ++c) s += gpart[c * total + i0];
  const size_t m = i0 / (QN * QN), r = i0 % (QN * QN);
  const size_t row = r / QN, col = r % QN;  // (p, i), (p', j)
  G[(((m * q.P + row / q.Csp) * q.P + col / q.Csp) * q.Csp + row % q.Csp) * q.Csp + col % q.Csp] = s;
}

// LDS of the MFMA form, or 0 when the (p, j) or a map does not fit it.
size_t gram_lds_bytes(const EccParams& q) {
  const int nt = (q.P * q.Csp + 15) / 16;
  const long long plane = (long long)((q.Ho - 1) * q.stride + q.dk) * ((q.Wo - 1) * q.stride + q.dk);
  if (nt > kMaxGramTiles || plane * q.Csp * 4 > 32 * 1024) return 0;
  return (size_t)(16 * nt) * (16 * nt) * 8 + ((size_t)plane * q.Csp + 1) * 4 + (size_t)16 * ((q.O + 15) / 16) * 4;
}

hipError_t launch_gram(const float* S, const EccParams& q, size_t lds, double* gpart, double* G, hipStream_t stream) {
  const int pw = (q.Wo - 1) * q.stride + q.dk, plane = ((q.Ho - 1) * q.stride + q.dk) * pw;
  const dim3 grid((unsigned)q.M, kGramChunks);
  const int nt = (q.P * q.Csp + 15) / 16;
  auto gram = nt == 1 ? ecc_gram_mfma_kernel<1> : nt == 2 ? ecc_gram_mfma_kernel<2> : nt == 3 ? ecc_gram_mfma_kernel<3>
                                                                                               : ecc_gram_mfma_kernel<4>;
  hipError_t e = allow_max_lds((const void*)gram);  // sums 32 KB, maps 32 KB, offsets of up to 8192 outputs 32 KB
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(gram, grid, dim3(kCThreads), lds, stream, S, q, pw, plane, gpart);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const size_t total = (size_t)q.M * q.P * q.P * q.Csp * q.Csp;
  hipLaunchKernelGGL(ecc_gram_sum_kernel, dim3((unsigned)ceil_div_z(total, kCThreads)), dim3(kCThreads), 0, stream,
                     (const double*)gpart, q, G);
  return hipGetLastError();
}

// E = T - sum_m sum_p D^(m)[k(c, p)]^T s_p as a float64 implicit GEMM on
// MFMA (v_mfma_f64_16x16x4_f64): rows are the output channels, columns the
// output positions of all images (g = n O + o), and the reduction runs over
// (kernel position p, input channel cs), p outer, so that a stage of
// kStartKB reduction indices mostly shares one p.  A workgroup of 4 waves
// owns 64 channels x 64 columns, wave w the channels 16 w .. 16 w + 15 as
// four 16 x 16 tiles.  Each thread loads its share of a stage (the decoded
// weights D^(m)[k(c, p)][a], cs = m C's + a: code, then sub-codeword entry;
// the input values, 0 outside the map) one stage ahead into registers,
// stores them into one of two LDS buffers, and every wave runs the stage's
// MFMAs from LDS.  Register i of lane l of a 16 x 16 f64 result holds row
// 4 i + l / 16, column l % 16.  Block sums of E^2 into
// opart[blockIdx.y gridDim.x + blockIdx.x].
constexpr int kStartTile = 64;          // channels and columns per workgroup
constexpr int kStartKB = 32;            // reduction indices per stage
constexpr int kStartLd = kStartKB + 1;  // LDS row stride in doubles (odd: spreads the rows over the banks)

template <int CSP>
__global__ __launch_bounds__(kCThreads) void ecc_start_kernel(const float* __restrict__ S,
                                                            const float* __restrict__ T, EccParams q,
                                                            const double* __restrict__ D64,
                                                            const uint8_t* __restrict__ ct, double* __restrict__ E,
                                                            double* __restrict__ opart) {
  static_assert(kCThreads == 256, "four waves, 8 values per thread and operand");
  __shared__ double As[2][kStartTile * kStartLd];  // [channel][index]
  __shared__ double Bs[2][kStartTile * kStartLd];  // [column][index]
  __shared__ double red[kCThreads / kWave];
  constexpr int PER = kStartTile * kStartKB / kCThreads;  // 8
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int c0 = blockIdx.x * kStartTile, g0 = blockIdx.y * kStartTile;
  const int ncol = q.N * q.O, KD = q.Cs * q.P;
  // this thread's share of a stage: row r (channel c0 + r of the weights,
  // column g0 + r of the inputs), reduction indices q0 .. q0 + PER - 1
  const int r = tid / (kStartKB / PER), q0 = (tid % (kStartKB / PER)) * PER;
  const int cw = c0 + r, gb = g0 + r;
  const bool rowa = cw < q.Ct, rowb = gb < ncol;
  const int nb = rowb ? gb / q.O : 0, ob = rowb ? gb - (gb / q.O) * q.O : 0;
  const int yb = (ob / q.Wo) * q.stride - q.pad, xb = (ob - (ob / q.Wo) * q.Wo) * q.stride - q.pad;
  const size_t HW = (size_t)q.H * q.W;
  const float* sb = S + (size_t)nb * q.Cs * HW;
  const int nst = (KD + kStartKB - 1) / kStartKB;
  float sv[PER];
  double wv[PER];
  auto load_stage = [&](int st) {
    const int k0 = st * kStartKB + q0;
    int p = k0 / q.Cs, cs = k0 - p * q.Cs;
    int code[PER], ma[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const bool okk = p < q.P;
      const int pp = okk ? p : 0, cc = okk ? cs : 0;
      const int ky = pp / q.dk, kx = pp - ky * q.dk;
      const int y = yb + ky, x = xb + kx;
      const bool oks = rowb && okk && (unsigned)y < (unsigned)q.H && (unsigned)x < (unsigned)q.W;
      const float v = sb[oks ? cc * HW + (size_t)y * q.W + x : 0];
      sv[i] = oks ? v : 0.f;
      const int m = cc / CSP;
      const bool okw = rowa && okk;
      const int cd = ct[okw ? ((size_t)m * q.Ct + cw) * q.P + pp : 0];
      code[i] = cd;
      ma[i] = okw ? (m * q.K) * CSP + (cc - m * CSP) : -1;
      if (++cs == q.Cs) {
        cs = 0;
        ++p;
      }
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const double w = D64[ma[i] >= 0 ? ma[i] + (size_t)code[i] * CSP : 0];
      wv[i] = ma[i] >= 0 ? w : 0.0;
    }
  };
  auto store_stage = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      As[buf][r * kStartLd + q0 + i] = wv[i];
      Bs[buf][r * kStartLd + q0 + i] = (double)sv[i];
    }
  };
  d4v acc[4];
#pragma unroll
  for (int t = 0; t < 4; ++t) acc[t] = d4v{0.0, 0.0, 0.0, 0.0};
  const int arow = 16 * wave + (lane & 15), kq = lane >> 4;
  load_stage(0);
  for (int st = 0; st < nst; ++st) {
    const int buf = st & 1;
    store_stage(buf);
    __syncthreads();  // the stage is in LDS; the other buffer's readers (stage st - 1) are done
    if (st + 1 < nst) load_stage(st + 1);
#pragma unroll
    for (int kk = 0; kk < kStartKB / 4; ++kk) {
      const double av = As[buf][arow * kStartLd + 4 * kk + kq];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const double bv = Bs[buf][(16 * t + (lane & 15)) * kStartLd + 4 * kk + kq];
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av, bv, acc[t], 0, 0, 0);
      }
    }
  }
  // acc[t][i]: channel c0 + 16 wave + 4 i + lane / 16, column g0 + 16 t + lane % 16
  double sq = 0.0;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const int g = g0 + 16 * t + (lane & 15);
    const int n = g / q.O, o = g - (g / q.O) * q.O;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = c0 + 16 * wave + 4 * i + kq;
      if (g < ncol && c < q.Ct) {
        const size_t at = ((size_t)n * q.Ct + c) * q.O + o;
        const double e = (double)T[at] - acc[t][i];
        E[at] = e;
        sq += e * e;
      }
    }
  }
  for (int off = kWave / 2; off > 0; off >>= 1) sq += __shfl_down(sq, off, kWave);
  if (lane == 0) red[wave] = sq;
  __syncthreads();
  if (tid == 0) {
    double s2 = 0.0;
    for (int w = 0; w < kCThreads / kWave; ++w) s2 += red[w];
    opart[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s2;
  }
}

// E -= sum_p delta[c][p]^T s_p for subspace ma; block sums of E^2.
template <int CSP>
__global__ __launch_bounds__(kCThreads) void ecc_apply_kernel(const float* __restrict__ S, EccParams q, int ma,
                                                            const double* __restrict__ delta,
                                                            double* __restrict__ E, double* __restrict__ opart) {
  __shared__ double red[kCThreads / kWave];
  const size_t i = (size_t)blockIdx.x * kCThreads + threadIdx.x;
  const size_t total = (size_t)q.N * q.Ct * q.O;
  double e = 0.0;
  if (i < total) {
    const int o = (int)(i % q.O);
    const int c = (int)((i / q.O) % q.Ct);
    const int n = (int)(i / ((size_t)q.O * q.Ct));
    e = E[i];
    const int yo = o / q.Wo, xo = o - yo * q.Wo;
    const size_t HW = (size_t)q.H * q.W;
    const float* sn = S + ((size_t)n * q.Cs + (size_t)ma * CSP) * HW;
    const double* dl = delta + (size_t)c * q.P * CSP;
    double d = 0.0;  // positions outside the input add exact zeros: skipped
    for (int ky = 0; ky < q.dk; ++ky) {
      const int y = yo * q.stride - q.pad + ky;
      if ((unsigned)y >= (unsigned)q.H) continue;
      for (int kx = 0; kx < q.dk; ++kx) {
        const int x = xo * q.stride - q.pad + kx;
        if ((unsigned)x >= (unsigned)q.W) continue;
        const double* dp = dl + (ky * q.dk + kx) * CSP;
#pragma unroll
        for (int j = 0; j < CSP; ++j) d += (double)sn[j * HW + (size_t)y * q.W + x] * dp[j];
      }
    }
    e -= d;
    E[i] = e;
  }
  ecc_block_sum(e * e, red, opart);
}

// part[chunk][c][p][j] = sum over the chunk's images and all o (in order) of
// s_p[j] E(c), for subspace m; one (c, p) per thread.
template <int CSP>
__global__ __launch_bounds__(kCThreads) void ecc_corr_kernel(const float* __restrict__ S, EccParams q, int m,
                                                           const double* __restrict__ E,
                                                           double* __restrict__ part) {
  const int i = blockIdx.x * kCThreads + threadIdx.x;
  if (i >= q.Ct * q.P) return;
  const int c = i / q.P, p = i - c * q.P;
  const int n0 = blockIdx.y * q.chunk, n1 = min(q.N, n0 + q.chunk);
  double acc[CSP];
#pragma unroll
  for (int j = 0; j < CSP; ++j) acc[j] = 0.0;
  const int ky = p / q.dk, kx = p - ky * q.dk;
  const size_t HW = (size_t)q.H * q.W;
  for (int n = n0; n < n1; ++n) {
    const double* er = E + ((size_t)n * q.Ct + c) * q.O;
    const float* sn = S + ((size_t)n * q.Cs + (size_t)m * CSP) * HW;
    for (int yo = 0; yo < q.Ho; ++yo) {
      const int y = yo * q.stride - q.pad + ky;
      if ((unsigned)y >= (unsigned)q.H) continue;  // exact zeros: skipped
      const double* erow = er + (size_t)yo * q.Wo;
      const float* srow = sn + (size_t)y * q.W;
#pragma unroll 4
      for (int xo = 0; xo < q.Wo; ++xo) {
        const int x = xo * q.stride - q.pad + kx;
        if ((unsigned)x >= (unsigned)q.W) continue;
        const double e = erow[xo];
#pragma unroll
        for (int j = 0; j < CSP; ++j) acc[j] += (double)srow[j * HW + x] * e;
      }
    }
  }
  double* dst = part + (((size_t)blockIdx.y * q.Ct + c) * q.P + p) * CSP;
#pragma unroll
  for (int j = 0; j < CSP; ++j) dst[j] = acc[j];
}

// Both of the above in one pass over E, on v_mfma_f64_16x16x4_f64, with E in
// registers between them: for 16 output positions x 16 channels,
//   E^T -= S_ma delta^T   (positions x (p, j), times (p, j) x channels)
//   H^T += S_m^T E^T      ((p, j) x positions, times positions x channels);
// register i of lane l of a result holds row 4 i + l / 16, column l % 16, and
// that is the second product's B operand of its reduction step i as it stands.
// A workgroup is 4 waves of 16 channels each over `tiles` 16-position tiles of
// `images` images, one after the other with H^T kept in registers (blockIdx.y =
// image group x parts + part); the two subspaces' input
// maps sit in LDS with their zero halos, and tables give an output's and a
// (p, j)'s offset in them.  Grid order of the sums: part[blockIdx.y][c][p][j],
// opart[blockIdx.y gridDim.x + blockIdx.x].
// Bound by the matrix cores' float64 rate (the residual's bytes, read and
// written once, take a third of that); apply and correlation as kernels of
// their own took 35 + 60 us at 384 channels, 32 x 13 x 13 outputs, 3x3, C's = 4.
struct PassShape {
  int images, groups;  // images per workgroup, groups of them
  int parts, tiles;    // workgroups per image and channel block, 16-position tiles of each
  int pw, plane;     // staged map: columns, positions per channel
};

constexpr int kMaxPassTiles = 8;  // (p, j) in tiles of 16: up to 128

template <int NT>
__global__ __launch_bounds__(kCThreads) void ecc_pass_kernel(const float* __restrict__ S, EccParams q, PassShape ps,
                                                           int ma, int m, const double* __restrict__ delta,
                                                           double* __restrict__ E, double* __restrict__ opart,
                                                           double* __restrict__ part) {
  extern __shared__ double smd[];
  const int QN = q.P * q.Csp, size = q.Csp * ps.plane;
  double* red = smd;                              // a sum per wave (no static LDS beside the largest dynamic)
  float* sa = reinterpret_cast<float*>(smd + kCThreads / kWave);  // subspace ma's maps
  float* sm = sa + size;                          // subspace m's
  int* qoff = reinterpret_cast<int*>(sm + size);  // [16 NT] offset of (p, j)
  int* ooff = qoff + 16 * NT;                     // [16 tiles] offset of an output
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const int group = blockIdx.y / ps.parts, t0 = (blockIdx.y - group * ps.parts) * ps.tiles;
  const int n0 = group * ps.images, n1 = min(q.N, n0 + ps.images);
  const int ntiles = min(ps.tiles, (q.O + 15) / 16 - t0);
  const size_t HW = (size_t)q.H * q.W;
  for (int i = tid; i < 16 * NT; i += kCThreads) {
    const int p = i / q.Csp, j = i - p * q.Csp;
    qoff[i] = i < QN ? j * ps.plane + (p / q.dk) * ps.pw + p % q.dk : 0;
  }
  for (int i = tid; i < 16 * ps.tiles; i += kCThreads) {
    const int o = t0 * 16 + i;
    ooff[i] = o < q.O ? (o / q.Wo) * q.stride * ps.pw + (o % q.Wo) * q.stride : 0;
  }
  const int col = lane & 15, quad = lane >> 4;
  const int c = (blockIdx.x * (kCThreads / kWave) + wave) * 16 + col;
  const bool live = c < q.Ct;
  // the change of ma as the first product's B operand (0 past the (p, j))
  double db[4 * NT];
#pragma unroll
  for (int kk = 0; kk < 4 * NT; ++kk) {
    const int i = 4 * kk + quad;
    db[kk] = ma >= 0 && live && i < QN ? delta[(size_t)c * QN + i] : 0.0;
  }
  d4v h[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) h[t] = d4v{0.0, 0.0, 0.0, 0.0};
  double sq = 0.0;
  for (int n = n0; n < n1; ++n) {
    if (n > n0) __syncthreads();  // the last image's maps are read
    for (int i = tid; i < size; i += kCThreads) {
      const int j = i / ps.plane, r = i - j * ps.plane;
      const int y = r / ps.pw - q.pad, x = r % ps.pw - q.pad;
      const bool in = (unsigned)y < (unsigned)q.H && (unsigned)x < (unsigned)q.W;
      const float* src = S + ((size_t)n * q.Cs + j) * HW + (in ? (size_t)y * q.W + x : 0);
      sa[i] = in && ma >= 0 ? src[(size_t)ma * q.Csp * HW] : 0.f;
      sm[i] = in && m >= 0 ? src[(size_t)m * q.Csp * HW] : 0.f;
    }
    __syncthreads();  // the maps, and the tables before the first image
    double* er = E + ((size_t)n * q.Ct + (live ? c : 0)) * q.O;
    double e[4];
    auto load_e = [&](int t, double (&v)[4]) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int o = (t0 + t) * 16 + 4 * i + quad;
        v[i] = live && o < q.O ? er[o] : 0.0;
      }
    };
    if (ntiles > 0) load_e(0, e);
    for (int t = 0; t < ntiles; ++t) {
      double en[4] = {0.0, 0.0, 0.0, 0.0};
      if (t + 1 < ntiles) load_e(t + 1, en);  // one tile ahead
      if (ma >= 0) {
        const float* base = sa + ooff[16 * t + col];
        d4v d = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int kk = 0; kk < 4 * NT; ++kk)
          if (4 * kk < QN) d = __builtin_amdgcn_mfma_f64_16x16x4f64((double)base[qoff[4 * kk + quad]], db[kk], d, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int o = (t0 + t) * 16 + 4 * i + quad;
          if (live && o < q.O) {
            e[i] -= d[i];
            er[o] = e[i];
            sq += e[i] * e[i];
          }
        }
      }
      if (m >= 0) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
          const float* base = sm + ooff[16 * t + 4 * kk + quad];
#pragma unroll
          for (int u = 0; u < NT; ++u)
            h[u] = __builtin_amdgcn_mfma_f64_16x16x4f64((double)base[qoff[16 * u + col]], e[kk], h[u], 0, 0, 0);
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) e[i] = en[i];
    }
  }
  if (m >= 0 && live) {
    double* dst = part + ((size_t)blockIdx.y * q.Ct + c) * QN;
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int r = 16 * u + 4 * i + quad;
        if (r < QN) dst[r] = h[u][i];
      }
  }
  if (ma >= 0) {
    for (int off = kWave / 2; off > 0; off >>= 1) sq += __shfl_down(sq, off, kWave);
    if (lane == 0) red[wave] = sq;
    __syncthreads();
    if (tid == 0) {
      double s = 0.0;
      for (int w = 0; w < kCThreads / kWave; ++w) s += red[w];
      opart[(size_t)blockIdx.y * gridDim.x + blockIdx.x] = s;
    }
  }
}

// The pass's split and LDS bytes for a layer, or 0 bytes when its (p, j) or
// its maps do not fit (ecc_apply_kernel and ecc_corr_kernel then run).
size_t pass_shape(const EccParams& q, PassShape* ps) {
  if (q.P * q.Csp > 16 * kMaxPassTiles) return 0;
  ps->pw = (q.Wo - 1) * q.stride + q.dk;
  const long long plane = (long long)((q.Ho - 1) * q.stride + q.dk) * ps->pw;
  if (2 * plane * q.Csp * 4 > 48 * 1024) return 0;
  ps->plane = (int)plane;
  // at least 1536 waves of 16 channels (1.5 per SIMD) as long as a piece keeps
  // 4 tiles: with fewer, SIMDs stay idle; with more, the sums over the pieces
  // grow
  const int tiles = (q.O + 15) / 16, cb = ceil_div(q.Ct, 16);
  // ... and past twice that a workgroup takes several images: the partial sums
  // stay at 3072 x 16 channels x (p, j) doubles whatever N (one per image was
  // d_k^2 C's / (H_o W_o) times the residual)
  ps->images = std::max(1, (int)((long long)q.N * cb / 3072));
  ps->groups = ceil_div(q.N, ps->images);
  const int waves = cb * ps->groups;
  int parts = std::max(1, std::min(ceil_div(1536, waves), tiles / 4));
  ps->tiles = ceil_div(tiles, parts);
  ps->parts = ceil_div(tiles, ps->tiles);
  return (size_t)kCThreads / kWave * 8 + (size_t)2 * q.Csp * plane * 4 + (size_t)16 * ((q.P * q.Csp + 15) / 16) * 4 + (size_t)16 * ps->tiles * 4;
}

hipError_t launch_pass(const float* S, const EccParams& q, const PassShape& ps, size_t lds, int ma, int m,
                       const double* delta, double* E, double* opart, double* part, hipStream_t stream) {
  const dim3 grid((unsigned)ceil_div(q.Ct, 64), (unsigned)(ps.groups * ps.parts));
  auto pass = ecc_pass_kernel<8>;
  switch ((q.P * q.Csp + 15) / 16) {
    case 1: pass = ecc_pass_kernel<1>; break;
    case 2: pass = ecc_pass_kernel<2>; break;
    case 3: pass = ecc_pass_kernel<3>; break;
    case 4: pass = ecc_pass_kernel<4>; break;
    case 5: pass = ecc_pass_kernel<5>; break;
    case 6: pass = ecc_pass_kernel<6>; break;
    case 7: pass = ecc_pass_kernel<7>; break;
  }
  const hipError_t e = allow_max_lds((const void*)pass);  // maps 48 KB, offsets of up to 6144 outputs 24 KB
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(pass, grid, dim3(kCThreads), lds, stream, S, q, ps, ma, m, delta, E, opart, part);
  return hipGetLastError();
}

// H[c][p][j] = sum over chunks (in order) of part + sum_p' sum_i G[p][p'][j][i] W(c, p')[i].
// One (c, p, j) per thread, sixteen chunks' loads in flight.
template <int CSP>
__global__ __launch_bounds__(kCThreads) void ecc_reduce_kernel(const double* __restrict__ part, EccParams q,
                                                             int nchunks, int m, const double* __restrict__ G,
                                                             const double* __restrict__ D64,
                                                             const uint8_t* __restrict__ ct,
                                                             double* __restrict__ H) {
  const int i = blockIdx.x * kCThreads + threadIdx.x, total = q.Ct * q.P * CSP;
  if (i >= total) return;
  const int cp = i / CSP, j = i - cp * CSP;
  const int c = cp / q.P, p = cp - c * q.P;
  double h = 0.0;
  for (int ch = 0; ch < nchunks; ch += 16) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = ch + u < nchunks ? part[(size_t)(ch + u) * total + i] : 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) h += v[u];
  }
  const double* Gp = G + (((size_t)m * q.P + p) * q.P * CSP + j) * CSP;
  const uint8_t* km = ct + ((size_t)m * q.Ct + c) * q.P;
  for (int p0 = 0; p0 < q.P; p0 += 3) {
    double w[3][CSP], g[3][CSP];
#pragma unroll
    for (int u = 0; u < 3; ++u) {
      const int p2 = min(p0 + u, q.P - 1);
      const double* ws = D64 + ((size_t)m * q.K + km[p2]) * CSP;
#pragma unroll
      for (int i2 = 0; i2 < CSP; ++i2) {
        w[u][i2] = ws[i2];
        g[u][i2] = Gp[(size_t)p2 * CSP * CSP + i2];
      }
    }
#pragma unroll
    for (int u = 0; u < 3; ++u)
      if (p0 + u < q.P)
#pragma unroll
        for (int i2 = 0; i2 < CSP; ++i2) h += g[u][i2] * w[u][i2];
  }
  H[i] = h;
}

__device__ __forceinline__ void wave_sync_lds() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
  __builtin_amdgcn_wave_barrier();
}

// x with A x = b for the normal matrix A of Eq. (19): elimination in channel
// order without row exchanges, one reciprocal per pivot; a pivot <= 1e-12 x
// the largest diagonal entry (or <= 0) drops that coordinate (x = 0).  A is
// read only; W is N x N working storage of the calling lane.
template <int N>
__device__ __forceinline__ void solve_rcp(const double* __restrict__ A, const double (&bin)[N], double* W,
                                          double (&x)[N]) {
  double y[N], inv[N];
  bool live[N];
  double scale = 0.0;
#pragma unroll
  for (int i = 0; i < N; ++i) {
#pragma unroll
    for (int j = 0; j < N; ++j) W[i * N + j] = A[i * N + j];
    y[i] = bin[i];
    scale = fmax(scale, A[i * N + i]);
  }
#pragma unroll
  for (int j = 0; j < N; ++j) {
    live[j] = W[j * N + j] > 1e-12 * scale && W[j * N + j] > 0.0;
    inv[j] = live[j] ? 1.0 / W[j * N + j] : 0.0;
    if (live[j]) {
#pragma unroll
      for (int i = j + 1; i < N; ++i) {
        const double f = W[i * N + j] * inv[j];
#pragma unroll
        for (int c = j; c < N; ++c) W[i * N + c] -= f * W[j * N + c];
        y[i] -= f * y[j];
      }
    }
  }
#pragma unroll
  for (int j = N - 1; j >= 0; --j) {
    double s = y[j];
#pragma unroll
    for (int i = j + 1; i < N; ++i)
      if (live[i]) s -= W[j * N + i] * x[i];
    x[j] = live[j] ? s * inv[j] : 0.0;
  }
}

// ---- Eq. (17)-(19) as a linear system.  With the pairs (c, p) on k,
//   A_k = B[k][k],  B[k][k'] = sum_{(c,p) on k} sum_{p': k(c,p') = k'} G[p][p'],
//   b_k = sum_{(c,p) on k} H[c][p],
// the update of sub-codeword k is A_k D_k = b_k - sum_{k' != k} B[k][k'] D_k'
// with D_k' new for k' < k and old for k' > k: one Gauss-Seidel sweep over
// the rows.  Everything but the D_k' new terms is independent of the order:
// ecc_rows_kernel makes row k in a workgroup of its own, r0_k = b_k -
// sum_{k'>k} B[k][k'] D_k' old included, and ecc_solve_kernel is left with
// r_k -= B[k][k'] D_k' for k' < k and D_k = A_k^-1 r_k.  (One workgroup that
// formed each sub-codeword's sums from its pairs in turn took 2.8 us per
// sub-codeword, 353 us a step at 384 channels, 3x3, K = 128, C's = 4.)
//
// The solve goes in blocks of kColBlock / C's sub-codewords: wave 0 solves a
// block, then every thread takes the block's new values out of its later row.  B is stored for that:
// [column block][column pair][row][2], so that a wave's loads are whole lines.
constexpr int kColBlock = 64;  // columns (sub-codeword entries) per block, one row of the block per lane
constexpr int kSolveThreads = 512;

template <int CSP> __host__ __device__ constexpr int block_codewords() { return kColBlock / CSP; }

template <int CSP> size_t system_doubles(int K) {
  const size_t blocks = ((size_t)K + block_codewords<CSP>() - 1) / block_codewords<CSP>();
  return blocks * kColBlock * (size_t)K * CSP;
}

template <int CSP> constexpr int rows_threads() { return CSP <= 4 ? 1024 : 512; }

// Entries of a column block whose shares are added at a time: 16 KB of LDS,
// whatever K (all C's^2 of them at once took 128 KB at K = 256, C's = 8, and
// with the codes and the list of 9375 pairs or more did not fit).
template <int CSP> constexpr int rows_slice() { return std::min(CSP * CSP, 2048 / rows_threads<CSP>()); }

// Counts of (k', p') for one p: kCountP positions p' at a time, rows of an odd
// number of words.
constexpr int kCountP = 16, kCountLd = kCountP + 1;

// Pairs of a sub-codeword up to which its row is made from the list: a count
// takes P ceil(P / kCountP) steps whatever the pairs.  us a sweep, list ->
// counts: 3x3, 24 channels, all 216 pairs on one of 16 codes 469 -> 280; 256
// channels, 288 a code 1220 -> 640; all 4608 on one of 256, C's = 8, 139000 ->
// 4030; 11x11, 40 channels, 151 pairs a code 19000 -> 27700.
__device__ __forceinline__ int list_pairs(int P) { return 128 * ((P + kCountP - 1) / kCountP); }

// LDS of the shares, and of the counts before them.
template <int CSP> __host__ __device__ constexpr size_t rows_area(int K) {
  return std::max((size_t)rows_slice<CSP>() * rows_threads<CSP>() * 8, ((size_t)K * kCountLd * 4 + 7) / 8 * 8);
}

// Row k = blockIdx.x.  LDS: the codes, the list of k's pairs in (c, p) order
// (one run of it per wave, compacted by that wave), the Gram blocks (GL).  A
// thread owns one column block k' and, of the `parts` threads that share it,
// every parts-th pair: it adds the G[p][p'] of the pair's positions on k'.
// The shares are added in order.  The kernel's time is that of the largest
// sub-codeword (some take ten times the mean number of pairs), hence as many
// threads per row as the sums' registers allow.  A sub-codeword of more than
// list_pairs is counted instead: per p, how many of its channels have k'
// at p' (integer counts, whatever their order), times G[p][p'], so that neither
// the number of its pairs nor how many share one k' makes a thread's chain
// longer.
template <int CSP, bool GL>
__global__ __launch_bounds__(rows_threads<CSP>()) void ecc_rows_kernel(const double* __restrict__ H, EccParams q,
                                                                     int m, const double* __restrict__ G,
                                                                     const double* __restrict__ D64,
                                                                     const uint8_t* __restrict__ ct,
                                                                     double* __restrict__ B, double* __restrict__ X,
                                                                     double* __restrict__ r0,
                                                                     int* __restrict__ used) {
  extern __shared__ double sh[];
  constexpr int NT = rows_threads<CSP>(), NW = NT / kWave, SQ = CSP * CSP, SE = rows_slice<CSP>();
  const int K = q.K, P = q.P, npairs = q.Ct * P;
  const int k = blockIdx.x;
  const int kp = (K + kWave - 1) / kWave * kWave;
  const int parts = NT / kp;
  double* red = sh;                      // [NT] partial sums
  double* Al = red + NT;                 // [C's][C's]
  double* share = Al + SQ;               // [SE][NT], before that the counts
  uint32_t* cnt = reinterpret_cast<uint32_t*>(share);
  double* Gl = share + rows_area<CSP>(K) / 8;
  int* wn = reinterpret_cast<int*>(Gl + (GL ? (size_t)P * P * SQ : 0));  // [NW] first entry of each wave's run
  uint16_t* list = reinterpret_cast<uint16_t*>(wn + NW + 1);
  uint8_t* cs = reinterpret_cast<uint8_t*>(list + npairs);
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  const double* Gg = G + (size_t)m * P * P * SQ;
  const double* Gm = GL ? Gl : Gg;
  for (int i = tid; i < npairs; i += NT) cs[i] = ct[(size_t)m * npairs + i];
  if (GL)
    for (int i = tid; i < P * P * SQ; i += NT) Gl[i] = Gg[i];
  const int kc = tid % kp, part = tid / kp;  // column block and share of this thread
  double dold[CSP];
#pragma unroll
  for (int j = 0; j < CSP; ++j)
    dold[j] = part == 0 && kc > k && kc < K ? D64[((size_t)m * K + kc) * CSP + j] : 0.0;
  __syncthreads();
  // each wave counts, then places, the pairs on k of its share of the codes
  const int share_n = (npairs + NW - 1) / NW;
  const int b0 = min(npairs, wave * share_n), b1 = min(npairs, b0 + share_n);
  int n = 0;
  for (int i0 = b0; i0 < b1; i0 += kWave) n += __popcll(__ballot(i0 + lane < b1 && cs[i0 + lane] == k));
  if (lane == 0) wn[wave] = n;
  __syncthreads();
  int at = 0, n_k = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    at += w < wave ? wn[w] : 0;
    n_k += wn[w];
  }
  if (tid == 0) used[k] = n_k;
  if (n_k == 0) return;  // unused: keeps its value, and its row is not read
  for (int i0 = b0; i0 < b1; i0 += kWave) {
    const bool on = i0 + lane < b1 && cs[i0 + lane] == k;
    const uint64_t ones = __ballot(on);
    if (on) list[at + __popcll(ones & ((1ull << lane) - 1ull))] = (uint16_t)(i0 + lane);
    at += __popcll(ones);
  }
  __syncthreads();

  // b_k: slot s = tid / C's takes pairs s, s + slots, ...; then the slots in order
  constexpr int slots = NT / CSP;
  {
    const int s = tid / CSP, j = tid - s * CSP;
    double v = 0.0;
    if (s < slots)
      for (int r = s; r < n_k; r += slots) v += H[(size_t)list[r] * CSP + j];
    red[tid] = v;
  }
  // this thread's share of column block k'
  const float rcp_p = 1.0f / (float)P;
  double acc[SQ];
#pragma unroll
  for (int i = 0; i < SQ; ++i) acc[i] = 0.0;
  const bool counted = n_k > list_pairs(P);
  if (counted) {
    for (int p = 0; p < P; ++p)
      for (int p0 = 0; p0 < P; p0 += kCountP) {
        __syncthreads();  // the counts before these are used
        for (int i = tid; i < K * kCountLd; i += NT) cnt[i] = 0;
        __syncthreads();
        for (int i = tid; i < q.Ct * kCountP; i += NT) {
          const int u = i % kCountP;
          const uint8_t* kk = cs + i / kCountP * P;
          if (p0 + u < P && kk[p] == k) atomicAdd(&cnt[kk[p0 + u] * kCountLd + u], 1u);
        }
        __syncthreads();
        if (part < parts && kc < K)
          for (int u = part; u < min(kCountP, P - p0); u += parts) {
            const uint32_t times = cnt[kc * kCountLd + u];
            if (times == 0) continue;
            const double* g = Gm + ((size_t)p * P + p0 + u) * SQ;
#pragma unroll
            for (int i = 0; i < SQ; ++i) acc[i] += (double)times * g[i];
          }
      }
  }
  for (int r = part < parts && !counted ? part : n_k; r < n_k; r += parts) {
    const int pr = list[r];
    const int c = (int)(((float)pr + 0.5f) * rcp_p), p = pr - c * P;  // exact: pr < 2^14
    const uint8_t* kk = cs + c * P;
    const double* grow = Gm + (size_t)p * P * SQ;
    for (int p0 = 0; p0 < P; p0 += 9) {
      int k2[9];
#pragma unroll
      for (int u = 0; u < 9; ++u) k2[u] = p0 + u < P ? kk[p0 + u] : -1;
#pragma unroll
      for (int u = 0; u < 9; ++u)
        if (k2[u] == kc) {
          const double* g = grow + (size_t)(p0 + u) * SQ;
#pragma unroll
          for (int i = 0; i < SQ; ++i) acc[i] += g[i];
        }
    }
  }
  __syncthreads();
  if (min(parts, n_k) > 1) {
#pragma unroll
    for (int i0 = 0; i0 < SQ; i0 += SE) {
      if (i0 > 0) __syncthreads();
      if (part > 0)
#pragma unroll
        for (int i = i0; i < i0 + SE && i < SQ; ++i) share[(i - i0) * NT + tid] = acc[i];
      __syncthreads();
      if (part == 0)
        for (int w = 1; w < min(parts, n_k); ++w)
#pragma unroll
          for (int i = i0; i < i0 + SE && i < SQ; ++i) acc[i] += share[(i - i0) * NT + w * kp + kc];
    }
  }
  double bk = 0.0;  // of thread j < C's
  if (tid < CSP) {
    const int ns = min(slots, n_k);
    for (int s0 = 0; s0 < ns; s0 += 8) {
      double v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = s0 + u < ns ? red[(s0 + u) * CSP + tid] : 0.0;
#pragma unroll
      for (int u = 0; u < 8; ++u) bk += v[u];
    }
  }
  // the row's columns k' < k; the old values of k' > k; A_k
  const bool mine = part == 0 && kc < K;
  double t[CSP];
#pragma unroll
  for (int i = 0; i < CSP; ++i) t[i] = 0.0;
  if (mine && kc < k) {
    constexpr int NB = block_codewords<CSP>();
    const size_t R = (size_t)K * CSP;
    const int kb = kc / NB, col0 = (kc - kb * NB) * CSP;
    double* dst = B + (size_t)kb * kColBlock * R;
#pragma unroll
    for (int i = 0; i < CSP; ++i) {
      if constexpr (CSP % 2 == 0) {
#pragma unroll
        for (int j = 0; j < CSP; j += 2)
          *reinterpret_cast<double2*>(dst + ((size_t)((col0 + j) >> 1) * R + (size_t)k * CSP + i) * 2) =
              double2{acc[i * CSP + j], acc[i * CSP + j + 1]};
      } else {
#pragma unroll
        for (int j = 0; j < CSP; ++j) {
          const int col = col0 + j;
          dst[((size_t)(col >> 1) * R + (size_t)k * CSP + i) * 2 + (col & 1)] = acc[i * CSP + j];
        }
      }
    }
  } else if (mine && kc > k) {
#pragma unroll
    for (int i = 0; i < CSP; ++i)
#pragma unroll
      for (int j = 0; j < CSP; ++j) t[i] += acc[i * CSP + j] * dold[j];
  } else if (mine) {
#pragma unroll
    for (int i = 0; i < SQ; ++i) Al[i] = acc[i];
  }
#pragma unroll
  for (int i = 0; i < CSP; ++i)
    for (int off = kWave / 2; off > 0; off >>= 1) t[i] += __shfl_down(t[i], off, kWave);
  __syncthreads();  // the slots' sums are read; A_k
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < CSP; ++i) red[wave * CSP + i] = t[i];
  __syncthreads();
  if (tid < CSP) {
    double v = bk;
    for (int w = 0; w < kp / kWave; ++w) v -= red[w * CSP + tid];
    r0[(size_t)k * CSP + tid] = v;
    // column tid of A_k^-1 (with the dropped coordinates' rows and columns 0)
    double unit[CSP], Aw[SQ], x[CSP];
#pragma unroll
    for (int i = 0; i < CSP; ++i) unit[i] = i == tid ? 1.0 : 0.0;
    solve_rcp<CSP>(Al, unit, Aw, x);
#pragma unroll
    for (int i = 0; i < CSP; ++i) X[((size_t)k * CSP + i) * CSP + tid] = x[i];
  }
}

template <int CSP, bool GL> size_t rows_lds_bytes(int K, int npairs, int P) {
  constexpr int NT = rows_threads<CSP>();
  const size_t dbl = NT + CSP * CSP + rows_area<CSP>(K) / 8 + (GL ? (size_t)P * P * CSP * CSP : 0);
  return dbl * 8 + (NT / kWave + 1) * 4 + (size_t)npairs * 3;
}

// The substitution, in one workgroup.  On the first round of a step (`first`)
// it also records the objective before the step (from the pass's block sums)
// and keeps the subspace's sub-codebook and codes as they were (Dold, cold)
// for delta.  At the end it stores qkg[p][k] = D_k^T G[p][p] D_k for the
// assignment kernel.  (Having the other workgroups of its XCD read B ahead
// into their L2 made no difference: it is not bound by B's latency.)
template <int CSP>
__global__ __launch_bounds__(kSolveThreads) void ecc_solve_kernel(EccParams q, int m, const double* __restrict__ G,
                                                                double* __restrict__ D64,
                                                                const uint8_t* __restrict__ ct, int first,
                                                                const double* __restrict__ B,
                                                                const double* __restrict__ X,
                                                                const double* __restrict__ r0,
                                                                const int* __restrict__ used,
                                                                double* __restrict__ Dold, uint8_t* __restrict__ cold,
                                                                double* __restrict__ qkg,
                                                                const double* __restrict__ opart, int nopart,
                                                                double* __restrict__ objective) {
  extern __shared__ double sh[];
  constexpr int NB = block_codewords<CSP>(), NC = NB * CSP;  // sub-codewords and columns of a block
  const int K = q.K, P = q.P, npairs = q.Ct * P, R = K * CSP;
  double* Ds = sh;              // [K][C's]
  double* rs = Ds + R;          // [K][C's] right-hand sides
  double* Xl2 = rs + R;         // [2][NB][C's][C's] A^-1 of a block
  double* diag2 = Xl2 + 2 * NB * CSP * CSP;               // [2][64][66] a block's own rows
  double* red = diag2 + 2 * kColBlock * (kColBlock + 2);  // [512]
  int* us = reinterpret_cast<int*>(red + kSolveThreads);  // [K]
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  for (int i = tid; i < R; i += kSolveThreads) {
    Ds[i] = D64[(size_t)m * R + i];
    rs[i] = r0[i];
    if (first) Dold[i] = Ds[i];
  }
  for (int i = tid; i < K; i += kSolveThreads) us[i] = used[i];
  if (first)
    for (int i = tid; i < npairs; i += kSolveThreads) cold[i] = ct[(size_t)m * npairs + i];
  if (first && objective) {
    double os = 0.0;
    for (int i = tid; i < nopart; i += kSolveThreads) os += opart[i];
    red[tid] = os;
    __syncthreads();
    for (int h = kSolveThreads / 2; h > 0; h >>= 1) {
      if (tid < h) red[tid] += red[tid + h];
      __syncthreads();
    }
    if (tid == 0) *objective = red[0];
  }

  // Wave 0 solves block kb (its columns' own rows and A^-1 in LDS) while the
  // others load those columns of the later rows, a row per thread, and the
  // next block's LDS.
  constexpr int LD = kColBlock + 2;  // doubles per row of a block's own rows
  const int blocks = (K + NB - 1) / NB;
  auto stage = [&](int kb, int first_thread) {  // block kb's own rows and A^-1 into buffer kb & 1
    double* diag = diag2 + (size_t)(kb & 1) * kColBlock * LD;
    double* Xl = Xl2 + (size_t)(kb & 1) * NB * CSP * CSP;
    const double* src = B + (size_t)kb * kColBlock * R;
    const int step = kSolveThreads - first_thread;
    for (int i = tid - first_thread; i < NC * (kColBlock / 2); i += step) {
      const int c2 = i / NC, rr = i - c2 * NC, row = kb * NC + rr;
      if (2 * c2 < NC && row < R) {
        const double2 v = *reinterpret_cast<const double2*>(src + ((size_t)c2 * R + row) * 2);
        diag[rr * LD + 2 * c2] = v.x;
        diag[rr * LD + 2 * c2 + 1] = v.y;
      }
    }
    for (int i = tid - first_thread; i < NB * CSP * CSP; i += step) {
      const size_t at = (size_t)kb * NB * CSP * CSP + i;
      if (at < (size_t)R * CSP) Xl[i] = X[at];
    }
  };
  stage(0, 0);
  for (int kb = 0; kb < blocks; ++kb) {
    __syncthreads();  // right-hand sides; the block's LDS
    const double* src = B + (size_t)kb * kColBlock * R;
    const int row0 = (kb + 1) * NC + tid - kWave;  // first later row of a thread past wave 0
    double bv[kColBlock];
    auto load_cols = [&](int row) {
#pragma unroll
      for (int c = 0; c < NC; c += 2) {
        const double2 v = *reinterpret_cast<const double2*>(src + ((size_t)(c >> 1) * R + row) * 2);
        bv[c] = v.x;
        bv[c + 1] = v.y;
      }
    };
    if (tid < kWave) {
      const double* diag = diag2 + (size_t)(kb & 1) * kColBlock * LD + lane * LD;
      const double* Xl = Xl2 + (size_t)(kb & 1) * NB * CSP * CSP;
      const int row = kb * NC + lane;
      double r = lane < NC && row < R ? rs[row] : 0.0;
      // Unrolled, with the operands of the next sub-codeword (which do not
      // wait for r) in registers of their own; lane l forms entry l % C's of
      // A_k^-1 r, broadcast through scalar registers.
      const int li = lane % CSP;
      double bq[2][CSP], aq[2][CSP];
      const uint64_t live = __ballot(lane < NB && kb * NB + lane < K && us[min(kb * NB + lane, K - 1)] > 0);
      auto fetch = [&](int kk, int slot) {
#pragma unroll
        for (int j = 0; j < CSP; ++j) {
          bq[slot][j] = diag[kk * CSP + j];
          aq[slot][j] = Xl[(kk * CSP + li) * CSP + j];
        }
      };
      auto spread = [&](double v, int first, double (&out)[CSP]) {
#pragma unroll
        for (int j = 0; j < CSP; ++j) {
          const long long bits = __double_as_longlong(v);
          const int lo = __builtin_amdgcn_readlane((int)bits, first + j);
          const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), first + j);
          out[j] = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
        }
      };
      auto dot = [&](const double (&u)[CSP], const double (&v)[CSP]) {
        double even = u[0] * v[0], odd = CSP > 1 ? u[CSP > 1] * v[CSP > 1] : 0.0;
#pragma unroll
        for (int j = 2; j < CSP; j += 2) even += u[j] * v[j];
#pragma unroll
        for (int j = 3; j < CSP; j += 2) odd += u[j] * v[j];
        return even + odd;
      };
      fetch(0, 0);
#pragma unroll
      for (int kk = 0; kk < NB; ++kk) {
        if (kk + 1 < NB) fetch(kk + 1, (kk + 1) & 1);
        __builtin_amdgcn_sched_barrier(0);
        if ((live >> kk) & 1) {  // uniform
          double g[CSP], x[CSP];
          spread(r, kk * CSP, g);
          const double own = dot(aq[kk & 1], g);
          spread(own, 0, x);
          const double d = dot(bq[kk & 1], x);
          if (lane >= (kk + 1) * CSP) r -= d;
          if (lane < CSP) Ds[(kb * NB + kk) * CSP + lane] = own;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    } else {
      if (row0 < R) load_cols(row0);
      if (kb + 1 < blocks) stage(kb + 1, kWave);
    }
    __syncthreads();  // the block's new values
    // ... taken out of the later rows (unused sub-codewords' columns are 0)
    if (tid >= kWave) {
      for (int row = row0; row < R; row += kSolveThreads - kWave) {
        if (row != row0) load_cols(row);
        double s4[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int c = 0; c < NC; ++c) s4[c & 3] += bv[c] * Ds[kb * NC + c];
        rs[row] -= (s4[0] + s4[1]) + (s4[2] + s4[3]);
      }
    }
  }
  __syncthreads();

  for (int i = tid; i < R; i += kSolveThreads) D64[(size_t)m * R + i] = Ds[i];
  const double* Gg = G + (size_t)m * P * P * CSP * CSP;
  for (int e = tid; e < P * K; e += kSolveThreads) {  // D_k^T G[p][p] D_k
    const int p = e / K, k = e - p * K;
    const double* Gpp = Gg + ((size_t)p * P + p) * CSP * CSP;
    double s2 = 0.0;
#pragma unroll
    for (int r = 0; r < CSP; ++r) {
      double g = 0.0;
#pragma unroll
      for (int i = 0; i < CSP; ++i) g += Gpp[r * CSP + i] * Ds[k * CSP + i];
      s2 += Ds[k * CSP + r] * g;
    }
    qkg[e] = s2;
  }
}

template <int CSP> size_t solve_lds_bytes(int K) {
  return ((size_t)2 * K * CSP + 2 * block_codewords<CSP>() * CSP * CSP + 2 * kColBlock * (kColBlock + 2) +
          kSolveThreads) * 8 + (size_t)K * 4;
}

// Eq. (20)-(21): one wave per output channel c, the kernel positions in
// order.  For position p, b = H[c][p] - sum_{p' != p} G[p][p'] D_{k(c,p')}
// (lanes take (p', row) terms; the rows are added over p' in a fixed order),
// then lane l tries candidates l, l + 64, ... and the wave keeps the first
// minimum of qkg[p][k] - 2 D_k^T b (ties to the lowest k).  On the last round
// it also writes delta[c][p] = D_{k_new} - Dold_{k_old}.
template <int CSP>
__global__ __launch_bounds__(kCThreads) void ecc_bupdate_kernel(const double* __restrict__ H, EccParams q, int m,
                                                              const double* __restrict__ G,
                                                              const double* __restrict__ D64,
                                                              const double* __restrict__ qkg,
                                                              uint8_t* __restrict__ ct,
                                                              const double* __restrict__ Dold,
                                                              const uint8_t* __restrict__ cold,
                                                              double* __restrict__ delta, int last) {
  extern __shared__ double sb[];
  constexpr int NW = kCThreads / kWave;
  constexpr int QS = kWave / CSP;
  const int K = q.K, P = q.P;
  double* Ds = sb;                                   // [K][C's]
  double* part = Ds + K * CSP;                       // [4][QS][C's] row partials per wave
  double* bb = part + NW * QS * CSP;                 // [4][C's]
  uint8_t* kc = reinterpret_cast<uint8_t*>(bb + NW * CSP);  // [4][P] this wave's codes
  const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
  for (int i = tid; i < K * CSP; i += kCThreads) Ds[i] = D64[(size_t)m * K * CSP + i];
  const int c = blockIdx.x * NW + wave;
  const bool col = c < q.Ct;
  uint8_t* kw = kc + wave * P;
  if (col)
    for (int p = lane; p < P; p += kWave) kw[p] = ct[((size_t)m * q.Ct + c) * P + p];
  __syncthreads();
  if (!col) return;  // no barriers below
  const double* Gg = G + (size_t)m * P * P * CSP * CSP;
  const int g = lane / CSP, j = lane - g * CSP;
  for (int p = 0; p < P; ++p) {
    // row j of sum_{p' != p} G[p][p'] D_{k(c,p')}: group g takes p' = g, g + QS, ...
    double t = 0.0;
    if (g < QS) {
      for (int p2 = g; p2 < P; p2 += QS) {
        if (p2 == p) continue;
        const double* gr = Gg + (((size_t)p * P + p2) * CSP + j) * CSP;
        const double* dk = Ds + kw[p2] * CSP;
#pragma unroll
        for (int i = 0; i < CSP; ++i) t += gr[i] * dk[i];
      }
      part[(wave * QS + g) * CSP + j] = t;
    }
    wave_sync_lds();
    if (lane < CSP) {
      double v = H[(((size_t)c * P + p) * CSP) + lane];
      double sub = 0.0;
      for (int g2 = 0; g2 < QS; ++g2) sub += part[(wave * QS + g2) * CSP + lane];
      bb[wave * CSP + lane] = v - sub;
    }
    wave_sync_lds();
    double b[CSP];
#pragma unroll
    for (int r = 0; r < CSP; ++r) b[r] = bb[wave * CSP + r];
    // this lane's candidates, then the wave's first minimum
    int best = -1;
    double bv = 0.0;
    const double* qp = qkg + (size_t)p * K;
    for (int k = lane; k < K; k += kWave) {
      double d = 0.0;
#pragma unroll
      for (int r = 0; r < CSP; ++r) d += Ds[k * CSP + r] * b[r];
      const double v = qp[k] - 2.0 * d;
      if (best < 0 || v < bv) {
        bv = v;
        best = k;
      }
    }
    for (int off = kWave / 2; off > 0; off >>= 1) {
      const double ov = __shfl_down(bv, off, kWave);
      const int ok = __shfl_down(best, off, kWave);
      if (ok >= 0 && (best < 0 || ov < bv || (ov == bv && ok < best))) {
        bv = ov;
        best = ok;
      }
    }
    best = __shfl(best, 0, kWave);
    if (lane == 0) kw[p] = (uint8_t)best;
    wave_sync_lds();
  }
  for (int p = lane; p < P; p += kWave) {
    const size_t i = (size_t)c * P + p;
    ct[(size_t)m * q.Ct * P + i] = kw[p];
    if (last)
#pragma unroll
      for (int r = 0; r < CSP; ++r) delta[i * CSP + r] = Ds[kw[p] * CSP + r] - Dold[cold[i] * CSP + r];
  }
}

// codebooks = fp32(D64), codes[c][p][m] = ct[m][c][p], and the final objective.
__global__ __launch_bounds__(kCThreads) void ecc_finish_kernel(const double* __restrict__ D64, EccParams q,
                                                             const uint8_t* __restrict__ ct,
                                                             float* __restrict__ D, uint8_t* __restrict__ codes,
                                                             const double* __restrict__ opart, int nopart,
                                                             double* __restrict__ objective) {
  const size_t tid = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
  const size_t nd = (size_t)q.M * q.K * q.Csp, nc = (size_t)q.M * q.Ct * q.P;
  for (size_t i = tid; i < nd; i += stride) D[i] = (float)D64[i];
  for (size_t i = tid; i < nc; i += stride) {  // i = (c P + p) M + m
    const size_t m = i % q.M, cp = i / q.M;
    codes[i] = ct[m * q.Ct * q.P + cp];
  }
  if (objective && blockIdx.x == 0) {  // the block sums in a fixed order: strided per thread, then a tree
    __shared__ double red[kCThreads];
    double s = 0.0;
    for (int b = threadIdx.x; b < nopart; b += kCThreads) s += opart[b];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int h = kCThreads / 2; h > 0; h >>= 1) {
      if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
      __syncthreads();
    }
    if (threadIdx.x == 0) *objective = red[0];
  }
}

EccParams make_params(int N, int Cs, int H, int W, int Ct, int dk, int stride, int pad, int M, int K, int Csp) {
  EccParams q{};
  q.N = N, q.Cs = Cs, q.H = H, q.W = W, q.Ct = Ct, q.dk = dk, q.stride = stride, q.pad = pad;
  q.Ho = (H + 2 * pad - dk) / stride + 1;
  q.Wo = (W + 2 * pad - dk) / stride + 1;
  q.M = M, q.K = K, q.Csp = Csp, q.P = dk * dk, q.O = q.Ho * q.Wo;
  // about 256 Ki correlation threads: (c, p) pairs times image chunks
  const int pairs = Ct * q.P;
  const int want = std::max(1, std::min(N, 262144 / std::max(1, pairs)));
  q.chunk = ceil_div(N, want);
  q.nchunks = ceil_div(N, q.chunk);
  return q;
}

}  // namespace

template <int CSP>
hipError_t launch_ecc_csp(const EccParams& q, const float* S, const float* T, float* D, uint8_t* codes, int sweeps,
                          int inner, double* objective, hipStream_t stream) {
  const size_t total = (size_t)q.N * q.Ct * q.O;
  const int npairs = q.Ct * q.P;
  const int eblocks = (int)ceil_div_z(total, kCThreads);
  const unsigned sbx = (unsigned)ceil_div(q.Ct, kStartTile), sby = (unsigned)ceil_div_z((size_t)q.N * q.O, kStartTile);
  const int sblocks = (int)(sbx * sby);  // the starting residual's block sums
  const int pblocks = ceil_div(npairs, kCThreads);
  // the Gram blocks go to LDS when they fit beside the rest
  const bool gl = rows_lds_bytes<CSP, true>(q.K, npairs, q.P) <= kLdsBytes;
  const size_t rlds = gl ? rows_lds_bytes<CSP, true>(q.K, npairs, q.P) : rows_lds_bytes<CSP, false>(q.K, npairs, q.P);
  const size_t slds = solve_lds_bytes<CSP>(q.K);
  constexpr int NW = kCThreads / kWave;
  const size_t blds = ((size_t)q.K * CSP + NW * (kWave / CSP) * CSP + NW * CSP) * 8 + (size_t)NW * q.P;
  if (rlds > kLdsBytes || slds > kLdsBytes || blds > kLdsBytes) return hipErrorInvalidValue;
  auto rows = gl ? ecc_rows_kernel<CSP, true> : ecc_rows_kernel<CSP, false>;
  auto solve = ecc_solve_kernel<CSP>;
  auto bupdate = ecc_bupdate_kernel<CSP>;
  hipError_t e = allow_max_lds((const void*)rows);
  if (e != hipSuccess) return e;
  if ((e = allow_max_lds((const void*)solve)) != hipSuccess) return e;
  if ((e = allow_max_lds((const void*)bupdate)) != hipSuccess) return e;
  Scratch scratch;
  size_t bytes = 0;
  PassShape ps{};
  const size_t pass_lds = pass_shape(q, &ps);
  const int nchunks = pass_lds ? ps.groups * ps.parts : q.nchunks;
  const int ablocks = pass_lds ? ceil_div(q.Ct, 64) * ps.groups * ps.parts : eblocks;  // block sums of a step's E^2
  const size_t szE = total * 8, szPart = (size_t)nchunks * npairs * CSP * 8, szH = (size_t)npairs * CSP * 8;
  const size_t szG = (size_t)q.M * q.P * q.P * CSP * CSP * 8, szD = (size_t)q.M * q.K * CSP * 8;
  const size_t szDelta = (size_t)npairs * CSP * 8, szOp = (size_t)std::max(std::max(eblocks, ablocks), sblocks) * 8, szCt = (size_t)q.M * npairs;
  const size_t szDold = (size_t)q.K * CSP * 8, szCold = (size_t)npairs, szQk = (size_t)q.P * q.K * 8;
  const size_t szB = system_doubles<CSP>(q.K) * 8, szX = (size_t)q.K * CSP * CSP * 8, szUsed = (size_t)q.K * 4;
  const size_t gram_lds = gram_lds_bytes(q), szGp = gram_lds ? kGramChunks * szG : 0;
  for (size_t b : {szE, szPart, szH, szG, szD, szDelta, szOp, szCt, szDold, szCold, szQk, szB, szX, szDold, szUsed, szGp})
    bytes += (b + 255) & ~(size_t)255;
  if ((e = scratch.acquire(stream, bytes)) != hipSuccess) return e;
  char* w = scratch.get();
  auto take = [&](size_t b) {
    char* r = w;
    w += (b + 255) & ~(size_t)255;
    return r;
  };
  double* E = reinterpret_cast<double*>(take(szE));
  double* part = reinterpret_cast<double*>(take(szPart));
  double* Hs = reinterpret_cast<double*>(take(szH));
  double* G = reinterpret_cast<double*>(take(szG));
  double* D64 = reinterpret_cast<double*>(take(szD));
  double* delta = reinterpret_cast<double*>(take(szDelta));
  double* opart = reinterpret_cast<double*>(take(szOp));
  uint8_t* ct = reinterpret_cast<uint8_t*>(take(szCt));
  double* Dold = reinterpret_cast<double*>(take(szDold));
  uint8_t* cold = reinterpret_cast<uint8_t*>(take(szCold));
  double* qkg = reinterpret_cast<double*>(take(szQk));
  double* B = reinterpret_cast<double*>(take(szB));
  double* X = reinterpret_cast<double*>(take(szX));
  double* r0 = reinterpret_cast<double*>(take(szDold));
  int* used = reinterpret_cast<int*>(take(szUsed));
  double* gpart = reinterpret_cast<double*>(take(szGp));

  const size_t ninit = std::max((size_t)q.M * q.K * CSP, (size_t)q.M * npairs);
  const unsigned iblocks = (unsigned)std::min<size_t>(8192, std::max<size_t>(1, ceil_div_z(ninit, kCThreads)));
  hipLaunchKernelGGL(ecc_init_kernel, dim3(iblocks), dim3(kCThreads), 0, stream, D, (const uint8_t*)codes, q, D64,
                     ct);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (gram_lds) {
    if ((e = launch_gram(S, q, gram_lds, gpart, G, stream)) != hipSuccess) return e;
  } else {
    const size_t ng = (size_t)q.M * q.P * q.P * CSP * CSP;
    hipLaunchKernelGGL(ecc_gram_kernel, dim3((unsigned)ceil_div_z(ng, kCThreads)), dim3(kCThreads), 0, stream, S, q,
                       G);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(ecc_start_kernel<CSP>, dim3(sbx, sby), dim3(kCThreads), 0, stream, S, T, q,
                     (const double*)D64, (const uint8_t*)ct, E, opart);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  int nstep = 0;
  int ma = -1;
  for (int s = 0; s < sweeps; ++s) {
    for (int m = 0; m < q.M; ++m, ++nstep) {
      if (pass_lds) {
        if ((e = launch_pass(S, q, ps, pass_lds, ma, m, delta, E, opart, part, stream)) != hipSuccess) return e;
      } else {
        if (ma >= 0) {
          hipLaunchKernelGGL(ecc_apply_kernel<CSP>, dim3((unsigned)eblocks), dim3(kCThreads), 0, stream, S, q, ma,
                             (const double*)delta, E, opart);
          if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        hipLaunchKernelGGL(ecc_corr_kernel<CSP>, dim3((unsigned)pblocks, (unsigned)q.nchunks), dim3(kCThreads), 0,
                           stream, S, q, m, (const double*)E, part);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      hipLaunchKernelGGL(ecc_reduce_kernel<CSP>, dim3((unsigned)ceil_div(npairs * CSP, kCThreads)), dim3(kCThreads), 0,
                         stream, (const double*)part, q, nchunks, m, (const double*)G, (const double*)D64,
                         (const uint8_t*)ct, Hs);
      if ((e = hipGetLastError()) != hipSuccess) return e;
      for (int it = 0; it < inner; ++it) {
        hipLaunchKernelGGL(rows, dim3((unsigned)q.K), dim3(rows_threads<CSP>()), rlds, stream, (const double*)Hs, q, m,
                           (const double*)G, (const double*)D64, (const uint8_t*)ct, B, X, r0, used);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(solve, dim3(1), dim3(kSolveThreads), slds, stream, q, m, (const double*)G, D64,
                           (const uint8_t*)ct, it == 0 ? 1 : 0, (const double*)B, (const double*)X,
                           (const double*)r0, (const int*)used, Dold, cold, qkg, (const double*)opart,
                           nstep == 0 ? sblocks : ablocks, objective ? objective + nstep : nullptr);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(bupdate, dim3((unsigned)ceil_div(q.Ct, NW)), dim3(kCThreads), blds, stream,
                           (const double*)Hs, q, m, (const double*)G, (const double*)D64, (const double*)qkg, ct,
                           (const double*)Dold, (const uint8_t*)cold, delta, it == inner - 1 ? 1 : 0);
        if ((e = hipGetLastError()) != hipSuccess) return e;
      }
      ma = m;
    }
  }
  if (ma >= 0 && pass_lds) {
    if ((e = launch_pass(S, q, ps, pass_lds, ma, -1, delta, E, opart, part, stream)) != hipSuccess) return e;
  } else if (ma >= 0) {
    hipLaunchKernelGGL(ecc_apply_kernel<CSP>, dim3((unsigned)eblocks), dim3(kCThreads), 0, stream, S, q, ma,
                       (const double*)delta, E, opart);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  hipLaunchKernelGGL(ecc_finish_kernel, dim3(iblocks), dim3(kCThreads), 0, stream, (const double*)D64, q,
                     (const uint8_t*)ct, D, codes, (const double*)opart, ma >= 0 ? ablocks : sblocks,
                     objective ? objective + nstep : nullptr);
  return hipGetLastError();
}

hipError_t launch_ec_conv(int N, int Cs, int H, int W, int Ct, int dk, int stride, int pad, int M, int K, int Csp,
                          const float* S, const float* T, float* D, uint8_t* codes, int sweeps, int inner,
                          double* objective, hipStream_t stream) {
  const EccParams q = make_params(N, Cs, H, W, Ct, dk, stride, pad, M, K, Csp);
#define QCNN_ECC_CASE(c) \
  case c: return launch_ecc_csp<c>(q, S, T, D, codes, sweeps, inner, objective, stream);
  switch (Csp) {
    QCNN_ECC_CASE(1) QCNN_ECC_CASE(2) QCNN_ECC_CASE(3) QCNN_ECC_CASE(4)
    QCNN_ECC_CASE(5) QCNN_ECC_CASE(6) QCNN_ECC_CASE(7) QCNN_ECC_CASE(8)
    default: return hipErrorInvalidValue;
  }
#undef QCNN_ECC_CASE
}

}  // namespace qcnn
