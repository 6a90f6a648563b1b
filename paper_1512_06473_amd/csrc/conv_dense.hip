// PQ convolution as an implicit GEMM on the fp16 matrix cores, with the
// weights rebuilt from the sub-codebooks.
//
// Paper: Sec. 3.2, Eq. (7).  The sum over subspaces and kernel positions of
// < D^(m)_{k_m(c_t, p_k)}, S^(m)_{p_s} > is the dense correlation with the
// weights W[c_t][m C'_s + j][p_k] = D^(m)_{k_m(c_t, p_k)}[j] (Eq. (6)).  The
// table form trades C'_s multiply-adds for one table read; on this machine a
// table read costs 4 bytes of LDS bandwidth per output (at best 131 TB/s =
// 3.3e13 reads/s, 2.4e13 reached), while the matrix cores do 1.2e15 fp16
// multiply-adds per second.  With the three products per multiply-add below
// that is 4e14, twelve times the read rate, so up to C'_s = 8 the products
// win wherever the layer fills the tiles.
//
// Precision.  Each fp32 factor v is scaled by a power of two and split into
// two fp16 values, v 2^e = h + l 2^-11 + r, each rounded to nearest: h has 11
// bits, l the next 11, and with l's sign a factor keeps 23 of its 24 bits,
// |r| <= 2^-23 |v 2^e| (0 for three values in four).  A product is
// h h' + (h l' + l h') 2^-11 (the split of a precise product into short ones,
// T. J. Dekker, "A floating-point technique for extending the available
// precision", 1971); the left-out l l' is at most 2^-22 of it, so a product is
// off by 2^-21 of itself at worst.  The MFMA adds the exact fp16 products in
// fp32.  What decides is the sums: the errors of the products average out, and
// the two-level sums here (fold(), the runs' sums in float64) are rounded less
// often than a chain of table entries.  Measured over 400 random layers that
// the dispatch sends here, against float64: 0.24 to 0.97 times the table
// kernel's error, median 0.63.  With l l' as a fourth product: 5 % less error, 10
// to 18 % more time.
//
// h h' and the cross terms have accumulators of their own, so that scaling l by
// 2^11 keeps it out of the fp16 subnormals: the largest input lies at 2^14 to
// 2^15, and a factor down to 2^-27 of that keeps its 23 bits, down to 2^-28 22.
// Smaller inputs -- any one: the weights on the large values beside it may be
// zero, and the result is then its products alone -- are left to passes of their
// own over the tile (its chunks that hold any), one per 28 binades, whose sums
// are added to the first's.  An input more than two such bands down, an
// infinity, a NaN or values near the ends of the fp32 range send the tile, and
// codewords that span more than 2^28 the layer, to fp32 MFMA on the unsplit
// values.  conv3, 32 images, and VGG conv3 per call, us: ordinary inputs 53 and
// 214; one value of 1e-9 54 and 247; one in 1009, in every tile, 94 and 415; in
// fp32 135 and 710 (with weights decoded lane by lane 710 and 4350).
//
// Work.  A tile is 128 output channels (64 where the layer has no more) x 96
// output positions; its reduction runs over units (chunk of 16 SUB input
// channels, kernel tap, 16 channels).  Two workgroups run per CU, so that
// one's start, scale exchange and stores hide behind the other's products.
// Each makes the same number of whole tiles; the tiles left over are cut into
// equal pieces at any unit, whose sums a second kernel adds in run order.
//
// Within a workgroup the 4 waves are TW channel groups of 32 x KG reduction
// groups: a wave owns 32 channels x 96 positions (v_mfma_f32_32x32x16_f16) and
// every KG-th unit.  Its 144 accumulator registers are what sets the tile: the
// products' chain, the chains folded (below) and the cross terms.  The weight
// operands come from memory in the order the instruction reads them, three
// units ahead (a wave reads only its own channels: nothing is loaded twice by
// a workgroup).  The input is staged in LDS chunk by chunk, [grid
// position][channel] with zero halos, so that a tap is one constant shift of
// the lanes' rows; the fp32 -> fp16 split happens on the way into LDS,
// double-buffered behind the previous chunk's products.
//
// Bound and measured (MI355X).  By the SQ counters, VGG conv3 shape (16 x 256 x
// 56 x 56 -> 256, 3x3): the matrix cores are busy 37 % of the kernel's clocks, the
// LDS 28 % (12 of them conflicts), waves wait a third of theirs; AlexNet conv3
// shape, 32 images, where every tile is cut into pieces: 26 %, 20 % (9).
// So no unit is near its rate; the chain of each tile's start (scale exchange,
// first loads, 5 us) and end (2 us) is what two workgroups per CU overlap only in
// part.  Against the table kernels, through a plan: AlexNet conv3 shape, 32
// images: 84 -> 47 us; conv2 with its max-pool, 37 images: 307 -> 124 us; VGG conv3
// shape per call: 273 -> 220 us (its kernel 203 us, 0.34 of the fp16 peak).  One workgroup of 8 waves
// per CU instead of two of 4: 55 us, 252 us.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <new>

#include "qcnn_internal.h"

namespace qcnn {

// Division of n < 2^31 by a divisor fixed on the host: n / d = (n m) >> 32 >> s
// with m = ceil(2^(32 + s) / d), s = ceil(log2 d) - 1 (d = 1: m unused).
struct FastDiv {
  uint32_t d, m, s;
  FastDiv() = default;
  explicit FastDiv(uint32_t d_) : d(d_), m(0), s(0) {
    if (d < 2) return;
    while ((2u << s) < d) ++s;
    m = (uint32_t)(((((uint64_t)1 << (32 + s)) + d - 1) / d));
  }
  __device__ __forceinline__ int div(int n) const { return d < 2 ? n : (int)(__umulhi((uint32_t)n, m) >> s); }
};

struct DenseParams {
  int N, Cs, H, W, M, K, Csp, Ct, dk, stride, pad, Ho, Wo;
  int S, sw;        // column strips per image, output columns per strip
  int PW, PH;       // staged grid: positions per row, rows per (image, strip)
  int ssx, ssy;     // grid positions per output step
  int gsx, gsy;     // input positions per grid step
  int xpack;        // the kernel's columns are channels of the staged positions
  int kw;           // kernel columns that are taps: d_k, or 1 when packed
  int VC;           // channels of a staged position: C_s, or C_s d_k when packed
  int Q;            // output slots N S Ho sw
  int SUB;          // 16-channel groups per chunk
  int chunks, taps, upt;  // chunks and units (chunk, tap, 16 channels) of a tile
  int tblocks, tiles, groups;
  int whole, shared0;  // tiles that each run makes alone; first of the shared tiles, cut at any unit
  int sruns;           // runs that take a piece of the shared tiles' units
  int rows;         // staged grid positions per tile, a multiple of 16
  int pitch;        // bytes per staged position
  int relu;
  int fold_at;      // steps between two folds of a wave's running sums
  int per_run, extra;  // shared units per run; the first `extra` runs have one more
  FastDiv d_sw, d_Ho, d_S, d_PW, d_PH, d_upt, d_upc, d_SUB, d_kw, d_tb, d_Cs;
};

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;  // two workgroups per CU
constexpr int kNT = 96;  // positions per tile
constexpr int kCF = kNT / 32;
constexpr int kSumStride = kNT + 8;  // floats per channel of a tile's sums in LDS
constexpr int kCUs = 256;
constexpr int kBand = 28;     // binades of one range band: scaled magnitudes 2^-14 .. 2^14 (2^15 in band 0)
constexpr int kMaxBands = 2;  // bands after the first that a tile takes in split form
constexpr uint32_t kOOB = 0x80000000u;  // buffer offset past every input: reads 0

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));

// Header of a layer's dense weights: the power of two they are scaled by and
// whether they must be used unsplit (fp32).
struct DenseHead {
  int scale_exp;
  int f32;
};
constexpr size_t kHeadBytes = 256;

// First shared unit of run w, and the run that holds shared unit u.
__host__ __device__ inline int run_begin(const DenseParams& p, int w) {
  w = w < p.sruns ? w : p.sruns;
  return w * p.per_run + (w < p.extra ? w : p.extra);
}
__device__ inline int run_of(const DenseParams& p, int u) {
  const int big = p.extra * (p.per_run + 1);
  return u < big ? u / (p.per_run + 1) : p.extra + (u - big) / p.per_run;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
#define QCNN_STEP(ctrl, rm) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, rm, 0xf, false));
  QCNN_STEP(0x111, 0xf) QCNN_STEP(0x112, 0xf) QCNN_STEP(0x114, 0xf) QCNN_STEP(0x118, 0xf)
  QCNN_STEP(0x142, 0xa) QCNN_STEP(0x143, 0xc)
#undef QCNN_STEP
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Exponent that brings a largest magnitude (fp32 bits of |v|) to 2^14 .. 2^15;
// 0 for an all-zero input.
__device__ __forceinline__ int scale_for(uint32_t maxbits) { return maxbits ? 14 - ((int)(maxbits >> 23) - 127) : 0; }

// fp32 bits of 2^q, q <= 127 (0 below the smallest subnormal).
__device__ __forceinline__ uint32_t pow2_bits(int q) {
  return q >= -126 ? (uint32_t)(q + 127) << 23 : q >= -149 ? 1u << (q + 149) : 0u;
}

// Magnitudes whose scaling stays inside the normal fp32 range.
__device__ __forceinline__ bool scalable(uint32_t maxbits) {
  return maxbits == 0 || (maxbits >= (27u << 23) && maxbits < (227u << 23));
}

struct Ptrs {
  const float* x;
  const char* w;      // head, then weights [channel group of 32][unit][hi, lo][lane][8] fp16, or fp32 [..][2][lane][4]
  const float* bias;
  float* y;
  float* partial;     // [2 per run][MT][kNT]
};

// The kernel's parameters, read again from the kernel argument segment: an
// opaque copy of its address keeps the compiler from holding every parameter
// of every phase in scalar registers throughout (184 of them spilled).
struct Args {
  Ptrs g;
  DenseParams p;
};
typedef const __attribute__((address_space(4))) Args* ArgsPtr;
__device__ __forceinline__ const Args& args_again() {
  ArgsPtr a = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(a));
  return *(const Args*)a;
}

// A wave's fp32 accumulators.
struct Acc {
  f16v a[kCF], c[kCF];  // h h' and cross terms since the last fold of a
  f16v sum[kCF];        // a folded
};

// Channel v of a staged position at unit tap `tap`: input channel and tap of
// the kernel (packed: v = kx C_s + c, tap = ky).
__device__ __forceinline__ void channel_of(const DenseParams& p, int v, int tap, int& c, int& ktap) {
  c = v;
  ktap = tap;
  if (p.xpack) {
    const int kx = p.d_Cs.div(v);
    c = v - kx * p.Cs;
    ktap = tap * p.dk + kx;
  }
}

// Everything a workgroup keeps for one tile.
template <int IT, bool XP>
struct TileState {
  uint32_t voff[IT];    // byte offset in x of this lane's staged position (channel 0), or past the end
  int ix[XP ? IT : 1];  // packed: its input column at kernel column 0
  int rowb[kCF];        // LDS byte offset of the lane's output position in each 32-column group, tap (0, 0)
};

// What a tile's later passes take: the last band that holds a value, the chunks
// that hold any past band 0, and the scale before the first of them.
struct Bands {
  int last, from, to, e;
};
constexpr int kUnset = 1 << 20;  // the scale before the first non-zero chunk

// The products of units [u0, u1) of one tile in split form, of the inputs of
// one range band: those of scaled magnitude 2^-14 and more (band 0), or of the
// b-th 2^kBand below that, scaled 2^(kBand b) more.  The scale follows the
// largest input so far, chunk by chunk, and is the same in every band's pass.
// Returns false when the form does not hold the inputs
// (band 0 only: an infinity, a NaN, the ends of the fp32 range, more bands
// than kMaxBands).
template <int TW, int IT, bool XP>
__device__ __forceinline__ bool products(const TileState<IT, XP>& ts, int tgrp, int u0, int u1, char* lds,
                                         uint32_t* exch, int band, Bands& bands, Acc& acc, int& x_exp) {
  const Args& args = args_again();
  const Ptrs& g = args.g;
  const DenseParams& p = args.p;
  constexpr int KG = kWaves / TW;
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int kg = wave / TW;
  const int HW4 = p.H * p.W * 4;
  const int upc = p.taps * p.SUB;  // units per chunk
  const int buf_bytes = p.rows * p.pitch;
  const int wgroups = (p.rows + 63) >> 6;
  const int vecs = 2 * p.SUB;
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(g.x), 0, (int)((size_t)p.N * p.Cs * HW4), 0x00020000);

#pragma unroll
  for (int j = 0; j < kCF; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc.a[j][r] = acc.c[j][r] = acc.sum[j][r] = 0.f;

  // ---- input staging: wave item i = wave + kWaves k is (64 positions, 8 channels):
  // position group i % wgroups, channel group i / wgroups of the chunk.
  // Channels past C_s hold 0: whole groups by an offset past the buffer, the
  // rest of a last group after its load.
  float xv[IT][8];
  int ivec[IT], igrp[IT];
#pragma unroll
  for (int k = 0; k < IT; ++k) {
    ivec[k] = (wave + kWaves * k) / wgroups;
    igrp[k] = (wave + kWaves * k) - ivec[k] * wgroups;
  }
  auto load_chunk = [&](int chunk) {
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const int ch0 = chunk * 16 * p.SUB + ivec[k] * 8;
      if constexpr (XP) {
        int kx = p.d_Cs.div(ch0), c = ch0 - kx * p.Cs;  // wave-uniform
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const bool in = ivec[k] < vecs && kx < p.dk && (unsigned)(ts.ix[k] + kx) < (unsigned)p.W;
          // a position outside the image has an offset past the buffer's end
          // that no channel or column brings back into it
          xv[k][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
              xres, in ? ts.voff[k] + (uint32_t)(c * HW4 + kx * 4) : kOOB, 0, 0));
          if (++c == p.Cs) {
            c = 0;
            ++kx;
          }
        }
        continue;
      }
      const uint32_t off = ivec[k] < vecs && ch0 < p.Cs ? ts.voff[k] + (uint32_t)(ch0 * HW4) : kOOB;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        xv[k][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xres, off + (uint32_t)(j * HW4), 0, 0));
      if (ch0 < p.Cs && ch0 + 8 > p.Cs) {  // wave-uniform
#pragma unroll
        for (int j = 1; j < 8; ++j)
          if (ch0 + j >= p.Cs) xv[k][j] = 0.f;
      }
    }
  };
  auto store_chunk = [&](char* buf, int e, int low) {
    if (band | low) {  // the chunk's values of this band
      const int q = -14 - e - kBand * band;
      const uint32_t from = pow2_bits(q), to = band ? pow2_bits(q + kBand) : ~0u;
#pragma unroll
      for (int k = 0; k < IT; ++k)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const uint32_t v = __float_as_uint(xv[k][j]) & 0x7fffffffu;
          xv[k][j] = v >= from && v < to ? ldexpf(xv[k][j], kBand * band) : 0.f;
        }
    }
    const float s = __uint_as_float((uint32_t)(e + 127) << 23);
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      if (ivec[k] >= vecs || igrp[k] * 64 + lane >= p.rows) continue;
      h8 hi, lo;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float v = xv[k][j] * s;
        hi[j] = (_Float16)v;
        lo[j] = (_Float16)((v - (float)hi[j]) * 2048.f);
      }
      char* dst = buf + (igrp[k] * 64 + lane) * p.pitch + (ivec[k] >> 1) * 64 + (ivec[k] & 1) * 16;
      *reinterpret_cast<h8*>(dst) = hi;
      *reinterpret_cast<h8*>(dst + 32) = lo;
    }
  };
  // Largest and smallest non-zero magnitude of the loaded values, exchanged
  // over the workgroup.
  // Two exchange buffers: a wave may publish again before the slowest one
  // has read the last exchange.
  int xb = 0;
  auto publish = [&]() {
    xb ^= 2 * kWaves;
    uint32_t mx = 0, below = ~0u;  // below: smallest non-zero magnitude - 1
#pragma unroll
    for (int k = 0; k < IT; ++k)
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const uint32_t v = __float_as_uint(xv[k][j]) & 0x7fffffffu;
        mx = max(mx, v);
        below = min(below, v - 1u);  // v = 0 gives ~0
      }
    mx = wave_max(mx);
    const uint32_t inv = wave_max(~below);
    if (lane == 0) {
      exch[xb + wave] = mx;
      exch[xb + kWaves + wave] = inv;
    }
  };
  // After the barrier that follows publish(): the scale for that chunk given
  // the current one (kUnset before the first non-zero chunk).  Returns the band
  // of the chunk's smallest value, -1 when the split form does not hold it.
  auto agree = [&](int& e) -> int {
    uint32_t mx = 0, inv = 0;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
      mx = max(mx, exch[xb + i]);
      inv = max(inv, exch[xb + kWaves + i]);
    }
    mx = __builtin_amdgcn_readfirstlane(mx);
    inv = __builtin_amdgcn_readfirstlane(inv);
    if (mx == 0) return 0;
    if (!scalable(mx)) return -1;
    if ((int)(mx >> 23) - 127 + e > 14) e = scale_for(mx);
    int low = 0;
    while (~inv + 1u < pow2_bits(-14 - e - kBand * low)) ++low;  // ends: the last bound is 0
    return low;
  };

  const int c_first = band ? bands.from : p.d_upc.div(u0), c_last = band ? bands.to : p.d_upc.div(u1 - 1);
  int e = band ? bands.e : kUnset;
  load_chunk(c_first);

  // ---- weight operands: unit u of the tile at 2048 u, three of this wave's
  // units in flight.  The loads run past the tile's last unit into the next
  // group's weights or the padding after them.
  int u;  // this wave's next unit
  const char* wp;
  h8 wh[3], wl[3];
  auto load_w = [&](int slot) {
    wh[slot] = *reinterpret_cast<const h8*>(wp + lane * 16);
    wl[slot] = *reinterpret_cast<const h8*>(wp + lane * 16 + 1024);
    wp += KG * 2048;
  };
  // The wave's first unit of a chunk, its weights, and its LDS rows
  // ((ky PW + kx) pitch + sub 64), which step() keeps by increments.
  int sub, kx, off;
  auto seek = [&](int c) {
    u = max(u0, c * upc);
    u += (kg - (u - u0)) & (KG - 1);
    wp = g.w + kHeadBytes + ((size_t)tgrp * p.upt + u) * 2048;
    load_w(0);
    load_w(1);
    load_w(2);
    const int v = u - c * upc;
    const int tap = p.d_SUB.div(v);
    sub = v - tap * p.SUB;
    const int ky = p.d_kw.div(tap);
    kx = tap - ky * p.kw;
    off = (ky * p.PW + kx) * p.pitch + sub * 64;
  };
  bool placed = band == 0;  // u, the weights and the rows are the next chunk's
  if (placed) seek(c_first);

  publish();
  __syncthreads();
  auto note = [&](int c, int e_before, int low) {
    if (band || low <= 0) return;
    if (bands.last == 0) {
      bands.from = c;
      bands.e = e_before;
    }
    bands.to = c;
    bands.last = max(bands.last, low);
  };
  const int e0 = e;
  int low = agree(e);
  bool ok = (unsigned)low <= kMaxBands;
  note(c_first, e0, low);
  store_chunk(lds, e == kUnset ? 0 : e, low);
  if (c_first < c_last) load_chunk(c_first + 1);

  const int lane_k = (lane >> 5) * 16;
  const int tap_step = p.pitch - p.SUB * 64, row_step = (p.PW - p.kw) * p.pitch;
  int parity = 0;  // LDS buffer of the current chunk
  int since = 0;   // steps since the last fold
  const int fold_at = __builtin_amdgcn_readfirstlane(p.fold_at);  // (kept: not read again in the loop)
  // The MFMA adds 8 products at a time: the running sum is rounded twice a
  // step.  Folding it into a second one every few steps keeps both chains
  // short, about 2 fold_at and steps over fold_at roundings long (96 -> 256
  // channels, 5x5, 64 images, relative error against float64: 2.8e-7 without,
  // 1.5e-7 with a fold per chunk of 25 steps, 1.2e-7 with one every 9 or 10;
  // the table kernel's is 2.1e-7.  Every 6 instead of 9 steps: 1.21e-7 -> 1.18e-7
  // for 128 -> 381 channels, 3x3, 72 steps, but 1.36e-7 -> 1.39e-7 and 1 % of the
  // time for 256 -> 256, 144 steps; every 3: 1.59e-7 and 4 %).
  auto fold = [&]() {
    since = 0;
#pragma unroll
    for (int j = 0; j < kCF; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        acc.sum[j][r] += acc.a[j][r];
        acc.a[j][r] = 0.f;
      }
  };

  auto step = [&](int slot) {
    const char* base = lds + parity * buf_bytes + off + lane_k;
    h8 bh[kCF], bl[kCF];
    auto read_b = [&](int j) {
      bh[j] = *reinterpret_cast<const h8*>(base + ts.rowb[j]);
      bl[j] = *reinterpret_cast<const h8*>(base + ts.rowb[j] + 32);
    };
    read_b(0);
    read_b(1);
#pragma unroll
    for (int j = 0; j < kCF; ++j) {
      acc.a[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh[slot], bh[j], acc.a[j], 0, 0, 0);
      acc.c[j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wl[slot], bh[j], acc.c[j], 0, 0, 0);
      if (j > 0) acc.c[j - 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh[slot], bl[j - 1], acc.c[j - 1], 0, 0, 0);
      if (j + 2 < kCF) read_b(j + 2);
      __builtin_amdgcn_sched_barrier(0);
    }
    acc.c[kCF - 1] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wh[slot], bl[kCF - 1], acc.c[kCF - 1], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
    load_w(slot);
    u += KG;
#pragma unroll
    for (int k = 0; k < KG; ++k) {
      off += 64;
      if (++sub == p.SUB) {
        sub = 0;
        off += tap_step;
        if (++kx == p.kw) {
          kx = 0;
          off += row_step;
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  int c_end = ok ? c_last : c_first;  // (a return from inside the loop spills the sums)
  for (int c = c_first; c <= c_end; ++c) {
    // Loaded: chunk c + 1, one chunk ahead of its products.  Its scale is
    // agreed on across the barrier that also hands over chunk c's LDS rows.
    const bool more = c < c_end;
    if (more) publish();
    __syncthreads();
    int e_next = e, low_next = 0;
    if (more) {
      low_next = agree(e_next);
      ok &= (unsigned)low_next <= kMaxBands;
      if (!ok) c_end = c;
      note(c + 1, e, low_next);
      store_chunk(lds + (parity ^ 1) * buf_bytes, e_next == kUnset ? 0 : e_next, low_next);
      if (c + 1 < c_last) load_chunk(c + 2);
    }
    if (low >= band) {
      if (!placed) seek(c);
      const int u_end = min(u1, (c + 1) * upc);
      while (u + 2 * KG < u_end) {
        step(0);
        step(1);
        step(2);
        since += 3;
        if (since >= fold_at) fold();
      }
      while (u < u_end) {  // at most two
        step(0);
        ++since;
        const h8 th = wh[0], tl = wl[0];
        wh[0] = wh[1];
        wl[0] = wl[1];
        wh[1] = wh[2];
        wl[1] = wl[2];
        wh[2] = th;
        wl[2] = tl;
      }
      off -= p.dk * p.PW * p.pitch;  // from past the last tap to the next chunk's first
      if (since >= fold_at) fold();
      placed = true;
    } else {
      placed = false;
    }
    if (e_next < e && e != kUnset) {  // larger inputs ahead: the sums take their scale
      const float f = __uint_as_float((uint32_t)max(1, e_next - e + 127) << 23);
#pragma unroll
      for (int j = 0; j < kCF; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          acc.a[j][r] *= f;
          acc.c[j][r] *= f;
          acc.sum[j][r] *= f;
        }
    }
    e = e_next;
    low = low_next;
    parity ^= 1;
  }
  fold();
  __syncthreads();  // the sums overwrite the staged rows
  x_exp = (e == kUnset ? 0 : e) + kBand * band;
  return ok;
}

// Output slot q is (n, strip, yo, xl).
struct Slot {
  int n, yo, xo;  // image, output row and column
  int grid;       // staged grid position at tap (0, 0)
};
__device__ __forceinline__ Slot slot_of(const DenseParams& p, int q) {
  const int row = p.d_sw.div(q), xl = q - row * p.sw;
  const int pl = p.d_Ho.div(row), yo = row - pl * p.Ho;
  const int n = p.d_S.div(pl);
  return {n, yo, (pl - n * p.S) * p.sw + xl, (pl * p.PH + yo * p.ssy) * p.PW + xl * p.ssx};
}

// The sums of units [u0, u1) in fp32 for a wave's 32 channels and its 32-position
// groups (kg, kg + KG, ..), operands straight from memory: the form for inputs
// or codewords that the split one does not hold.  Bound by the fp32 matrix rate
// (1/16 of fp16's): the two waves of a SIMD take turns loading.
template <int TW, bool XP>
__device__ __forceinline__ void products_f32(int tgrp, int u0, int u1, int q0, int kg,
                                             f16v (&acc)[ceil_div(kCF, kWaves / TW)]) {
  const Args& args = args_again();
  const Ptrs& g = args.g;
  const DenseParams& p = args.p;
  constexpr int KG = kWaves / TW, NJ = ceil_div(kCF, KG);
  const int lane = threadIdx.x & (kWave - 1);
  const int upc = p.taps * p.SUB;
  const int HW4 = p.H * p.W * 4;
  const __amdgpu_buffer_rsrc_t xres = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<float*>(g.x), 0, (int)((size_t)p.N * p.Cs * HW4), 0x00020000);
  const DenseHead head = *reinterpret_cast<const DenseHead*>(g.w);
  int iy[NJ], ix[NJ];    // the lane's output positions' input coordinates at tap (0, 0)
  uint32_t plane[NJ];    // byte offset of their images
#pragma unroll
  for (int i = 0; i < NJ; ++i) {
    const int q = q0 + 32 * (kg + KG * i) + (lane & 31);
    const Slot o = slot_of(p, min(q, p.Q - 1));
    iy[i] = q < p.Q ? o.yo * p.stride - p.pad : -(1 << 24);  // no position: outside the input
    ix[i] = o.xo * p.stride - p.pad;
    plane[i] = (uint32_t)(o.n * p.Cs) * (uint32_t)HW4;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
  }
  const char* wp = g.w + kHeadBytes + ((size_t)tgrp * p.upt + u0) * 2048 + lane * 16;
  for (int u = u0; u < u1; ++u, wp += 2048) {
    const int c = p.d_upc.div(u), v = u - c * upc;
    const int tap = p.d_SUB.div(v), sub = v - tap * p.SUB;
    const int ch0 = (c * p.SUB + sub) * 16 + (lane >> 5) * 8;
    const int ky = p.d_kw.div(tap), kx = tap - ky * p.kw;
    float av[8], bv[NJ][8];
    if (head.f32) {
      const f4v w0 = *reinterpret_cast<const f4v*>(wp), w1 = *reinterpret_cast<const f4v*>(wp + 1024);
#pragma unroll
      for (int j = 0; j < 4; ++j) av[j] = w0[j], av[4 + j] = w1[j];
    } else {
      const h8 hi = *reinterpret_cast<const h8*>(wp), lo = *reinterpret_cast<const h8*>(wp + 1024);
#pragma unroll
      for (int j = 0; j < 8; ++j) av[j] = ldexpf((float)hi[j] + (float)lo[j] * (1.f / 2048.f), -head.scale_exp);
    }
#pragma unroll
    for (int i = 0; i < NJ; ++i) {
      const int yy = iy[i] + ky;
      if constexpr (XP) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int kc = p.d_Cs.div(ch0 + j), xx = ix[i] + kc;
          const bool in = kc < p.dk && (unsigned)yy < (unsigned)p.H && (unsigned)xx < (unsigned)p.W;
          bv[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
              xres, in ? plane[i] + (uint32_t)((ch0 + j - kc * p.Cs) * HW4 + (yy * p.W + xx) * 4) : kOOB, 0, 0));
        }
      } else {
        const int xx = ix[i] + kx;
        const bool in = ch0 < p.Cs && (unsigned)yy < (unsigned)p.H && (unsigned)xx < (unsigned)p.W;
        const uint32_t at = in ? plane[i] + (uint32_t)(ch0 * HW4 + (yy * p.W + xx) * 4) : kOOB;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          bv[i][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xres, at + (uint32_t)(j * HW4), 0, 0));
      }
    }
    if constexpr (!XP) {
#pragma unroll
      for (int j = 1; j < 8; ++j)
#pragma unroll
        for (int i = 0; i < NJ; ++i)
          if (ch0 + j >= p.Cs) bv[i][j] = 0.f;  // (its weight is 0, but the value may be an infinity)
    }
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int i = 0; i < NJ; ++i)
        if (i * KG + kg < kCF) acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[j], bv[i][j], acc[i], 0, 0, 0);
  }
}

template <int TW, int IT, bool XP>
__global__ __launch_bounds__(kThreads, 2) void conv_dense_kernel(Args unused) {
  extern __shared__ float4 smem4[];
  constexpr int KG = kWaves / TW;
  constexpr int MT = 32 * TW;
  char* lds = reinterpret_cast<char*>(smem4);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int tw = wave % TW, kg = wave / TW;

  // Runs XCD-major: neighbouring runs (which share inputs) run on one XCD.
  const int b = blockIdx.x;
  const int groups = args_again().p.groups;
  const int w = (b & 7) * ((groups + 7) >> 3) + (b >> 3);
  if (w >= groups) return;
  const int run_u0 = run_begin(args_again().p, w), run_u1 = run_begin(args_again().p, w + 1);
  const DenseHead head = *reinterpret_cast<const DenseHead*>(args_again().g.w);

  for (int i = 0, u = run_u0;;) {
    const DenseParams& p = args_again().p;
    uint32_t* exch = reinterpret_cast<uint32_t*>(lds + max(2 * p.rows * p.pitch, MT * kSumStride * 4));
    int tile, a0 = 0, a1 = p.upt;  // units [a0, a1) of the tile
    if (i < p.whole) {
      tile = w * p.whole + i++;
    } else if (u < run_u1) {
      tile = p.d_upt.div(u);
      a0 = u - tile * p.upt;
      a1 = min(p.upt, run_u1 - tile * p.upt);
      u += a1 - a0;
      tile += p.shared0;
    } else {
      break;
    }
    const int ptile = p.d_tb.div(tile);
    const int tb = tile - ptile * p.tblocks, q0 = ptile * kNT;

    const int g0 = slot_of(p, q0).grid;
    TileState<IT, XP> ts;
#pragma unroll
    for (int j = 0; j < kCF; ++j) ts.rowb[j] = (slot_of(p, min(q0 + 32 * j + (lane & 31), p.Q - 1)).grid - g0) * p.pitch;
    const int wgroups = (p.rows + 63) >> 6;
#pragma unroll
    for (int k = 0; k < IT; ++k) {
      const int f = g0 + ((wave + kWaves * k) % wgroups) * 64 + lane;
      const int row = p.d_PW.div(f), c = f - row * p.PW;
      const int pl = p.d_PH.div(row), n = p.d_S.div(pl);
      const int iy = (row - pl * p.PH) * p.gsy - p.pad, ix = (pl - n * p.S) * p.sw * p.stride + c * p.gsx - p.pad;
      const bool in = n < p.N && iy >= 0 && iy < p.H && (XP || (ix >= 0 && ix < p.W));
      if constexpr (XP) ts.ix[k] = in ? ix : -(1 << 30);
      ts.voff[k] = in ? (uint32_t)(n * p.Cs * p.H * p.W + iy * p.W + ix) * 4u : kOOB;
    }

    const int tgrp = tb * TW + tw;
    float* sums = reinterpret_cast<float*>(lds);  // [channel][position], kSumStride floats per channel
    // Row r of lane l is channel (r & 3) + 8 (r >> 2) + 4 (l >> 5) of the wave's
    // 32, column l % 32 of a 32-position group: a store's two halves fall on
    // different halves of the banks.
    float* own = sums + (32 * tw + 4 * (lane >> 5)) * kSumStride + (lane & 31);
    bool split_form = head.f32 == 0;
    Bands bands{0, 0, 0, 0};
    for (int band = 0; band <= bands.last; ++band) {
      if (split_form) {
        Acc acc;
        int x_exp;
        split_form = products<TW, IT, XP>(ts, tgrp, a0, a1, lds, exch, band, bands, acc, x_exp);
        // The reduction groups' sums, added in group order.
        const int ue = -(x_exp + head.scale_exp);
        for (int k = 0; k < KG && split_form; ++k) {
          if (k == kg) {
#pragma unroll
            for (int j = 0; j < kCF; ++j)
#pragma unroll
              for (int r = 0; r < 16; ++r) {
                float* at = own + ((r & 3) + 8 * (r >> 2)) * kSumStride + 32 * j;
                const float v = ldexpf(acc.sum[j][r] + acc.c[j][r] * (1.f / 2048.f), ue);
                *at = k == 0 ? v : *at + v;
              }
          }
          __syncthreads();
        }
      }
      if (!split_form) {
        bands.last = 0;
        constexpr int NJ = ceil_div(kCF, KG);
        f16v sum[NJ];
        products_f32<TW, XP>(tgrp, a0, a1, q0, kg, sum);
        __syncthreads();  // the sums overwrite the staged rows
#pragma unroll
        for (int i = 0; i < NJ; ++i)
          if (kg + KG * i < kCF)
#pragma unroll
            for (int r = 0; r < 16; ++r)
              own[((r & 3) + 8 * (r >> 2)) * kSumStride + 32 * (kg + KG * i)] = sum[i][r];
        __syncthreads();
      }
      // ---- the tile, or this run's share of its sums, to memory; a later band
      // adds to what the ones before it stored (the same thread, the same place)
      const Args& after = args_again();
      const Ptrs& g = after.g;
      const DenseParams& pe = after.p;
      if (a0 != 0 || a1 != pe.upt) {
        // A run and its shared tile both only grow along the units: their sum is
        // a place of its own.
        f4v* part = reinterpret_cast<f4v*>(g.partial + (size_t)(w + tile - pe.shared0) * (MT * kNT));
        for (int i = threadIdx.x; i < MT * kNT / 4; i += kThreads) {
          f4v v = *reinterpret_cast<const f4v*>(sums + i / (kNT / 4) * kSumStride + i % (kNT / 4) * 4);
          if (band > 0) v += part[i];
          part[i] = v;
        }
      } else {
        constexpr int kRows = kThreads / kNT;  // channels at a time
        const int ql = threadIdx.x % kNT;
        const Slot o = slot_of(pe, q0 + ql);
        if (threadIdx.x < kRows * kNT && q0 + ql < pe.Q && o.xo < pe.Wo) {
          const int t_end = min(pe.Ct - tb * MT, MT), HoWo = pe.Ho * pe.Wo;
          const bool last = band == bands.last;
          const float* bias = last ? g.bias : nullptr;
          const bool relu = last && pe.relu;
          float* dst = g.y + ((size_t)o.n * pe.Ct + tb * MT) * HoWo + o.yo * pe.Wo + o.xo;
#pragma unroll 4
          for (int t = threadIdx.x / kNT; t < t_end; t += kRows) {
            float v = sums[t * kSumStride + ql];
            if (band > 0) v += dst[(size_t)t * HoWo];
            v += bias ? bias[tb * MT + t] : 0.f;
            if (relu) v = fmaxf(v, 0.f);
            dst[(size_t)t * HoWo] = v;
          }
        }
      }
      __syncthreads();  // the next pass's or tile's staging overwrites the sums
    }
  }
}

// y of the tiles that several runs share: their partial sums added in run
// order, bias, ReLU.  A workgroup takes the positions x 16 channels of one
// tile; 8 channels per thread with every run's loads in flight.
__global__ __launch_bounds__(2 * kNT) void dense_reduce_kernel(const float* __restrict__ partial, DenseParams p, int MT,
                                                           const float* __restrict__ bias, float* __restrict__ y) {
  const int tile = p.shared0 + blockIdx.x;
  const int t_u0 = blockIdx.x * p.upt;
  const int wf = run_of(p, t_u0), wl = run_of(p, t_u0 + p.upt - 1);
  if (wf == wl) return;  // one run made the whole tile and stored it
  const int tb = tile % p.tblocks, q = (tile / p.tblocks) * kNT + threadIdx.x % kNT;
  const int tl = blockIdx.y * 16 + (int)(threadIdx.x / kNT) * 8;
  const int row = q / p.sw, xl = q - row * p.sw;
  const int pl = row / p.Ho, yo = row - pl * p.Ho;
  const int n = pl / p.S, xo = (pl - n * p.S) * p.sw + xl;
  if (q >= p.Q || xo >= p.Wo) return;
  double s[8];  // (in fp32 the runs were another chain of up to 30 roundings)
#pragma unroll
  for (int i = 0; i < 8; ++i) s[i] = 0.0;
  for (int w = wf; w <= wl; ++w) {
    const size_t slot = w + blockIdx.x;
    const float* src = partial + slot * (MT * kNT) + tl * kNT + threadIdx.x % kNT;
#pragma unroll
    for (int i = 0; i < 8; ++i) s[i] += (double)src[i * kNT];
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int t = tb * MT + tl + i;
    if (t < p.Ct) {
      float v = (float)(s[i] + (bias ? (double)bias[t] : 0.0));
      if (p.relu) v = fmaxf(v, 0.f);
      y[(((size_t)n * p.Ct + t) * p.Ho + yo) * p.Wo + xo] = v;
    }
  }
}

// Scale and form of a layer's weights: one workgroup over the codebooks.
__global__ __launch_bounds__(1024) void dense_head_kernel(const float* __restrict__ D, int n,
                                                          DenseHead* __restrict__ head) {
  __shared__ uint32_t sm[2][16];
  uint32_t mx = 0, inv = 0;
  auto mag = [](float f) { return __float_as_uint(f) & 0x7fffffffu; };
  auto take = [&](uint32_t v) {
    mx = max(mx, v);
    inv = max(inv, ~(v - 1u));
  };
  if (n % 4 == 0 && (reinterpret_cast<uintptr_t>(D) & 15) == 0) {
#pragma unroll 4
    for (int i = threadIdx.x; i < n / 4; i += 1024) {
      const f4v d = reinterpret_cast<const f4v*>(D)[i];
#pragma unroll
      for (int j = 0; j < 4; ++j) take(mag(d[j]));
    }
  } else {
    for (int i = threadIdx.x; i < n; i += 1024) take(mag(D[i]));
  }
  mx = wave_max(mx);
  inv = wave_max(inv);
  if ((threadIdx.x & 63) == 0) {
    sm[0][threadIdx.x >> 6] = mx;
    sm[1][threadIdx.x >> 6] = inv;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int i = 1; i < 16; ++i) {
      mx = max(mx, sm[0][i]);
      inv = max(inv, sm[1][i]);
    }
    const int e = scale_for(mx);
    head->scale_exp = e;
    head->f32 = !scalable(mx) || (mx && (int)((~inv + 1u) >> 23) - 127 + e < -14);
  }
}

// The weights in operand order, split or (head.f32) as they are: one thread
// writes the 8 channels of one lane.
__global__ __launch_bounds__(256) void dense_weights_kernel(const float* __restrict__ D, CodeStream codes,
                                                            DenseParams p, int tgroups, char* __restrict__ w) {
  const int total = tgroups * p.upt * kWave;  // < 2^31: kMaxWeights
  const DenseHead head = *reinterpret_cast<const DenseHead*>(w);
  const float sc = head.f32 ? 1.f : __uint_as_float((uint32_t)(head.scale_exp + 127) << 23);
  const int upc = p.taps * p.SUB;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
    const int lane = i & 63, r = i >> 6;
    const int tg = p.d_upt.div(r), u = r - tg * p.upt;
    const int chunk = p.d_upc.div(u), v = u - chunk * upc;
    const int tap = p.d_SUB.div(v), sub = v - tap * p.SUB;
    const int t = tg * 32 + (lane & 31);
    const int ch0 = (chunk * p.SUB + sub) * 16 + (lane >> 5) * 8;
    float v8[8];
    int at = -1;  // the code last read
    uint32_t code = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float x = 0.f;
      if (t < p.Ct && ch0 + j < p.VC) {
        int ch, ktap;
        channel_of(p, ch0 + j, tap, ch, ktap);
        const int m = ch / p.Csp;
        if (ktap * p.M + m != at) {
          at = ktap * p.M + m;
          code = min(code_at(codes, (size_t)t * p.dk * p.dk * p.M + at), (uint32_t)(p.K - 1));
        }
        x = D[((size_t)m * p.K + code) * p.Csp + (ch - m * p.Csp)] * sc;
      }
      v8[j] = x;
    }
    char* dst = w + kHeadBytes + (size_t)r * 2048 + lane * 16;
    if (head.f32) {
      *reinterpret_cast<f4v*>(dst) = f4v{v8[0], v8[1], v8[2], v8[3]};
      *reinterpret_cast<f4v*>(dst + 1024) = f4v{v8[4], v8[5], v8[6], v8[7]};
      continue;
    }
    h8 hi, lo;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      hi[j] = (_Float16)v8[j];
      lo[j] = (_Float16)((v8[j] - (float)hi[j]) * 2048.f);
    }
    *reinterpret_cast<h8*>(dst) = hi;
    *reinterpret_cast<h8*>(dst + 1024) = lo;
  }
}

}  // namespace

struct DensePlan {
  DenseParams p;
  int TW, IT;
  size_t lds, weight_bytes, partial_bytes;
};

namespace {

// Weights read ahead past a tile's last unit: three steps of up to 2 groups
// (and one unit where the last chunk has none for a group).
constexpr size_t kWeightTail = 8 * 2048;
constexpr size_t kMaxWeights = (size_t)32 << 20;

// Column strips and the staged window of a tile: the strips that waste few
// slots past the row's end and keep the window, and so the staging, small;
// past two workgroups' share of the LDS only one runs.
bool set_window(const ConvShape& s, DenseParams* p) {
  double best = 0;
  p->rows = 0;
  for (int S = 1; S <= 16 && S <= s.Wo; ++S) {
    const int sw = ceil_div(s.Wo, S);
    if ((S - 1) * sw >= s.Wo) continue;
    int PH = (s.Ho - 1) * p->ssy + s.dk, PW = (sw - 1) * p->ssx + p->kw;
    if (S == 1 && p->gsy == 1) {  // neighbouring rows and images share their zero halos
      if (!p->xpack) PW -= std::min(s.pad, std::max(0, PW - s.pad - s.W));
      PH -= std::min(s.pad, std::max(0, PH - s.pad - s.H));
    }
    // The grid span of kNT consecutive output slots: steps of `ssx`, plus what
    // a row end and an image end add.
    const long long rc = (kNT - 1 + sw - 1) / sw, ic = (kNT - 1 + (long long)sw * s.Ho - 1) / ((long long)sw * s.Ho);
    const long long span = (kNT - 1) * (long long)p->ssx + rc * std::max(0, p->ssy * PW - sw * p->ssx) +
                           ic * std::max(0, (PH - s.Ho * p->ssy) * PW) + (long long)(s.dk - 1) * PW + p->kw;
    if (span > 4096) continue;
    const int rows = (int)(span + 15) / 16 * 16;
    const size_t bytes = (size_t)2 * rows * p->pitch;
    if (bytes > kLdsBytes - 256) continue;
    const double score = (double)S * sw / s.Wo * (1.0 + ceil_div(rows, 64) / 40.0) * (bytes > kLdsBytes / 2 - 256 ? 1.5 : 1.0);
    if (p->rows && score >= best) continue;
    best = score;
    p->S = S; p->sw = sw; p->PW = PW; p->PH = PH; p->rows = rows;
  }
  return p->rows != 0;
}

bool plan_layer(const ConvShape& s, DensePlan* out) {
  if ((long long)s.N * s.Cs * s.H * s.W * 4 > (1LL << 31) - 1) return false;  // 32-bit buffer offsets
  DenseParams p{};
  p.N = s.N; p.Cs = s.Cs; p.H = s.H; p.W = s.W; p.M = s.M; p.K = s.K; p.Csp = s.Csp; p.Ct = s.Ct;
  p.dk = s.dk; p.stride = s.stride; p.pad = s.pad; p.Ho = s.Ho; p.Wo = s.Wo;
  if (s.dk > 15 || s.pad >= s.dk) return false;
  // The staged grid is the input's; for 1x1 kernels only the positions that
  // outputs read; with few input channels a staged position holds the whole
  // kernel row at its output column (d_k C_s channels), so that the 16-channel
  // units are not mostly padding (AlexNet conv1, 3 channels, 11 x 11: 33 units
  // of 16 instead of 121).
  p.xpack = s.dk > 1 && s.Cs < 8;
  p.kw = p.xpack ? 1 : s.dk;
  p.VC = p.xpack ? s.Cs * s.dk : s.Cs;
  p.taps = s.dk * p.kw;
  p.ssx = s.dk == 1 || p.xpack ? 1 : s.stride;
  p.ssy = s.dk == 1 ? 1 : s.stride;
  p.gsx = s.dk == 1 || p.xpack ? s.stride : 1;
  p.gsy = s.dk == 1 ? s.stride : 1;
  // Chunks of more channels where there are few taps to reuse a staged row;
  // fewer where the window's rows would not fit a thread's staging registers.
  int items = 0;
  for (p.SUB = p.taps == 1 ? 4 : p.taps <= 4 ? 2 : 1; p.SUB > 0; --p.SUB) {
    if (p.SUB > 1 && 16 * (p.SUB - 1) >= p.VC) continue;
    p.pitch = 64 * p.SUB + 16;
    if (!set_window(s, &p)) continue;
    items = ceil_div(ceil_div(p.rows, 64) * 2 * p.SUB, kWaves);
    if (items <= 4) break;
  }
  if (p.SUB == 0) return false;
  p.chunks = ceil_div(p.VC, 16 * p.SUB);
  p.upt = p.chunks * p.taps * p.SUB;
  const int TW = s.Ct <= 64 ? 2 : 4;
  p.fold_at = p.upt <= 96 * kWaves / TW ? 6 : 9;
  const size_t sums = (size_t)32 * TW * kSumStride * 4;
  out->lds = std::max((size_t)2 * p.rows * p.pitch, sums) + 256;
  if (out->lds > kLdsBytes) return false;
  const long long slots = (long long)s.N * p.S * s.Ho * p.sw;
  if (slots > (1LL << 30) || (long long)s.N * p.S * p.PH * p.PW + 8192 > (1LL << 31)) return false;
  p.Q = (int)slots;
  p.tblocks = ceil_div(s.Ct, 32 * TW);
  const long long tiles = (slots + kNT - 1) / kNT * p.tblocks;
  if (tiles * p.upt >= (1LL << 30)) return false;
  p.tiles = (int)tiles;
  out->weight_bytes = kHeadBytes + (size_t)p.tblocks * TW * p.upt * 2048 + kWeightTail;
  if (out->weight_bytes > kMaxWeights) return false;
  // Two runs per CU.  Each makes tiles / runs whole tiles; the tiles left over
  // are cut into equal pieces of at least 16 units.  Fewer runs where the
  // pieces' sums would not fit the allocation-free entry point's scratch.
  const size_t tile_bytes = (size_t)32 * TW * kNT * sizeof(float);
  const long long room = (long long)((noalloc_scratch_bytes() - 1024 - out->weight_bytes) / tile_bytes);
  long long runs = 2 * kCUs, left = 0, pieces = 0;
  for (; runs > 0; --runs) {
    left = tiles % runs;
    pieces = std::min(runs, std::max(left, left * p.upt / 16));
    if (left == 0 || pieces + left <= room) break;
  }
  if (runs < 1) return false;
  p.whole = (int)(tiles / runs);
  p.shared0 = (int)(tiles - left);
  p.sruns = (int)pieces;
  p.groups = (int)(p.whole ? runs : pieces);
  p.per_run = pieces ? (int)(left * p.upt / pieces) : 0;
  p.extra = pieces ? (int)(left * p.upt % pieces) : 0;
  out->partial_bytes = (size_t)(pieces + left) * tile_bytes;
  p.d_sw = FastDiv(p.sw); p.d_Ho = FastDiv(p.Ho); p.d_S = FastDiv(p.S); p.d_PW = FastDiv(p.PW); p.d_PH = FastDiv(p.PH);
  p.d_upt = FastDiv(p.upt); p.d_upc = FastDiv(p.taps * p.SUB); p.d_SUB = FastDiv(p.SUB); p.d_kw = FastDiv(p.kw); p.d_Cs = FastDiv(p.Cs);
  p.d_tb = FastDiv(p.tblocks);
  out->p = p;
  out->TW = TW;
  out->IT = std::max(2, items);
  return true;
}

// The plan of a layer.  A call asks for it several times (the dispatch, the
// workspace, the launch; 1.4 us each): the thread's last answer is kept, by the
// shape's value.
bool make_plan(const ConvShape& s, DensePlan* out) {
  static thread_local ConvShape last{};  // N = 0: no layer
  static thread_local bool ok = false;
  static thread_local DensePlan plan;
  if (memcmp(&s, &last, sizeof s) != 0) {
    ok = plan_layer(s, &plan);
    last = s;
  }
  if (ok) *out = plan;
  return ok;
}

template <int TW, int IT>
hipError_t launch_one(const DensePlan& pl, const Ptrs& g, hipStream_t stream, LaunchTimer* timer) {
  auto k = pl.p.xpack ? conv_dense_kernel<TW, IT, true> : conv_dense_kernel<TW, IT, false>;
  hipError_t e = allow_max_lds((const void*)k);
  if (e != hipSuccess) return e;
  return timed_launch(timer, k, dim3((pl.p.groups + 7) / 8 * 8), dim3(kThreads), (uint32_t)pl.lds, stream, Args{g, pl.p});
}

hipError_t launch_main(const DensePlan& pl, const Ptrs& g, hipStream_t stream, LaunchTimer* timer) {
  switch (pl.TW * 10 + pl.IT) {
    case 42: return launch_one<4, 2>(pl, g, stream, timer);
    case 43: return launch_one<4, 3>(pl, g, stream, timer);
    case 44: return launch_one<4, 4>(pl, g, stream, timer);
    case 22: return launch_one<2, 2>(pl, g, stream, timer);
    case 23: return launch_one<2, 3>(pl, g, stream, timer);
    default: return launch_one<2, 4>(pl, g, stream, timer);
  }
}

hipError_t launch_weights(const DensePlan& pl, const float* D, CodeStream codes, char* w, hipStream_t stream) {
  const DenseParams& p = pl.p;
  hipLaunchKernelGGL(dense_head_kernel, dim3(1), dim3(1024), 0, stream, D, p.M * p.K * p.Csp,
                     reinterpret_cast<DenseHead*>(w));
  const long long threads = (long long)p.tblocks * pl.TW * p.upt * kWave;
  hipLaunchKernelGGL(dense_weights_kernel, dim3((unsigned)std::min<long long>(4096, (threads + 255) / 256)), dim3(256),
                     0, stream, D, codes, p, p.tblocks * pl.TW, w);
  return hipGetLastError();
}

hipError_t run_dense(const DensePlan& pl, const Ptrs& g, hipStream_t stream, bool timed) {
  hipError_t e;
  {
    LaunchTimer timer(timed);
    e = launch_main(pl, g, stream, &timer);
  }
  const DenseParams& p = pl.p;
  const int shared = p.tiles - p.shared0;
  if (e == hipSuccess && shared > 0 && !(p.extra == 0 && p.per_run % p.upt == 0)) {
    hipLaunchKernelGGL(dense_reduce_kernel, dim3(shared, 2 * pl.TW), dim3(2 * kNT), 0, stream, g.partial, p, 32 * pl.TW,
                       g.bias, g.y);
    e = hipGetLastError();
  }
  return e;
}

size_t up256(size_t b) { return (b + 255) & ~(size_t)255; }

}  // namespace

bool conv_dense_supported(const ConvShape& s) {
  DensePlan pl;
  if (!make_plan(s, &pl)) return false;
  return true;
}

// Where the products are the better way.  `table_chain`: how many table
// entries the layer's table kernel adds up one after the other (0: none can
// tile it but the generic kernel).
//   * Precision: the table kernels' relative error grows with the square root
//     of that chain (9 to 18 entries 1.0e-7, 48 1.1e-7 to 1.3e-7, 72 1.5e-7, 144
//     2.1e-7, 288 3.1e-7), this one's stays at 0.9e-7 to 1.4e-7 from 200 to 5000
//     products: not larger from 48 entries on (0.99 of it there, 0.9 at 50).
//   * Time: the generic table kernel is slower by a factor of 10 or more
//     (256 channels 13 x 13, 3x3, K = 256, 8 images: 1841 us against 28 us).  Against
//     the other two a call has about 6 us more to win back, in a layer of at
//     least 1.5e8 multiply-adds for C's <= 4 (256 -> 384 channels, 3x3 on
//     13 x 13: 26 -> 21 us for one image, 177 -> 84 us for 64) and twice that for
//     C's <= 8, whose table reads do twice the work (512 -> 512 channels, 14 x 14:
//     28 -> 26 us for one, 284 -> 204 us for 64); and a tile has to be long enough
//     for its first and last microseconds: 256 products per output, with
//     64 output channels or fewer 512 (a tile then stages twice the input per
//     product: 32 -> 64 channels on 28 x 28, 64 images: 33 us against 35 us).
//     With fewer than 64 channels most of a tile is padding, and 3x3 kernels of
//     C's = 7 and 8 have the cheapest table: from 1.7e9 padded multiply-adds on
//     (us per call; 64 -> 24 channels, 28 x 28, 55 images, 1.6e9: 33 against 42; 512 ->
//     16, 14 x 14, 22 images, 1.3e9: 33 against 41; 42 images, 2.4e9: 47 against
//     46).
//     A packed kernel row (fewer than 8 input channels) is padded to whole
//     units and stages several rows per output row: from 1e9 multiply-adds on
//     (AlexNet conv1: 38 us against 44 us for 4 images, 71 against 60 us for
//     16, 263 against 182 us for 64).
bool conv_dense_better(const ConvShape& s, int table_chain) {
  if (!conv_dense_supported(s)) return false;
  if (table_chain == 0) return s.M * s.dk * s.dk >= 48;
  return table_chain >= 48 && conv_dense_large(s);
}

// The rule's sizes alone (no plan).
bool conv_dense_large(const ConvShape& s) {
  const int products = s.Cs * s.dk * s.dk;
  const double macs = (double)s.N * s.Ho * s.Wo * s.Ct * products;
  if (s.Csp > 6 && s.dk <= 3 && s.Ct < 64 && macs * 64 / s.Ct < 1.7e9) return false;
  return products >= (s.Ct <= 64 ? 512 : 256) && macs >= (s.dk > 1 && s.Cs < 8 ? 1e9 : s.Csp <= 4 ? 1.5e8 : 3e8);
}

size_t conv_dense_workspace(const ConvShape& s) {
  DensePlan pl;
  return make_plan(s, &pl) ? up256(pl.weight_bytes) + pl.partial_bytes : 0;
}

size_t conv_dense_weight_bytes(const ConvShape& s) {
  DensePlan pl;
  return make_plan(s, &pl) ? up256(pl.weight_bytes) : 0;
}

hipError_t launch_conv_dense_weights(const ConvShape& s, const float* D, CodeStream codes, char* w,
                                     hipStream_t stream) {
  DensePlan pl;
  if (!make_plan(s, &pl)) return hipErrorInvalidConfiguration;
  return launch_weights(pl, D, codes, w, stream);
}

DensePlan* conv_dense_plan_new(const ConvShape& s) {
  DensePlan* pl = new (std::nothrow) DensePlan;
  if (pl && !make_plan(s, pl)) {
    delete pl;
    pl = nullptr;
  }
  return pl;
}

void conv_dense_plan_delete(DensePlan* pl) { delete pl; }

hipError_t launch_conv_dense(const ConvShape& s, const float* x, const float* D, CodeStream codes, const char* w,
                             const float* bias, int relu, float* y, hipStream_t stream, const Workspace* ws,
                             const PoolSpec* pool, const DensePlan* plan) {
  DensePlan pl;
  if (plan)
    pl = *plan;
  else if (!make_plan(s, &pl))
    return hipErrorInvalidConfiguration;
  pl.p.relu = relu;
  const size_t wb = w ? 0 : up256(pl.weight_bytes), pb = up256(pl.partial_bytes);
  const size_t full = pool ? (size_t)s.N * s.Ct * s.Ho * s.Wo * sizeof(float) : 0;
  Scratch scratch;
  hipError_t e = scratch.take(stream, wb + pb + full, ws);
  if (e != hipSuccess) return e;
  char* base = scratch.get();
  if (!w) {
    e = launch_weights(pl, D, codes, base, stream);
    if (e != hipSuccess) return e;
    w = base;
  }
  float* ymap = pool ? reinterpret_cast<float*>(base + wb + pb) : y;
  const Ptrs g{x, w, bias, ymap, reinterpret_cast<float*>(base + wb)};
  e = run_dense(pl, g, stream, ws == nullptr || ws->timed);
  if (e != hipSuccess || !pool) return e;
  return launch_maxpool(ymap, s.N, s.Ct, s.Ho, s.Wo, pool->k, pool->s, pool->Hp, pool->Wp, y, stream);
}

}  // namespace qcnn
