// Float matrix products on the CDNA4 matrix cores, any shape and alignment.  They carry the float mode.
//
//   op 0  C[M,N]  = A[M,K] B[N,K]^T (+R)   A, B k-contiguous
//   op 1  C[M,N]  = A[M,K] B[K,N]          B k-strided
//   op 2  C[M,N] += A[K,M]^T B[K,N]        both k-strided; added atomically
//
// On the bf16 instruction (v_mfma_f32_16x16x32_bf16, 16 times the rate of the float one): a float is the sum of three
// bfloat16s, exactly (8 + 8 + 8 bits), and a product of two floats the sum of nine products of those, each exact.  Six are
// formed; the three left out (middle x low, low x middle, low x low) are below 2^-24 of the product, less than its rounding
// to a float.  Sums are floats as with the float instruction, and fewer: its error against 64 bits (2-norm, unit normals; the
// float instruction over the same runs of 64 k / this) 1.45e-7 / 1.00e-7 at K = 288, 1.58 / 1.17 at 768, 1.73 / 1.36 at
// 1536, 2.04 / 1.80 at 4096, 2.83 / 2.70 at 11264.  Leaving out nothing changes no digit of these.  Parts below the smallest
// bfloat16 are lost: an operand below 2^-110 (8e-34) keeps an absolute error of up to 2^-134.
//
// For ops 0 and 1 the tile of B is the instruction's row operand, so a lane ends with four consecutive output columns of
// one row (16-byte stores, and whole rotary pairs for the epilogue); for op 2 the tile of A is, so that a wavefront's atomics
// cover 64 contiguous bytes of four rows.
//
// What bounds it: the split.  A tile's operands are split once per tile, 5.5 vector instructions a value, and beside matrix
// instructions that keep their core busy a SIMD issues another vector instruction every 6.5 cycles; LDS holds 6 bytes a value.
// A step (32 k) of a 128-tile takes 2700 cycles: 1580 of matrix instructions on every SIMD, 1500 of the split's issue, 1570 of
// LDS.  Tried for it and not better: every wavefront splitting and multiplying in turn (3800 cycles: a wavefront's own
// matrix instruction hides 1.5 vector ones, another's 2.5), the leading part taken off by v_dot2_f32_bf16 (half the
// instructions, each 9 cycles beside matrix instructions), the stages of several quads interleaved.
// us per launch, float instruction (two thirds of its 157 TFLOP/s) -> this: op 0 2048 x 1024 x 1024 43 -> 30, 2048 x 3072 x 1024
// 131 -> 74, 2048 x 1024 x 5632 220 -> 140, 4096 x 4096 x 4096 1135 -> 657 (209 TFLOP/s), op 1 2048 x 1024 x 5632 235 -> 145, op 2
// 1024 x 1024 x 2048 61 -> 39, 3072 x 1024 x 2048 123 -> 81, 5632 x 1024 x 2048 237 -> 147; small ones even: op 0 1024 x 288 x 1536
// 22 -> 20.  The stage of the 500M shape on 2 x 2 x 512 tokens 7.18 -> 5.09 ms, the 50M shape on 4 x 4 x
// 256 tokens 5.60 -> 4.93 ms a pass.
//
// Every entry is summed in one order (runs of 64 k), with the same instructions, whatever the tile: that follows the
// number of rows, and a microbatch's rows must not depend on how many microbatches share its group; a weight gradient is
// added with one atomic per entry and launch, so that it repeats to the bit.
#include <type_traits>

#include "devutil.h"
#include "internal.h"

namespace sp {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;

constexpr int BK = 32;
constexpr int kThreads = 512;

// Runs of 64 k are summed from zero and added up in turn: with one chain over the whole reduction the error grows with its
// length (4.2e-7 at K = 768, 1.0e-6 at 4096).  It takes one more set of accumulators.
// The instruction rounds the sum of its products towards minus infinity, so that all entries are off in one direction (the mean
// of the errors at K = 1536 is 3.5e-8 of an entry, four times what chance leaves; through a model's residual additions
// such errors add up, not their squares).  So every second run is formed of the negated A, and subtracted.  Gradients of whole models
// against 64 bits, float instruction / this / this without the negation: 50M widths, 2 x 256 tokens 6.3e-7 / 5.8e-7 / 9.0e-7, 500M
// widths, 2 x 128 tokens 8.3e-7 / 7.0e-7 / 12.4e-7.
constexpr int kRun = 64 / BK;   // steps
enum { kEpiPlain = 0, kEpiRope = 1, kEpiSwiglu = 2, kEpiSwigluBwd = 3 };   // as in the bf16 kernels

struct Args {
  const float *A, *B, *R;
  float *C, *aux;
  int M, N, K, tiles_m, tiles_n;
  RopeArgs rope;
};

// element t of a fragment quad; VEC: the four are one aligned 16-byte access and all inside or all outside
template <bool VEC>
__device__ __forceinline__ f32x4 load4(const float* p, int valid) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (VEC) {
    if (valid > 0) v = *reinterpret_cast<const f32x4*>(p);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < valid) v[e] = p[e];
  }
  return v;
}

template <bool VEC>
__device__ __forceinline__ void store4(float* p, const f32x4& v, int valid) {
  if (VEC) {
    if (valid > 0) *reinterpret_cast<f32x4*>(p) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (e < valid) p[e] = v[e];
  }
}

__device__ __forceinline__ bool finite(float v) { return fabsf(v) <= __FLT_MAX__; }

// Four consecutive output columns n .. n+3 of row m leave for memory (ops 0 and 1).
template <int OP, int EPI, bool VEC>
__device__ __forceinline__ void emit(const Args& g, int m, int n, f32x4 v) {
  const int left = g.N - n;
  const int64_t at = (int64_t)m * g.N + n;
  if (EPI == kEpiSwigluBwd) {   // v = d(act); R = gate | up (rows of 2 N), C = d(gate) | d(up)
    const int64_t a2 = (int64_t)m * 2 * g.N + n;
    const f32x4 gt = load4<VEC>(g.R + a2, left), up = load4<VEC>(g.R + a2 + g.N, left);
    f32x4 og, ou;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float sg = 1.0f / (1.0f + expf(-gt[e]));
      og[e] = v[e] * up[e] * sg * (1.0f + gt[e] * (1.0f - sg));
      ou[e] = v[e] * gt[e] * sg;
    }
    store4<VEC>(g.C + a2, og, left);
    store4<VEC>(g.C + a2 + g.N, ou, left);
    return;
  }
  if (EPI == kEpiRope) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {   // a pair never straddles the end of the rotated columns: their number is even
      const int c = n + 2 * p;
      if (c < g.rope.rot_cols) {
        const float2 cs = reinterpret_cast<const float2*>(g.rope.table)[(int64_t)(m % g.rope.T) * (g.rope.hd / 2) + (c % g.rope.hd) / 2];
        const float a = v[2 * p], b = v[2 * p + 1];
        v[2 * p] = a * cs.x - b * cs.y;
        v[2 * p + 1] = a * cs.y + b * cs.x;
      }
    }
  }
  if (OP == 0 && EPI == kEpiPlain && g.R) v += load4<VEC>(g.R + at, left);
  store4<VEC>(g.C + at, v, left);
}

// gate and up of four consecutive features f .. f+3 of row m
template <bool VEC>
__device__ __forceinline__ void emit_swiglu(const Args& g, int m, int f, const f32x4& gt, const f32x4& up) {
  const int h = g.N / 2, left = h - f;
  f32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = gt[e] / (1.0f + expf(-gt[e])) * up[e];
  store4<VEC>(g.C + (int64_t)m * g.N + f, gt, left);
  store4<VEC>(g.C + (int64_t)m * g.N + h + f, up, left);
  store4<VEC>(g.aux + (int64_t)m * h + f, o, left);
}

// Ids that land on one XCD (id mod 8) get neighbouring tiles; tiles run down M inside bands of 8 tile columns.
__device__ __forceinline__ void tile_of(const Args& g, int id, int& tm, int& tn) {
  constexpr int kBand = 8;
  const int band = id / (kBand * g.tiles_m), band_w = min(kBand, g.tiles_n - band * kBand), in = id - band * kBand * g.tiles_m;
  tm = in / band_w;
  tn = band * kBand + in % band_w;
}
__device__ __forceinline__ int xcd_major(int id, int n) {
  const int per = n / 8, rem = n % 8, x = id % 8;
  return x * per + min(x, rem) + id / 8;
}

// ---- three-way split, x = h + m + l
__device__ __forceinline__ uint32_t lead2(float x0, float x1) {   // two values' nearest bfloat16s, one instruction
  typedef __attribute__((ext_vector_type(2))) float f2;
  typedef __attribute__((ext_vector_type(2))) __bf16 b2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{x0, x1}, b2));
}
struct Split { uint2 h, m, l; };   // four values' parts, in order
__device__ __forceinline__ uint32_t rest2(float& x0, float& x1) {   // lead2, leaving what is left of the values
  const uint32_t p = lead2(x0, x1);
  x0 -= bf16_bits_to_float(p & 0xffffu);
  x1 -= __uint_as_float(p & 0xffff0000u);
  return p;
}
__device__ __forceinline__ Split split4(float a, float b, float c, float d) {
  Split s;
  s.h.x = rest2(a, b); s.h.y = rest2(c, d);
  s.m.x = rest2(a, b); s.m.y = rest2(c, d);
  s.l = make_uint2(lead2(a, b), lead2(c, d));
  return s;
}

// An operand's tile of T rows (columns of a k-strided operand) x BK in LDS: three planes [T][BK] of parts, 64 bytes a row,
// unpadded.  Row r lies at position r / 4 + (r % 4) T / 4 and its 16-byte chunks are permuted by r % 4, so that the 16 rows of
// a fragment read and the four rows of 32 k that half a wavefront writes of a k-contiguous operand each fall in all 64 banks (no
// conflict is counted in op 0).  The 4 k x columns that it writes of a k-strided one do not: 4 conflict cycles a store of 512 bytes,
// as many as it takes without them, are counted in ops 1 (B) and 2 (A and B).
template <int T>
struct Planes {
  static constexpr int kPlane = T * BK * 2, kBytes = 3 * kPlane;
  static __device__ __forceinline__ int at(int row, int chunk) { return ((row >> 2) + (row & 3) * (T / 4)) * 64 + ((chunk ^ (row & 3)) << 4); }
};
struct Frag { bf16x8 p[3]; };   // h, m, l of row base + lane % 16, k = (lane / 16) * 8 .. + 7; base a multiple of 16
template <int T>
__device__ __forceinline__ Frag frag(const char* lds, int base, int lane_at) {   // lane_at: of row lane % 16
  Frag f;
#pragma unroll
  for (int i = 0; i < 3; ++i) f.p[i] = *reinterpret_cast<const bf16x8*>(lds + i * Planes<T>::kPlane + base * 16 + lane_at);
  return f;
}
// acc += X Y without the three smallest products (below 2^-24 of a product), the smallest first
constexpr int kTerms = 6;
constexpr int kTermX[kTerms] = {2, 0, 1, 1, 0, 0}, kTermY[kTerms] = {0, 2, 1, 0, 1, 0};

// The parts of a value that is not finite, or rounds past the largest bfloat16, are infinities and NaN.  Entries of the blocks of
// 16 x 16 in `sum` that come out as either are formed anew from the floats themselves, on the float instruction and in the same
// runs (k-slots may stand for any k: a lane takes four neighbours of every 16).  NaN stays NaN: a block whose entries all
// have come to that is done, so that a pass through which it has spread costs about one run a block.  us, op 0 / 1 / 2, 4096 x
// 1024 x 2816: finite 130 / 119 / 118, NaN throughout 126 / 131 / 150, NaN in the last k alone or an infinity in every row 1080 /
// 1570 / 1820, an infinity in one row 343 / 461 / 530.  (The loads of a whole run at once, 720 / 1130 / 1470, took 25 registers
// more, and with them a workgroup of 128 x 64.)
// row_m(j), row_n(i): lane's row of A and row (column) of B in block (j, i).
template <int OP, bool VEC, int NA, int NB, class RowM, class RowN>
__device__ __forceinline__ void mend(const Args& g, f32x4 (&sum)[NA][NB], RowM row_m, RowN row_n, int kg) {
  constexpr bool AS = OP == 2, BS = OP != 0;
  uint32_t todo = 0;
#pragma unroll
  for (int j = 0; j < NA; ++j)
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      const f32x4 v = sum[j][i];
      if (__ballot(!(finite(v[0]) && finite(v[1]) && finite(v[2]) && finite(v[3])))) todo |= 1u << (j * NB + i);
    }
  const int K = g.K;
  while (todo) {
    const int blk = __builtin_ctz(todo);
    todo &= todo - 1;
    const int m = row_m(blk / NB), n = row_n(blk % NB);
    f32x4 v, c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (blk == j * NB + i) v = sum[j][i];
    // the block's first row (column) is uniform; a lane's place in it
    const int m_first = __builtin_amdgcn_readfirstlane(m), n_first = __builtin_amdgcn_readfirstlane(n);
    const float* pa = g.A + (AS ? (int64_t)m_first : (int64_t)m_first * K);
    const float* pb = g.B + (BS ? (int64_t)n_first : (int64_t)n_first * K);
    typedef std::conditional_t<AS, uint32_t, int64_t> LA;   // 15 columns, or 15 rows
    typedef std::conditional_t<BS, uint32_t, int64_t> LB;
    const LA la = AS ? (LA)(m - m_first) : (LA)(m - m_first) * K;
    const LB lb = BS ? (LB)(n - n_first) : (LB)(n - n_first) * K;
    for (int k0 = 0; k0 < K; k0 += kRun * BK) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int h = k0; h < k0 + kRun * BK; h += 16) {
        f32x4 a, b;
        const int k = h + kg * 4;
        if (AS) {
#pragma unroll
          for (int e = 0; e < 4; ++e) a[e] = k + e < K ? pa[(int64_t)(k + e) * g.M + la] : 0.f;
        } else a = load4<VEC>(pa + la + k, K - k);
        if (BS) {
#pragma unroll
          for (int e = 0; e < 4; ++e) b[e] = k + e < K ? pb[(int64_t)(k + e) * g.N + lb] : 0.f;
        } else b = load4<VEC>(pb + lb + k, K - k);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = OP == 2 ? __builtin_amdgcn_mfma_f32_16x16x4f32(a[e], b[e], acc, 0, 0, 0) : __builtin_amdgcn_mfma_f32_16x16x4f32(b[e], a[e], acc, 0, 0, 0);
      }
      c += acc;
      bool open = false;
#pragma unroll
      for (int r = 0; r < 4; ++r) open = open || (!finite(v[r]) && c[r] == c[r]);
      if (!__ballot(open)) break;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = finite(v[r]) ? v[r] : c[r];
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int i = 0; i < NB; ++i)
        if (blk == j * NB + i) sum[j][i] = v;
  }
}

// How a product's operands are reached.  kAligned: pointers and widths are multiples of 16 bytes / 4.  kUnaligned: buffer loads
// need 4-byte alignment only, so all is loaded alike; what crosses the end of the matrix is loaded again one by one.  kFar: a
// tile reaches further than 31 bits (gemm_f32_far): one by one from pointers.
// us, one by one from pointers (as all that are not aligned were; float instruction before that) / this: op 0 1024 x 1023 x 1021 58
// (41) / 21, 4096 x 2050 x 515 152 (186) / 78, op 1 2048 x 287 x 289 20 (16) / 9.2, op 2 1024 x 1023 x 1021 70 (48) / 24, 999 x 1024 x
// 5632 474 (234) / 89 (aligned, 1024: 88).
enum { kFar = 0, kUnaligned = 1, kAligned = 2 };

// The share of one of NW wavefronts in bringing an operand's tile from memory to LDS: units of a row's 4 consecutive k
// (k-contiguous) or of 4 k of XW neighbouring columns (k-strided).
// Buffer loads from a descriptor that starts at the step, so that a lane's offsets are the same for all steps and k past
// the end of a k-strided operand reads as zeros.  Rows (columns) past the edge are read as the last one (k-strided: as
// what follows); nothing of them is stored.
template <bool KS, int T, int NW, int ACC>
struct Share {
  static constexpr int Q = T / (8 * NW);                          // quads of 4 k
  static constexpr int XW = KS ? (Q < 4 ? Q : 4) : 1, NU = Q / XW;
  const char* base;      // the first byte that the tile can reach, and how many follow it
  int64_t left;
  uint32_t off[NU];
  const float* p[NU];    // kFar: a unit's row or first column, and where its other columns are
  int dx[NU][3], row[NU], lds[NU], k;
  template <class RowOf>
  __device__ __forceinline__ void init(const float* X, int ld, int x0, int cols, int K, int wave, int lane, RowOf row_of) {
    const int64_t first = KS ? (int64_t)x0 : (int64_t)x0 * ld;
    base = reinterpret_cast<const char*>(X + first);
    left = ((int64_t)(KS ? K : cols) * ld - first) * 4;
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      if (KS) {   // a wavefront: 8 x 4 k by 8 groups of XW columns
        row[u] = ((wave + NW * u) * 8 + (XW == 4 ? (lane & 3) + (lane >> 5) * 4 : lane & 7)) * XW;
        k = (XW == 4 ? (lane >> 2) & 7 : lane >> 3) * 4;
        off[u] = ((uint32_t)k * (uint32_t)ld + row[u]) * 4u;
        const int c = min(x0 + row[u], cols - 1);
        p[u] = X + c;
#pragma unroll
        for (int e = 1; e < 4; ++e) dx[u][e - 1] = min(x0 + row[u] + e, cols - 1) - c;
      } else {    // 8 rows of 32 k, four apart and neighbours; two wavefronts take 16 rows
        row[u] = (NW == 1 ? 2 * u : ((wave >> 1) + NW / 2 * u) * 16 + (wave & 1) * 2) + ((lane >> 3) & 3) * 4 + (lane >> 5);
        k = (lane & 7) * 4;
        const int r = row_of(row[u]);
        off[u] = ((uint32_t)(r - x0) * (uint32_t)ld + k) * 4u;
        p[u] = X + (int64_t)r * ld;
      }
      lds[u] = Planes<T>::at(row[u], k >> 3) + (k & 4) * 2;
    }
  }
  // v[q]: quad q = unit * XW + column
  __device__ __forceinline__ void load(float (*v)[4], int k0, int K, int ld) const {
    if constexpr (ACC == kFar) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int c = 0; c < XW; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int at = min(k0 + k + e, K - 1);
            const float x = KS ? p[u][(int64_t)at * ld + (c ? dx[u][c ? c - 1 : 0] : 0)] : p[u][at];
            v[u * XW + c][e] = k0 + k + e < K ? x : 0.f;
          }
    } else {
      const rsrc_t rs = make_rsrc(base + (int64_t)k0 * (KS ? ld : 1) * 4, bytes(k0, ld));
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        if constexpr (KS) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int o = (int)(off[u] + (uint32_t)e * (uint32_t)ld * 4u);
            if constexpr (XW == 4) {
              const f32x4 x = __builtin_bit_cast(f32x4, buffer_load16(rs, o));
#pragma unroll
              for (int c = 0; c < 4; ++c) v[u * XW + c][e] = x[c];
            } else if constexpr (XW == 2) {
              const float2 x = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rs, o, 0, 0));
              v[u * XW][e] = x.x; v[u * XW + 1][e] = x.y;
            } else {
              v[u][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, o, 0, 0));
            }
          }
        } else {
          const f32x4 x = __builtin_bit_cast(f32x4, buffer_load16(rs, off[u]));
#pragma unroll
          for (int e = 0; e < 4; ++e) v[u][e] = x[e];
        }
      }
    }
  }
  __device__ __forceinline__ uint32_t bytes(int k0, int ld) const {   // from step k0 to the end of the matrix, as the descriptor holds it
    const int64_t rest = left - (int64_t)k0 * (KS ? ld : 1) * 4;
    return (uint32_t)(rest > 0x7fffffff ? 0x7fffffff : rest);
  }
  // is there something to finish in step k0 or before it (a load of four from the third row before the last may cross the end: rows
  // of one float)
  static __device__ __forceinline__ bool unfinished(int k0, int K) { return ACC != kFar && k0 + BK + (ACC == kUnaligned ? 3 : 0) > K; }
  // What load() brought of the last steps, made right before it is used (a choice at the load instead keeps the compiler from
  // leaving loads in flight: 1.05 to 1.2 x).  A load of several floats that crosses the end of the matrix: one by one.  k past the
  // end become zeros, in both operands: what a k-contiguous one holds there are the first values of its next row, and if those
  // are not finite, zeros in the other operand alone would leave NaN in this row.
  __device__ __forceinline__ void finish(float (*v)[4], int k0, int K, int ld) const {
    if (!unfinished(k0, K)) return;
    if constexpr (ACC == kUnaligned && (!KS || XW > 1)) {
      const uint32_t end = bytes(k0, ld);
      bool crosses = false;
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < (KS ? 4 : 1); ++e) {
          const uint32_t o = off[u] + (uint32_t)e * (uint32_t)ld * 4u;
          crosses = crosses || (o < end && o + (KS ? XW : 4) * 4 > end);
        }
      if (__ballot(crosses)) {
        const rsrc_t rs = make_rsrc(base + (int64_t)k0 * (KS ? ld : 1) * 4, end);
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
          for (int c = 0; c < XW; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              v[u * XW + c][e] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)(off[u] + (KS ? (uint32_t)e * (uint32_t)ld + c : e) * 4u), 0, 0));
      }
    }
    if (!KS) {
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) v[u][e] = k0 + k + e < K ? v[u][e] : 0.f;
    }
  }
  template <bool NEG>   // negated (a modifier of the split's instructions)
  __device__ __forceinline__ void put(char* tile, float (*v)[4]) const {
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const Split s = NEG ? split4(-v[q][0], -v[q][1], -v[q][2], -v[q][3]) : split4(v[q][0], v[q][1], v[q][2], v[q][3]);
      char* p = tile + (q % XW ? Planes<T>::at(row[q / XW] + q % XW, k >> 3) + (k & 4) * 2 : lds[q / XW]);
      *reinterpret_cast<uint2*>(p) = s.h;
      *reinterpret_cast<uint2*>(p + Planes<T>::kPlane) = s.m;
      *reinterpret_cast<uint2*>(p + 2 * Planes<T>::kPlane) = s.l;
    }
  }
};

// The feeding wavefronts' work: a step per barrier into the buffer that the multiplying ones have left; loads U steps ahead.
// fetch(step, quads) and put(step, quads): all of the wavefront's quads of a step; finish(step, quads) before it in the last two.
template <int Q, class Fetch, class Finish, class Put>
__device__ __forceinline__ void feed(int steps, Fetch fetch, Finish finish, Put put) {
  constexpr int U = Q > 6 ? 2 : Q > 4 ? 3 : Q > 3 ? 4 : 6;
  float raw[U][Q][4];
  auto load = [&](int s, int u) {   // past the last step the last one again
    fetch(min(s, steps - 1), raw[u]);
    __builtin_amdgcn_sched_barrier(0);   // loads stay in the order they are waited for
  };
#pragma unroll
  for (int u = 0; u < U; ++u) load(u, u);
  int s = 0;
  for (; s + U + 2 <= steps; s += U)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      put(s + u, raw[u]);
      load(s + u + U, u);
      __syncthreads();
    }
  for (; s < steps; s += U)
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (s + u < steps) {
        finish(s + u, raw[u]);
        put(s + u, raw[u]);
        load(s + u + U, u);
        __syncthreads();
      }
}

// Tiles of TM x TN, eight wavefronts (or twelve), a barrier per step.  The first four (a share of TM / 2 x TN / 2 each) only read fragments
// and multiply, the others only bring the operands of the next step to LDS, split on the way, U steps of loads in flight: a
// SIMD holds one of either, and beside the matrix instructions of one wavefront (16 cycles each) another can issue 2.5
// others, where one that does both gets 1.5 for nothing.
// FEED of them bring operands.  What a 32-tile takes alone on its CU is the chain of a feeding wavefront's instructions (70 a step), and
// eight that have half of it each are faster while two such workgroups are all that a CU gets (three of four feeding ones fit): op 2
// 828 x 152 x 3768 (130 tiles) 39 -> 31 us, 288 x 768 x 4096 (216) 42 -> 32, by tiles a CU (op 0 / 1 / 2) one 0.79 / 0.81 / 0.78 times, two 0.91 / 0.94 / 0.90, three 1.05 /
// 1.06 / 1.02.
constexpr int kFeed = 4, kFeedFew = 8;
template <int TN, int FEED> constexpr int kTileThreads = TN == 16 ? kThreads : 64 * (4 + FEED);
// wg of n_wgs: the workgroup's number among those of the product
template <int OP, int EPI, int TM, int TN, int ACC, int FEED>
__device__ __forceinline__ void gemm_tile(const Args& g, int wg, int n_wgs) {
  constexpr bool AS = OP == 2, BS = OP != 0;
  // SwiGLU in 32-tiles: a wavefront holds 16 gate columns and the 16 up columns, so the tile of B has 64 rows
  constexpr int NSEG = EPI == kEpiSwiglu && TN == 32 ? 2 : 1, TB = TN * NSEG;
  constexpr int WM = TM / 2, WN = TN / 2, NA = WM / 16, NB = WN / 16 * NSEG;   // a wavefront's share, in blocks of 16
  constexpr int kBuf = Planes<TM>::kBytes + Planes<TB>::kBytes;
  __shared__ __attribute__((aligned(16))) char smem[2 * kBuf];
  const int lane = threadIdx.x & 63, lr = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tm, tn;
  tile_of(g, xcd_major(wg, n_wgs), tm, tn);
  const int m0 = tm * TM, n0 = tn * TN, K = g.K, steps = (K + BK - 1) / BK, lda = AS ? g.M : K, ldb = BS ? g.N : K;
  const int b0 = EPI == kEpiSwiglu && NSEG == 1 ? n0 / 2 : n0;   // the tile's first row (column) of B
  // memory row of the tile's row t of B (k-contiguous).  SwiGLU: a wavefront's share holds gate rows and the up rows of the
  // same features (h = N / 2 of them)
  auto b_row = [&](int t) {
    if (EPI != kEpiSwiglu) return min(n0 + t, g.N - 1);
    const int h = g.N / 2;
    if (NSEG == 2) return (t & 16 ? h : 0) + min(b0 + (t >> 5) * 16 + (t & 15), h - 1);
    const int w = t / WN, in = t % WN, f = b0 + w * (WN / 2) + in % (WN / 2);
    return (in < WN / 2 ? 0 : h) + min(f, h - 1);
  };
  if (wave >= 4) {
    if (steps == 0) return;
    auto a_row = [&](int t) { return min(m0 + t, g.M - 1); };
    auto buf = [&](int s) { return smem + (s & 1) * kBuf; };
    auto put_a = [&](const auto& a, int s, float (*v)[4]) {   // every second run negated (kRun)
      if (s & kRun) a.template put<true>(buf(s), v);
      else a.template put<false>(buf(s), v);
    };
    auto put_b = [&](const auto& b, int s, float (*v)[4]) { b.template put<false>(buf(s) + Planes<TM>::kBytes, v); };
    // Tiles of the same size: half of the wavefronts for each operand (wider loads); else all for both.
    constexpr int NW = FEED / 2;
    if constexpr (TM == TB) {
      if (wave < 4 + NW) {
        Share<AS, TM, NW, ACC> a;
        a.init(g.A, lda, m0, g.M, K, wave - 4, lane, a_row);
        feed<a.Q>(steps, [&](int s, float (*v)[4]) { a.load(v, s * BK, K, lda); }, [&](int s, float (*v)[4]) { a.finish(v, s * BK, K, lda); },
                  [&](int s, float (*v)[4]) { put_a(a, s, v); });
      } else {
        Share<BS, TB, NW, ACC> b;
        b.init(g.B, ldb, b0, g.N, K, wave - 4 - NW, lane, b_row);
        feed<b.Q>(steps, [&](int s, float (*v)[4]) { b.load(v, s * BK, K, ldb); }, [&](int s, float (*v)[4]) { b.finish(v, s * BK, K, ldb); },
                  [&](int s, float (*v)[4]) { put_b(b, s, v); });
      }
    } else {
      Share<AS, TM, 4, ACC> a;
      Share<BS, TB, 4, ACC> b;
      a.init(g.A, lda, m0, g.M, K, wave - 4, lane, a_row);
      b.init(g.B, ldb, b0, g.N, K, wave - 4, lane, b_row);
      feed<a.Q + b.Q>(
          steps,
          [&](int s, float (*v)[4]) {
            a.load(v, s * BK, K, lda);
            b.load(v + a.Q, s * BK, K, ldb);
          },
          [&](int s, float (*v)[4]) {
            a.finish(v, s * BK, K, lda);
            b.finish(v + a.Q, s * BK, K, ldb);
          },
          [&](int s, float (*v)[4]) {
            put_a(a, s, v);
            put_b(b, s, v + a.Q);
          });
    }
    return;
  }
  const int wm = wave >> 1, wn = wave & 1, base_a = wm * WM, base_b = wn * WN * NSEG;
  f32x4 acc[NA][NB], sum[NA][NB];
#pragma unroll
  for (int j = 0; j < NA; ++j)
#pragma unroll
    for (int i = 0; i < NB; ++i) acc[j][i] = sum[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int at_a = Planes<TM>::at(lr, kg), at_b = Planes<TB>::at(lr, kg);
  Frag fa[2], fb[NB];
  auto read_a = [&](int s, int j) { return frag<TM>(smem + (s & 1) * kBuf, base_a + j * 16, at_a); };
  auto read_b = [&](int s, int i) { return frag<TB>(smem + (s & 1) * kBuf + Planes<TM>::kBytes, base_b + i * 16, at_b); };
  // blocks i0 .. i1 - 1 of row j of blocks
  auto multiply = [&](int j, int i0, int i1, const Frag& a, auto begins) {
#pragma unroll
    for (int t = 0; t < kTerms; ++t)
#pragma unroll
      for (int i = i0; i < i1; ++i) {
        const f32x4 c = decltype(begins)::value && t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[j][i];
        // ops 0 and 1: B is the instruction's row operand (X), A its column operand; op 2: the other way round
        acc[j][i] = OP == 2 ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(a.p[kTermX[t]], fb[i].p[kTermY[t]], c, 0, 0, 0)
                            : __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[i].p[kTermX[t]], a.p[kTermY[t]], c, 0, 0, 0);
      }
  };
  if (steps > 0) {
    __syncthreads();   // step 0 is in LDS
#pragma unroll
    for (int i = 0; i < NB; ++i) fb[i] = read_b(0, i);
    fa[0] = read_a(0, 0);
    // The fragments of a row of blocks are read while the row before it is multiplied.  All of a step's are read by its
    // last row: there the barrier stands, and behind it the next step's are read as registers come free, half a row of
    // blocks before they are used.  A row's sums of a run are added up while the next row is multiplied.
    constexpr int H = NB == 1 ? 1 : NB / 2;   // blocks of half a row
    auto add_up = [&](int j, float sign) {
#pragma unroll
      for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[j][i][r] = __builtin_fmaf(acc[j][i][r], sign, sum[j][i][r]);
    };
    auto step = [&](int s, auto begins, auto par) {   // par: which of fa holds the step's first row
      constexpr int P = decltype(par)::value;
      constexpr bool first = decltype(begins)::value;
      const bool more = s + 1 < steps;
      const float sign = s & kRun ? -1.f : 1.f;
#pragma unroll
      for (int j = 0; j < NA; ++j) {
        if (j + 1 < NA) fa[(P + j + 1) & 1] = read_a(s, j + 1);
        else if (more) {
          __syncthreads();
          fa[(P + NA) & 1] = read_a(s + 1, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NB; i += H) {
          multiply(j, i, i + H, fa[(P + j) & 1], begins);
          if (i == 0 && NA > 1) {
            if (j > 0 && !first) add_up(j - 1, sign);
            if (j == 0 && first) add_up(NA - 1, -sign);   // of the run before (zeros in the first)
          }
          __builtin_amdgcn_sched_barrier(0);
          if (j == NA - 1 && more)
#pragma unroll
            for (int e = 0; e < H; ++e) fb[i + e] = read_b(s + 1, i + e);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (NA == 1 && !first) add_up(0, sign);
    };
    static_assert(kRun == 2, "a step that begins a run and one that ends it");
    constexpr int odd = NA & 1;   // an odd number of rows: the next step starts in the other of fa
    for (int s = 0; s < steps; s += 2) {
      step(s, std::true_type(), std::integral_constant<int, 0>());
      if (s + 1 < steps) step(s + 1, std::false_type(), std::integral_constant<int, odd>());
    }
    // what the loop left: a run of one step, and the last row of one of two
    if (steps & 1)
#pragma unroll
      for (int j = 0; j < NA; ++j) add_up(j, (steps - 1) & kRun ? -1.f : 1.f);
    else if (NA > 1) add_up(NA - 1, (steps - 1) & kRun ? -1.f : 1.f);
  }
  mend<OP, ACC == kAligned>(g, sum, [&](int j) { return min(m0 + base_a + j * 16 + lr, g.M - 1); },
                [&](int i) { return BS ? min(n0 + base_b + i * 16 + lr, g.N - 1) : b_row(base_b + i * 16 + lr); }, kg);
  if (OP == 2) {
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int n = n0 + base_b + i * 16 + lr;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + base_a + j * 16 + kg * 4 + r;
          if (m < g.M && n < g.N) unsafeAtomicAdd(g.C + (int64_t)m * g.N + n, sum[j][i][r]);
        }
      }
    return;
  }
#pragma unroll
  for (int j = 0; j < NA; ++j) {
    const int m = m0 + base_a + j * 16 + lr;
    if (m >= g.M) continue;
    if (EPI == kEpiSwiglu) {
      const int f0 = b0 + wn * (NSEG == 2 ? 16 : WN / 2);   // the share's first feature
#pragma unroll
      for (int i = 0; i < NB / 2; ++i) emit_swiglu<ACC == kAligned>(g, m, f0 + i * 16 + kg * 4, sum[j][i], sum[j][i + NB / 2]);
    } else {
#pragma unroll
      for (int i = 0; i < NB; ++i) emit<OP, EPI, ACC == kAligned>(g, m, n0 + base_b + i * 16 + kg * 4, sum[j][i]);
    }
  }
}

// Lanes of one wavefront exchange values through LDS, whose operations of one wavefront are in order: no instruction, but the
// compiler, which keeps the order of one lane's accesses only, has to leave them on their sides of this.
__device__ __forceinline__ void exchange() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// For products too small to fill the chip, where the time is one chain of latencies: tiles of 16 x 16 (SwiGLU: rows x
// features), eight wavefronts that each form whole runs of 64 k, in turn, from loads and splits of their own (no barrier:
// exchange() above), the next run's loads on their way.  After every eight runs the first
// wavefront adds them up in order, so that entries have the bits that the other tiles give them.
template <int OP, int EPI, int ACC>
__device__ __forceinline__ void gemm_few(const Args& g, int wg, int n_wgs) {
  constexpr bool AS = OP == 2, BS = OP != 0;
  constexpr int NB = EPI == kEpiSwiglu ? 2 : 1, NW = kThreads / 64;
  typedef Share<AS, 16, 1, ACC> SA;
  typedef Share<BS, 16, 1, ACC> SB;
  constexpr int kTile = Planes<16>::kBytes;
  __shared__ __attribute__((aligned(16))) char tiles[NW][(1 + NB) * kTile];
  __shared__ __attribute__((aligned(16))) f32x4 found[2][NW][NB][64];
  const int lane = threadIdx.x & 63, lr = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int tm, tn;
  tile_of(g, xcd_major(wg, n_wgs), tm, tn);
  const int m0 = tm * 16, n0 = tn * 16, K = g.K, steps = (K + BK - 1) / BK, runs = (steps + kRun - 1) / kRun;
  const int cols = NB == 2 ? g.N / 2 : g.N, lda = AS ? g.M : K, ldb = BS ? g.N : K;
  f32x4 sums[1][NB];
  f32x4 (&sum)[NB] = sums[0];
#pragma unroll
  for (int i = 0; i < NB; ++i) sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (runs > 0) {
    SA a;
    SB b[NB];
    a.init(g.A, lda, m0, g.M, K, 0, lane, [&](int t) { return min(m0 + t, g.M - 1); });
#pragma unroll
    for (int i = 0; i < NB; ++i) b[i].init(g.B, ldb, i * cols + n0, NB == 2 ? 2 * cols : cols, K, 0, lane, [&](int t) { return i * cols + min(n0 + t, cols - 1); });
    float ra[kRun][SA::Q][4], rb[kRun][NB][SB::Q][4];
    char* const mine = tiles[wave];
    const int at = Planes<16>::at(lr, kg);
    auto load = [&](int run) {   // past the end: the last step again
#pragma unroll
      for (int e = 0; e < kRun; ++e) {
        const int k0 = min(run * kRun + e, steps - 1) * BK;
        a.load(ra[e], k0, K, lda);
#pragma unroll
        for (int i = 0; i < NB; ++i) b[i].load(rb[e][i], k0, K, ldb);
      }
    };
    auto form = [&](auto ends) {   // ends: the last step has something to finish (a branch for it takes 1.07 x)
      load(wave);
      for (int r0 = 0, par = 0; r0 < runs; r0 += NW, par ^= 1) {
        const int run = r0 + wave;
        if (run < runs) {
          f32x4 acc[NB];
          if (decltype(ends)::value && a.unfinished((run + 1) * kRun * BK - BK, K))
#pragma unroll
            for (int e = 0; e < kRun; ++e)
              if (run * kRun + e < steps) {
                a.finish(ra[e], (run * kRun + e) * BK, K, lda);
#pragma unroll
                for (int i = 0; i < NB; ++i) b[i].finish(rb[e][i], (run * kRun + e) * BK, K, ldb);
              }
#pragma unroll
          for (int e = 0; e < kRun; ++e) {
            if (run * kRun + e < steps) {
              if (run & 1) a.template put<true>(mine, ra[e]);
              else a.template put<false>(mine, ra[e]);
#pragma unroll
              for (int i = 0; i < NB; ++i) b[i].template put<false>(mine + (1 + i) * kTile, rb[e][i]);
              exchange();
              const Frag fa = frag<16>(mine, 0, at);
              Frag fb[NB];
#pragma unroll
              for (int i = 0; i < NB; ++i) fb[i] = frag<16>(mine + (1 + i) * kTile, 0, at);
              exchange();   // the next step's values may follow
#pragma unroll
              for (int i = 0; i < NB; ++i) {
#pragma unroll
                for (int t = 0; t < kTerms; ++t) {
                  const f32x4 c = e == 0 && t == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[i];
                  acc[i] = OP == 2 ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa.p[kTermX[t]], fb[i].p[kTermY[t]], c, 0, 0, 0)
                                   : __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[i].p[kTermX[t]], fa.p[kTermY[t]], c, 0, 0, 0);
                }
              }
            }
          }
          if (run + NW < runs) load(run + NW);
#pragma unroll
          for (int i = 0; i < NB; ++i) found[par][wave][i][lane] = acc[i];
        }
        __syncthreads();   // the other half of `found` is free: the first wavefront read it before it came here
        if (wave == 0) {
          const int n = min(NW, runs - r0);
#pragma unroll
          for (int w = 0; w < NW; ++w)
            if (w < n)
#pragma unroll
              for (int i = 0; i < NB; ++i) {
                const f32x4 v = found[par][w][i][lane];
#pragma unroll
                for (int e = 0; e < 4; ++e) sum[i][e] = __builtin_fmaf(v[e], w & 1 ? -1.f : 1.f, sum[i][e]);
              }
        }
      }
    };
    if (a.unfinished((steps - 1) * BK, K)) form(std::true_type());
    else form(std::false_type());
  }
  if (wave) return;
  static_assert(NW % 2 == 0, "a wavefront's runs are all odd or all even");
  mend<OP, ACC == kAligned>(g, sums, [&](int) { return min(m0 + lr, g.M - 1); }, [&](int i) { return i * cols + min(n0 + lr, cols - 1); }, kg);
  if (OP == 2) {
    const int n = n0 + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + kg * 4 + r;
      if (m < g.M && n < g.N) unsafeAtomicAdd(g.C + (int64_t)m * g.N + n, sum[0][r]);
    }
    return;
  }
  const int m = m0 + lr, n = n0 + kg * 4;
  if (m >= g.M) return;
  if (EPI == kEpiSwiglu) emit_swiglu<ACC == kAligned>(g, m, n, sum[0], sum[NB - 1]);
  else emit<OP, EPI, ACC == kAligned>(g, m, n, sum[0]);
}

// Wavefronts a SIMD: LDS holds one workgroup with tiles of 128, two with 128 x 64 (128 registers; with more, and one workgroup, op 2
// 2048 x 3072 x 1024 takes 97 us for 80).
constexpr int waves_of(int tm, int tn, int feed) { return tm * tn > 128 * 64 || tn == 16 ? 2 : feed == kFeedFew ? 6 : 4; }
template <int OP, int EPI, int TM, int TN, int ACC, int FEED = kFeed>
__global__ __launch_bounds__((kTileThreads<TN, FEED>), waves_of(TM, TN, FEED)) void k_gemm_f32(Args g) {
  gemm_tile<OP, EPI, TM, TN, ACC, FEED>(g, blockIdx.x, gridDim.x);
}
template <int OP, int EPI, int ACC>
__global__ __launch_bounds__(kThreads, 2) void k_gemm_f32_few(Args g) { gemm_few<OP, EPI, ACC>(g, blockIdx.x, gridDim.x); }

// the weight gradients of a layer in one launch, all in tiles of one size
template <int TM, int TN, int ACC, int FEED = kFeed>
__global__ __launch_bounds__((kTileThreads<TN, FEED>), waves_of(TM, TN, FEED)) void k_gemm_f32_grads(GradGroup l) {
  int i = 0;
  while (i + 1 < kGrads && (int)blockIdx.x >= l.first[i + 1]) ++i;
  const int wg = (int)blockIdx.x - l.first[i], n = l.first[i + 1] - l.first[i];
  const Args g{(const float*)l.A[i], (const float*)l.B[i], nullptr, l.C[i], nullptr, l.M[i], l.N[i], l.K, l.tm[i], l.tn[i], RopeArgs{nullptr, 1, 2, 0}};
  if constexpr (TN == 16) gemm_few<2, kEpiPlain, ACC>(g, wg, n);
  else gemm_tile<2, kEpiPlain, TM, TN, ACC, FEED>(g, wg, n);
}

inline bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

// Tile and its grid for a product: the least of (steps + ends) x time of a step of the CU with the most tiles.  Times are fits
// (us, op 0 to 2 within 5 %): a 128-tile 1.25; 128 x 64 0.78 alone on its CU, 0.72 each of several; a 64-tile 0.58 alone, 0.88
// two, 0.44 each of more; a 32-tile 0.23 (SwiGLU, with four feeding wavefronts and 64 rows of B, 0.46), 0.36 two, 0.52 three, 0.18 each of
// more (SwiGLU 1.6 x).  What starts and ends a tile counts as 4.8, 4, 4 and 6 steps (10 of 0.23); in op 2, whose large tiles have many atomics to
// themselves, as 6, 5, 4 and 6; with the SwiGLU gradient, whose loads and arithmetic a large tile has alone on its CU, as 12, 8, 5 and
// 6.  A 16-tile of k_gemm_f32_few: 0.17 a run (op 2, whose loads take 64 bytes of a row, 0.23) and 0.45 (SwiGLU 1.85 x), 1 once.  With
// one set of ends and runs for all, op 2 828 x 152 x 3768 went to tiles of 16 (47 us, 39 in tiles of 32 with four feeding wavefronts),
// the gradient 3728 x 2352 over k = 48 to 128 x 64 (41 us, 33 in 64); over 1500 sizes 119 choices differed, 0.75 to 1.06 times the
// time, the median 0.90.
// A product is not cut along k over workgroups: their sums would be added in the order in which they end, and neither would a
// microbatch's rows have the same bits alone and in a group, nor two passes of the mode that gradients are checked in agree.
// us by tile, 128 / 128 x 64 / 64 / 32 (four feeding wavefronts): op 0 1024 x 1024 x 1024 39 / 29 / 22 / 28, 2048 x 1024 x 5632 188 / 143 / 157 /
// 236, 3072 x 1024 x 1024 42 / 46 / 46 / 66, 4096 x 768 x 288 17 / 18 / 17 / 23, 1024 x 288 x 1536 55 / 39 / 27 / 20, op 2 5632 x 1024 x 2048
// 164 / 147 / 166 / 253, 288 x 768 x 4096 139 / 105 / 64 / 38.  32 / 16: op 0 128 x 288 x 1536 16.6 / below 7.5 (the launch), 512 x 288 x 1536
// 16.9 / 14.2, 1024 x 288 x 1536 21 / 22, 64 x 1024 x 5632 53 / 21, 512 x 768 x 288 7.7 / 8.9.
constexpr int kEdges[5][2] = {{128, 128}, {128, 64}, {64, 64}, {32, 32}, {16, 16}};
static double f32_us(int op, int t, int64_t tiles, int64_t K, int epi) {
  const int64_t cus = cu_count(), steps = (K + BK - 1) / BK, load = (tiles + cus - 1) / cus;
  const double c = (double)load;
  if (t == 4) return 1.0 + c * ((op == 2 ? 0.23 : 0.17) * (double)((steps + kRun - 1) / kRun) + 0.45) * (epi == kEpiSwiglu ? 1.85 : 1.0);
  const double step = t == 0 ? 1.25 * c : t == 1 ? (load == 1 ? 0.78 : 0.72 * c) : t == 2 ? (load == 1 ? 0.58 : 0.44 * c)
                      : (load == 1 ? (epi == kEpiSwiglu ? 0.29 : 0.23) : load == 2 ? 0.36 : load == 3 ? 0.52 : 0.18 * c) * (epi == kEpiSwiglu ? 1.6 : 1.0);
  constexpr double kEnds[3][4] = {{4.8, 4, 4, 6}, {6, 5, 4, 6}, {12, 8, 5, 6}};
  if (t == 3 && load == 1 && epi != kEpiSwiglu) return step * ((double)steps + 10.0);
  return step * ((double)steps + kEnds[epi == kEpiSwigluBwd ? 2 : op == 2 ? 1 : 0][t]);
}
static bool feed_few(int64_t tiles, int epi) { return tiles <= 2 * (int64_t)cu_count() && epi != kEpiSwiglu; }   // see gemm_tile
struct F32Shape { int tile_m, tile_n, tm, tn; };
static F32Shape choose_f32(int op, int64_t M, int64_t N, int64_t K, int epi, bool far) {   // far: tiles of 64 only
  const int64_t out = epi == kEpiSwiglu ? N / 2 : N;   // width of one stored run of columns
  F32Shape best{};
  double best_us = 0;
  for (int t = far ? 2 : 0; t < (far ? 3 : 5); ++t) {
    const int m = kEdges[t][0], n = kEdges[t][1], w = epi == kEpiSwiglu && t < 3 ? n / 2 : n;   // w: stored columns of one run
    const int64_t tm = (M + m - 1) / m, tn = (out + w - 1) / w;
    const double us = f32_us(op, t, tm * tn, K, epi);
    if (best.tm && us >= best_us) continue;
    best_us = us;
    best = {m, n, (int)tm, (int)tn};
  }
  return best;
}

GemmShape gemm_f32_shape(int op, int64_t M, int64_t N, int64_t K, int epi) {
  const F32Shape c = choose_f32(op, M, N, K, epi, gemm_f32_far(op, M, N, K, epi));
  return {c.tile_n, c.tm * c.tn, c.tm * c.tn};
}

// A tile of some operand reaches further than 31 bits: 127 rows of K, 31 rows of a k-strided one's width, all up rows from the gate
// rows on.
bool gemm_f32_far(int op, int64_t M, int64_t N, int64_t K, int epi) {
  constexpr int64_t kRow = 1 << 22, kWidth = 1 << 24;
  return op == 0 ? K > kRow || (epi == kEpiSwiglu && (N / 2 + 128) * K >= 1ll << 29) : op == 1 ? K > kRow || N > kWidth : M > kWidth || N > kWidth;
}

// epi as in gemm_mfma: 0 plain (R optional), 1 rotary, 2 SwiGLU (N = 2h, aux = act), 3 SwiGLU backward (N = h, R =
// gate|up, C = d(gate)|d(up)).
void gemm_f32(hipStream_t s, int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C, const void* R,
              const RopeArgs* rope, int epi, void* aux) {
  Args g{(const float*)A, (const float*)B, (const float*)R, (float*)C, (float*)aux, (int)M, (int)N, (int)K, 0, 0,
         rope ? *rope : RopeArgs{nullptr, 1, 2, 0}};
  if (rope) epi = kEpiRope;
  const int64_t out = epi == kEpiSwiglu ? N / 2 : N;   // width of one stored run of columns
  const bool aligned = al16(A) && al16(B) && al16(C) && al16(R) && al16(aux) && out % 4 == 0 && (op == 2 ? M % 4 == 0 : K % 4 == 0);
  const bool far = gemm_f32_far(op, M, N, K, epi);
  const F32Shape c = choose_f32(op, M, N, K, epi, far);
  g.tiles_m = c.tm;
  g.tiles_n = c.tn;
  const dim3 grid((unsigned)(c.tm * c.tn));
#define SP_GO_32(OP, EPI, ACC, FEED) \
  hipLaunchKernelGGL((k_gemm_f32<OP, EPI, 32, 32, ACC, FEED>), grid, dim3(kTileThreads<32, FEED>), 0, s, g)
#define SP_GO(OP, EPI, ACC)                                                                                             \
  do {                                                                                                                  \
    if (c.tile_n == 128) hipLaunchKernelGGL((k_gemm_f32<OP, EPI, 128, 128, ACC>), grid, dim3(kThreads), 0, s, g);           \
    else if (c.tile_m == 128) hipLaunchKernelGGL((k_gemm_f32<OP, EPI, 128, 64, ACC>), grid, dim3(kThreads), 0, s, g);       \
    else if (c.tile_n == 64) hipLaunchKernelGGL((k_gemm_f32<OP, EPI, 64, 64, ACC>), grid, dim3(kThreads), 0, s, g);         \
    else if (c.tile_n == 32 && feed_few(c.tm * c.tn, EPI)) SP_GO_32(OP, EPI, ACC, (EPI == kEpiSwiglu ? kFeed : kFeedFew));  \
    else if (c.tile_n == 32) SP_GO_32(OP, EPI, ACC, kFeed);                                                                 \
    else hipLaunchKernelGGL((k_gemm_f32_few<OP, EPI, ACC>), grid, dim3(kThreads), 0, s, g);                                 \
  } while (0)
#define SP_GO_V(OP, EPI)                                                                                                \
  do {                                                                                                                  \
    if (far) hipLaunchKernelGGL((k_gemm_f32<OP, EPI, 64, 64, kFar>), grid, dim3(kThreads), 0, s, g);                    \
    else if (aligned) SP_GO(OP, EPI, kAligned);                                                                         \
    else SP_GO(OP, EPI, kUnaligned);                                                                                    \
  } while (0)
  if (op == 0 && epi == kEpiRope) SP_GO_V(0, kEpiRope);
  else if (op == 0 && epi == kEpiSwiglu) SP_GO_V(0, kEpiSwiglu);
  else if (op == 0) SP_GO_V(0, kEpiPlain);
  else if (op == 1 && epi == kEpiSwigluBwd) SP_GO_V(1, kEpiSwigluBwd);
  else if (op == 1) SP_GO_V(1, kEpiPlain);
  else SP_GO_V(2, kEpiPlain);
#undef SP_GO_V
#undef SP_GO
#undef SP_GO_32
}

// One tile for all of them; entries as in gemm_f32, bit for bit.
void gemm_f32_grads(hipStream_t s, int64_t K, const GradItem (&items)[kGrads]) {
  GradGroup g{};
  bool aligned = true;
  for (const GradItem& i : items) aligned = aligned && al16(i.A) && al16(i.B) && al16(i.C) && i.M % 4 == 0 && i.N % 4 == 0;
  int tile = 0;
  double best_us = 0;
  for (int t = 0; t < 5; ++t) {
    int64_t tiles = 0;
    for (const GradItem& i : items) tiles += ((i.M + kEdges[t][0] - 1) / kEdges[t][0]) * ((i.N + kEdges[t][1] - 1) / kEdges[t][1]);
    const double us = f32_us(2, t, tiles, K, kEpiPlain);
    if (t && us >= best_us) continue;
    best_us = us;
    tile = t;
  }
  for (int i = 0; i < kGrads; ++i) {
    const GradItem& x = items[i];
    g.A[i] = x.A; g.B[i] = x.B; g.C[i] = x.C;
    g.M[i] = (int)x.M; g.N[i] = (int)x.N;
    g.tm[i] = (int)((x.M + kEdges[tile][0] - 1) / kEdges[tile][0]);
    g.tn[i] = (int)((x.N + kEdges[tile][1] - 1) / kEdges[tile][1]);
    g.first[i + 1] = g.first[i] + g.tm[i] * g.tn[i];
  }
  g.K = (int)K;
  const dim3 grid(g.first[kGrads]);
#define SP_GO(TM, TN, FEED)                                                                                                                      \
  do {                                                                                                                                           \
    if (aligned) hipLaunchKernelGGL((k_gemm_f32_grads<TM, TN, kAligned, FEED>), grid, dim3(kTileThreads<TN, FEED>), 0, s, g);                    \
    else hipLaunchKernelGGL((k_gemm_f32_grads<TM, TN, kUnaligned, FEED>), grid, dim3(kTileThreads<TN, FEED>), 0, s, g);                          \
  } while (0)
  if (tile == 0) SP_GO(128, 128, kFeed);
  else if (tile == 1) SP_GO(128, 64, kFeed);
  else if (tile == 2) SP_GO(64, 64, kFeed);
  else if (tile == 3 && feed_few(g.first[kGrads], kEpiPlain)) SP_GO(32, 32, kFeedFew);
  else if (tile == 3) SP_GO(32, 32, kFeed);
  else SP_GO(16, 16, kFeed);
#undef SP_GO
}

}  // namespace sp
