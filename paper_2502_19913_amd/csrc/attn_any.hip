// Causal attention for any element type and even head dimension up to 256: the float mode, on the float matrix instruction
// (v_mfma_f32_16x16x4_f32), and bf16 with head dimensions the bf16 kernels (attn_flash.hip) do not take, on the bf16 one, with
// probabilities and score gradients still floats (Stored<bf16> below).  Also the dispatch over the two families.
//
// Same plan as the bf16 kernels: a workgroup of four wavefronts (or two sets of four, below) owns 64 queries (16 per
// wavefront; 64 keys in the dK/dV kernel) of one head and walks the other side in tiles of 32 rows through LDS, two
// buffers, loaded into registers one tile ahead, one barrier per tile.  Scores are formed transposed, S^T[key][query]
// = K Q^T, so a lane (query lane % 16) ends with the scores of keys 4 kg .. 4 kg + 3 (kg = lane / 16), and its row
// statistics are per-lane scalars; the instruction's four k-slots may stand for any keys, so accumulator r of all
// lanes is directly the operand of the r-th instruction of the next product (O^T += V^T P^T).  The dK/dV kernel is
// the mirror image.
//
// In float the row-wise operand of a product is one 16-byte LDS read per four instructions, the transposed one a 4-byte read
// per instruction; LDS rows are padded by 16 bytes, which keeps both free of bank conflicts.  One LDS read per
// 32-cycle instruction leaves LDS idle most of the time; what bounds a workgroup is the chain of its tiles.  In bf16 the
// matrix instructions are a fifth of that and vector instructions bound it (four wavefronts a SIMD, 285 a tile and wavefront of
// the forward kernel before, 190 now): tiles lie in LDS as stored, the transposed operand comes by the LDS transpose read,
// exponentials take two thirds of expf's instructions, masks only stand where some key is hidden.  Heads of 48, forward | backward
// us, float instruction and float tiles -> this: 3 x 333 positions x 6 heads 17 | 43 -> 10 | 25, 16 x 256 x 6 22 | 53 -> 12 |
// 31, 8 x 1024 x 16 263 | 646 -> 106 | 287; the 50M shape on 3 x 333 tokens 3.60 -> 2.96 ms a pass.  (Float, of the same
// exponentials and masks: 8 x 1024 x 16 heads of 48 312 | 891 -> 284 | 856.)  HD is the head dimension rounded up to a compiled
// size; columns past the real one are zeros.  One wavefront per row of
// scores (the kernels these replaced) left the matrix cores idle and re-read K and V for every query.  Measured,
// forward | backward (dQ and dK/dV), us: 6 sequences x 512 x 16 heads of 64 in float 542 -> 90 (36 TFLOP/s of the
// causal half) | 7825 -> 269; 16 x 256 x 6 heads of 48 129 -> 33 | 1522 -> 82; 2 x 64 x 6 heads of 48, where launches
// are most of it, 8 | 30 -> 18 (the delta pass rides in the dQ kernel); the two sets took the heads of 48 on 256
// positions from 27 | 75 to 21 | 63 beside the weight-gradient products.
//
// Layout: qkv rows of (H + 2*Hkv)*hd elements = query heads | key heads | value heads; rows are B sequences of T
// positions; o rows of H*hd; lse[b][a][i] = log sum_j exp(q_i.k_j/sqrt(hd)).
#include "devutil.h"
#include "internal.h"

namespace sp {

namespace {

constexpr int kMaxHd = 256;
constexpr int kThreads = 256;
constexpr int KT = 32;    // rows of a tile of the walked side
constexpr int BQ = 64;    // rows a workgroup owns
// Sets of four wavefronts that take the tiles of the walked side in turn.  A workgroup's time is the chain of its tiles
// (score products, exponentials, second products, LDS round trips: three to four times the matrix instructions alone),
// and small models have one or two wavefronts per SIMD to overlap it.  Two sets up to a head dimension of 48: heads of
// 48, 50M shape in bf16 on 3 x 333 tokens 4.40 -> 3.89 ms, in float on 4 x 256 tokens 6.14 -> 5.81 ms, on 64 tokens
// 2.02 -> 1.96 ms a pass; heads of 32 alone, forward | backward us with one set -> two, 3 x 333 x 6 heads in float 18 |
// 50 -> 14 | 39, in bf16 18 | 45 -> 13 | 32, 8 x 1024 x 16 heads in float 219 | 615 -> 205 | 619, in bf16 177 | 435 -> 167 |
// 396 (heads of 16, which run as 32 columns, the same); only the bf16 forward of 8 x 1024 x 16 heads of 48 loses, 238 ->
// 262.  At 64 the stage of 2 x 512 tokens was 0.5 % slower with two sets, and from 96 on their buffers take the room of
// a CU's second workgroup.
template <int HD> constexpr int kSets = HD <= 48 ? 2 : 1;

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ f32x4 mfma(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }

// exp(x): 2^n times 2^f of x log2(e), f formed from two parts of the constant; two thirds of expf's instructions (which also looks after
// overflow), and as that one the subnormal results, which the instruction alone returns as zero.  n ends at -200, where nothing is
// left of a float, so that f is a number for all x but infinities, and -inf for -inf.
__device__ __forceinline__ float exp_(float x) {
  constexpr float kL = 1.44269502f, kLl = 1.92596299e-8f;   // log2(e) and what is left of it
  const float n = fmaxf(rintf(x * kL), -200.f), f = __builtin_fmaf(x, kLl, __builtin_fmaf(x, kL, -n));
  return __builtin_ldexpf(__builtin_amdgcn_exp2f(f), (int)n);
}

// What differs between the two storage types.  Quad: four values of a row as they travel and lie in LDS (LD values a row).
//   dot2    the two products whose operands both come from storage (scores, and dO V^T): a0, a1 four columns of the walked
//           side, b0, b1 of the side that stays in registers, c0, c1 two independent sums.
//   times   acc[c] (columns 16 c + lr) += products of probabilities (or score gradients) with the tile's 32 rows: lane
//           group kg holds those of rows 4 kg .. 4 kg + 3 of either half (p0, p1).
// Probabilities and score gradients are floats in either type.  bf16 storage takes the bf16 instruction for both: stored
// operands are used as they are, their products are exact and the sums float, and a probability is the sum of three
// bfloat16s, exactly (one below 2^-110 to 2^-134): three instructions over 32 rows (48 cycles) instead of eight float ones (256).
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
template <class T> struct Stored {
  typedef f32x4 Quad;
  template <int HD> static constexpr int LD = HD + 4;
  static __device__ __forceinline__ Quad of(float a, float b, float c, float d) { return Quad{a, b, c, d}; }
  static __device__ __forceinline__ f32x4 floats(const Quad& q) { return q; }
  static __device__ __forceinline__ void dot2(const Quad& a0, const Quad& b0, f32x4& c0, const Quad& a1, const Quad& b1, f32x4& c1) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      c0 = mfma(a0[e], b0[e], c0);
      c1 = mfma(a1[e], b1[e], c1);
    }
  }
  template <int LD, int NS>
  static __device__ __forceinline__ void times(const f32x4& p0, const f32x4& p1, const float* tile, int lr, int kg, f32x4 (&acc)[NS]) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float* row = tile + (t * 16 + kg * 4 + e) * LD + lr;
#pragma unroll
        for (int c = 0; c < NS; ++c) acc[c] = mfma(row[c * 16], t ? p1[e] : p0[e], acc[c]);
      }
  }
};
template <> struct Stored<bf16> {
  typedef s16x4 Quad;
  template <int HD> static constexpr int LD = HD + 8;
  static __device__ __forceinline__ Quad of(bf16 a, bf16 b, bf16 c, bf16 d) {
    typedef __attribute__((ext_vector_type(4))) __bf16 B;
    return __builtin_bit_cast(Quad, B{a, b, c, d});
  }
  static __device__ __forceinline__ f32x4 floats(const Quad& v) {
    const uint2 q = __builtin_bit_cast(uint2, v);
    return f32x4{bf16_bits_to_float(q.x & 0xffffu), __uint_as_float(q.x & 0xffff0000u), bf16_bits_to_float(q.y & 0xffffu), __uint_as_float(q.y & 0xffff0000u)};
  }
  static __device__ __forceinline__ void dot2(const Quad& a0, const Quad& b0, f32x4& c0, const Quad& a1, const Quad& b1, f32x4& c1) {
    c0 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a0, b0, c0, 0, 0, 0);
    c1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a1, b1, c1, 0, 0, 0);
  }
  // The walked side column by column with the LDS transpose read (within 16 lanes, lane s addresses row s / 4 and columns
  // 4 (s % 4) .. + 3 of a block of 4 rows x 16 columns and receives column s of the four rows).
  template <int LD, int NS>
  static __device__ __forceinline__ void times(const f32x4& p0, const f32x4& p1, const bf16* tile, int lr, int kg, f32x4 (&acc)[NS]) {
    typedef __attribute__((ext_vector_type(2))) float f2;
    typedef __attribute__((ext_vector_type(2))) __bf16 b2;
    typedef __attribute__((ext_vector_type(4))) uint32_t U;
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    float v[8] = {p0[0], p0[1], p0[2], p0[3], p1[0], p1[1], p1[2], p1[3]};
    U part[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const uint32_t p = __builtin_bit_cast(uint32_t, __builtin_convertvector(f2{v[2 * w], v[2 * w + 1]}, b2));
        part[i][w] = p;
        v[2 * w] -= bf16_bits_to_float(p & 0xffffu);
        v[2 * w + 1] -= __uint_as_float(p & 0xffff0000u);
      }
    const bf16* at = tile + (kg * 4 + (lr >> 2)) * LD + (lr & 3) * 4;
#pragma unroll
    for (int c = 0; c < NS; ++c) {
      const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + c * 16));
      const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(at + 16 * LD + c * 16));
      typedef __attribute__((ext_vector_type(8))) short s16x8;
      const bf16x8 x = __builtin_bit_cast(bf16x8, s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
#pragma unroll
      for (int i = 2; i >= 0; --i) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, __builtin_bit_cast(bf16x8, part[i]), acc[c], 0, 0, 0);
    }
  }
};

// columns c .. c+3 of a row of hd, zeros past it; vec: every row starts 4-element aligned and hd is a multiple of 4
template <class T>
__device__ __forceinline__ typename Stored<T>::Quad row4(const T* row, int c, int hd, bool vec) {
  typedef typename Stored<T>::Quad Quad;
  const T zero = from_float<T>(0.f);
  Quad v = Stored<T>::of(zero, zero, zero, zero);
  if (vec) {
    if (c < hd) v = *reinterpret_cast<const Quad*>(row + c);
  } else {
    v = Stored<T>::of(c < hd ? row[c] : zero, c + 1 < hd ? row[c + 1] : zero, c + 2 < hd ? row[c + 2] : zero, c + 3 < hd ? row[c + 3] : zero);
  }
  return v;
}
template <class T>
__device__ __forceinline__ void put4(T* row, int c, int hd, bool vec, const f32x4& v) {
  if (vec) {
    if (c < hd) {
      if constexpr (sizeof(T) == 4) *reinterpret_cast<f32x4*>(row + c) = v;
      else *reinterpret_cast<uint2*>(row + c) = make_uint2(pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3]));
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (c + e < hd) row[c + e] = from_float<T>(v[e]);
  }
}
// gradient of a rotated vector -> gradient before the rotation, columns c .. c+3 at position pos
__device__ __forceinline__ void unrotate4(f32x4& v, const float* tab, int pos, int c, int hd) {
#pragma unroll
  for (int p = 0; p < 2; ++p)
    if (c + 2 * p < hd) {
      const float2 cs = reinterpret_cast<const float2*>(tab)[(int64_t)pos * (hd / 2) + c / 2 + p];
      const float a = v[2 * p], b = v[2 * p + 1];
      v[2 * p] = a * cs.x + b * cs.y;
      v[2 * p + 1] = b * cs.x - a * cs.y;
    }
}
// over the four lanes that hold one query's (key's) values
__device__ __forceinline__ float sum4(float v) { v += __shfl_xor(v, 16); return v + __shfl_xor(v, 32); }
__device__ __forceinline__ float max4(float v) { v = fmaxf(v, __shfl_xor(v, 16)); return fmaxf(v, __shfl_xor(v, 32)); }

// A masked probability (or score gradient) is zero, but zero times a value that is not finite is NaN, and the matrix
// instruction takes every row of a tile for all of its columns: a NaN or an infinity would reach positions that do not see
// its row.  So a wavefront whose sums come out as NaN forms those rows anew, each over the positions it sees (below): a
// row that sees the value gets its NaN again, the others their results.  So do rows that met a whole tile of scores of
// -inf first, whose running maximum is then no number to subtract.  A check of the sums once at the end costs nothing
// that can be measured; looking through the one tile that a row sees in part cost 1 % of a pass (50M shape in bf16).

// The rows (queries or keys, 16 a wavefront, bit lane % 16) with a NaN among a lane's sums.
template <int NS>
__device__ __forceinline__ uint32_t nan_rows(const f32x4 (&v)[NS]) {
  f32x4 t = v[0];
#pragma unroll
  for (int c = 1; c < NS; ++c) t += v[c];   // infinities of both signs may add a row that has no NaN: no harm
  const float u = (t[0] + t[1]) + (t[2] + t[3]);
  const uint64_t m = __ballot(u != u);
  return (uint32_t)(m | m >> 16 | m >> 32 | m >> 48) & 0xffffu;
}

// One wavefront: 64 positions at a time, then columns lane, lane + 64, ..
template <class T>
__device__ __forceinline__ float dot_rows(const T* a, const T* b, int hd) {
  float d = 0.f;
  for (int c = 0; c < hd; ++c) d += to_float(a[c]) * to_float(b[c]);
  return d;
}
// acc[u] += sum over n rows, one per lane's w, of w * row[lane + 64 u]
template <class T, int NU>
__device__ __forceinline__ void add_rows(float (&acc)[NU], float w, const T* rows, int64_t ld, int n, int hd, int lane) {
  for (int i = 0; i < n; ++i) {
    const float x = __shfl(w, i);
#pragma unroll
    for (int u = 0; u < NU; ++u)
      if (lane + 64 * u < hd) acc[u] += x * to_float(rows[i * ld + lane + 64 * u]);
  }
}
template <class T, int NU>
__device__ __forceinline__ void put_row(T* row, const float (&v)[NU], int hd, int lane) {
#pragma unroll
  for (int u = 0; u < NU; ++u)
    if (lane + 64 * u < hd) row[lane + 64 * u] = from_float<T>(v[u]);
}
// as unrotate4; the other value of a pair is the neighbouring lane's
template <int NU>
__device__ __forceinline__ void unrotate_row(float (&v)[NU], const float* tab, int pos, int hd, int lane) {
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int c = min(lane + 64 * u, hd - 1);
    const float2 cs = reinterpret_cast<const float2*>(tab)[(int64_t)pos * (hd / 2) + c / 2];
    const float other = __shfl_xor(v[u], 1);
    v[u] = c & 1 ? v[u] * cs.x - other * cs.y : v[u] * cs.x + other * cs.y;
  }
}
// a query over its n keys
template <class T, int HD>
__device__ void fwd_row(const T* q, const T* k, const T* v, int64_t ld, int n, int hd, float scale, T* o, float* lse, int lane) {
  float m = -INFINITY, l = 0.f, acc[(HD + 63) / 64] = {};
  for (int j = lane; j < n; j += 64) m = fmaxf(m, dot_rows(q, k + j * ld, hd) * scale);
  m = wave_max(m);
  for (int j0 = 0; j0 < n; j0 += 64) {
    const float p = j0 + lane < n ? expf(dot_rows(q, k + (j0 + lane) * ld, hd) * scale - m) : 0.f;
    l += p;
    add_rows(acc, p, v + j0 * ld, ld, min(64, n - j0), hd, lane);
  }
  l = wave_sum(l);
#pragma unroll
  for (int u = 0; u < (HD + 63) / 64; ++u) acc[u] /= l;
  put_row(o, acc, hd, lane);
  if (lane == 0) *lse = m + logf(l);
}
template <class T, int HD>
__device__ void dq_row(const T* q, const T* dO, const T* k, const T* v, int64_t ld, int n, int hd, float scale, float L, float dlt,
                       const float* rope_tab, T* dq, int lane) {
  float acc[(HD + 63) / 64] = {};
  for (int j0 = 0; j0 < n; j0 += 64) {
    float ds = 0.f;
    if (j0 + lane < n) {
      const int64_t at = (j0 + lane) * ld;
      ds = expf(dot_rows(q, k + at, hd) * scale - L) * (dot_rows(dO, v + at, hd) - dlt) * scale;
    }
    add_rows(acc, ds, k + j0 * ld, ld, min(64, n - j0), hd, lane);
  }
  if (rope_tab) unrotate_row(acc, rope_tab, n - 1, hd, lane);
  put_row(dq, acc, hd, lane);
}
// a key at position pos over the queries of `rep` heads from its position on; q, dO: the first of these heads at position 0
template <class T, int HD>
__device__ void dkv_row(const T* k, const T* v, const T* q, const T* dO, const float* lse, const float* delta, int64_t ld, int64_t ldo,
                        int rep, int pos, int T_, int hd, float scale, const float* rope_tab, T* dk, T* dv, int lane) {
  float ak[(HD + 63) / 64] = {}, av[(HD + 63) / 64] = {};
  for (int a = 0; a < rep; ++a, q += hd, dO += hd, lse += T_, delta += T_)
    for (int i0 = pos; i0 < T_; i0 += 64) {
      float p = 0.f, ds = 0.f;
      if (const int i = i0 + lane; i < T_) {
        p = expf(dot_rows(q + i * ld, k, hd) * scale - lse[i]);
        ds = p * (dot_rows(dO + i * ldo, v, hd) - delta[i]) * scale;
      }
      add_rows(ak, ds, q + i0 * ld, ld, min(64, T_ - i0), hd, lane);
      add_rows(av, p, dO + i0 * ldo, ldo, min(64, T_ - i0), hd, lane);
    }
  if (rope_tab) unrotate_row(ak, rope_tab, pos, hd, lane);
  put_row(dk, ak, hd, lane);
  put_row(dv, av, hd, lane);
}

// Two matrices' tiles of KT rows on their way from memory to LDS: [KT][LD] values each.
template <class T, int HD>
struct Pair {
  typedef Stored<T> S;
  typedef typename S::Quad Quad;
  static constexpr int LD = S::template LD<HD>, N4 = (KT * HD / 4 + kThreads - 1) / kThreads;
  Quad x[N4], y[N4];
  // rows r0 .. of X (row stride ldx) and Y (ldy); rows at or past `rows` are zeros
  __device__ __forceinline__ void load(const T* X, int64_t ldx, const T* Y, int64_t ldy, int r0, int rows, int hd, bool vec, int tid) {
    const T *xt = X + (int64_t)r0 * ldx, *yt = Y + (int64_t)r0 * ldy;
#pragma unroll
    for (int j = 0; j < N4; ++j) {
      const int i = tid + kThreads * j, in = i / (HD / 4), c = i % (HD / 4) * 4;
      const T zero = from_float<T>(0.f);
      x[j] = y[j] = S::of(zero, zero, zero, zero);
      if (r0 + in < rows && i < KT * HD / 4) {   // 32 rows of at most 3 x 65535 heads of 256: offsets fit 32 bits
        x[j] = row4(xt + (uint32_t)in * (uint32_t)ldx, c, hd, vec);
        y[j] = row4(yt + (uint32_t)in * (uint32_t)ldy, c, hd, vec);
      }
    }
  }
  __device__ __forceinline__ void store(T* lx, T* ly, int tid) const {
#pragma unroll
    for (int j = 0; j < N4; ++j) {
      const int i = tid + kThreads * j, at = i / (HD / 4) * LD + i % (HD / 4) * 4;
      if (i < KT * HD / 4) {
        *reinterpret_cast<Quad*>(lx + at) = x[j];
        *reinterpret_cast<Quad*>(ly + at) = y[j];
      }
    }
  }
};

// The second set's HD / 16 accumulators of every lane on their way to the first set, quad by quad; the place past them,
// which both return, has room for two more floats of a lane (kThreads apart).  All of it fits a set's buffers:
// kThreads * (HD / 4 + 2) floats <= 4 KT LD values (checked below).
template <int HD>
__device__ __forceinline__ float* give(float* at, const f32x4* v, int tid) {
  static_assert(kThreads * (HD / 4 + 2) * 4 <= 4 * KT * (HD + 8) * 2, "two sets' exchange fits one set's buffers (of the smaller type)");
#pragma unroll
  for (int c = 0; c < HD / 16; ++c) reinterpret_cast<f32x4*>(at)[c * kThreads + tid] = v[c];
  return at + HD / 16 * 4 * kThreads + tid;
}
template <int HD>
__device__ __forceinline__ const float* take(const float* at, f32x4* v, int tid) {
#pragma unroll
  for (int c = 0; c < HD / 16; ++c) v[c] = reinterpret_cast<const f32x4*>(at)[c * kThreads + tid];
  return at + HD / 16 * 4 * kThreads + tid;
}

template <class T, int HD>
__global__ __launch_bounds__(kThreads * kSets<HD>) void k_attn_fwd(const T* __restrict__ qkv, int T_, int H, int Hkv, int hd, bool vec, float scale,
                                                       T* __restrict__ o, float* __restrict__ lse) {
  typedef Stored<T> S;
  typedef typename S::Quad Quad;
  constexpr int LD = S::template LD<HD>, NS = HD / 16, SETS = kSets<HD>;
  __shared__ __attribute__((aligned(16))) T smem_all[SETS][2][2][KT * LD];
  const int set = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), tid = threadIdx.x % kThreads;
  const int lane = tid & 63, lr = lane & 15, kg = lane >> 4, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto& smem = smem_all[set];
  const int a = blockIdx.y, b = blockIdx.z, kvh = a / (H / Hkv);
  const int q0 = (int)(gridDim.x - 1 - blockIdx.x) * BQ;   // the longest blocks of a head first
  const int qw0 = q0 + wave * 16, q = qw0 + lr;
  const int64_t ld = (int64_t)(H + 2 * Hkv) * hd;
  const T* base = qkv + (int64_t)b * T_ * ld;
  const T *kp = base + (H + kvh) * hd, *vp = base + (H + Hkv + kvh) * hd;
  Quad qf[NS];
  f32x4 oacc[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    qf[s] = row4(base + (int64_t)min(q, T_ - 1) * ld + a * hd, s * 16 + kg * 4, hd, vec);
    oacc[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  float m_i = -INFINITY, l_i = 0.f;
  const int tiles = (min(T_, q0 + BQ) + KT - 1) / KT;
  Pair<T, HD> in;
  in.load(kp, ld, vp, ld, set * KT, T_, hd, vec, tid);   // a row past the end is zeros
  in.store(smem[0][0], smem[0][1], tid);
  __syncthreads();
  for (int i = 0; i * SETS < tiles; ++i) {   // every wavefront the same number of rounds
    const int kt = i * SETS + set, k0 = kt * KT;
    if (kt + SETS < tiles) in.load(kp, ld, vp, ld, k0 + SETS * KT, T_, hd, vec, tid);
    const T *lk = smem[i & 1][0], *lv = smem[i & 1][1];
    if (kt < tiles && k0 <= qw0 + 15) {   // some key of the tile is visible to this wavefront
      f32x4 st[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
#pragma unroll
      for (int s = 0; s < NS; ++s) {
        const Quad f0 = *reinterpret_cast<const Quad*>(lk + lr * LD + s * 16 + kg * 4);
        const Quad f1 = *reinterpret_cast<const Quad*>(lk + (16 + lr) * LD + s * 16 + kg * 4);
        S::dot2(f0, qf[s], st[0], f1, qf[s], st[1]);
      }
      if (k0 + KT - 1 > qw0) {   // not every key is visible to every query
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (k0 + t * 16 + kg * 4 + r > q) st[t][r] = -INFINITY;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, st[t][r]);
      const float m_new = fmaxf(m_i, max4(mx) * scale);   // -inf while every score is: NaN, formed anew
      const float alpha = exp_(m_i - m_new);
      float rs = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          st[t][r] = exp_(st[t][r] * scale - m_new);
          rs += st[t][r];
        }
      l_i = l_i * alpha + rs;
      m_i = m_new;
#pragma unroll
      for (int c = 0; c < NS; ++c) oacc[c] *= alpha;
      S::template times<LD>(st[0], st[1], lv, lr, kg, oacc);
    }
    if (kt + SETS < tiles) in.store(smem[(i + 1) & 1][0], smem[(i + 1) & 1][1], tid);
    __syncthreads();
  }
  if (SETS == 2) {   // the other set's maximum, sum and outputs come over through LDS; it may have seen no key (-inf, 0, 0)
    if (set == 1) {
      float* p = give<HD>(reinterpret_cast<float*>(&smem_all[0][0][0][0]), oacc, tid);
      p[0] = m_i;
      p[kThreads] = l_i;
    }
    __syncthreads();
    if (set == 1) return;
    f32x4 o1[NS];
    const float* p = take<HD>(reinterpret_cast<const float*>(&smem_all[0][0][0][0]), o1, tid);
    const float m1 = p[0], m_new = fmaxf(m_i, m1), a0 = expf(m_i - m_new), a1 = expf(m1 - m_new);
    l_i = l_i * a0 + p[kThreads] * a1;
    m_i = m_new;
#pragma unroll
    for (int c = 0; c < NS; ++c) oacc[c] = oacc[c] * a0 + o1[c] * a1;
  }
  const float l = sum4(l_i);
  uint32_t anew = nan_rows(oacc);
  if (q < T_ && !(anew >> lr & 1)) {
    T* row = o + ((int64_t)b * T_ + q) * H * hd + a * hd;
#pragma unroll
    for (int c = 0; c < NS; ++c) put4(row, c * 16 + kg * 4, hd, vec, oacc[c] / l);
    if (kg == 0) lse[((int64_t)b * H + a) * T_ + q] = m_i + logf(l);
  }
  for (; anew; anew &= anew - 1) {
    const int r = qw0 + __builtin_ctz(anew);
    if (r < T_)
      fwd_row<T, HD>(base + r * ld + a * hd, kp, vp, ld, r + 1, hd, scale, o + ((int64_t)b * T_ + r) * H * hd + a * hd,
                     lse + ((int64_t)b * H + a) * T_ + r, lane);
  }
}

// dq_i = sum_{j<=i} ds_ij k_j,  ds_ij = p_ij (dO_i.v_j - delta_i) / sqrt(hd),  p_ij = exp(s_ij - lse_i), and on the way
// delta_i = dO_i.o_i for the dK/dV kernel, which runs after this one
template <class T, int HD>
__global__ __launch_bounds__(kThreads * kSets<HD>) void k_attn_bwd_dq(const T* __restrict__ qkv, const T* __restrict__ o, const float* __restrict__ lse,
                                                          float* __restrict__ delta, const T* __restrict__ dO, int T_, int H, int Hkv,
                                                          int hd, bool vec, float scale, const float* __restrict__ rope_tab,
                                                          T* __restrict__ dqkv) {
  typedef Stored<T> S;
  typedef typename S::Quad Quad;
  constexpr int LD = S::template LD<HD>, NS = HD / 16, SETS = kSets<HD>;
  __shared__ __attribute__((aligned(16))) T smem_all[SETS][2][2][KT * LD];
  const int set = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), tid = threadIdx.x % kThreads;
  const int lane = tid & 63, lr = lane & 15, kg = lane >> 4, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto& smem = smem_all[set];
  const int a = blockIdx.y, b = blockIdx.z, kvh = a / (H / Hkv);
  const int q0 = (int)(gridDim.x - 1 - blockIdx.x) * BQ;
  const int qw0 = q0 + wave * 16, q = qw0 + lr, qc = min(q, T_ - 1);
  const int64_t ld = (int64_t)(H + 2 * Hkv) * hd, row = (int64_t)b * T_ + qc, stat = ((int64_t)b * H + a) * T_ + qc;
  const T* base = qkv + (int64_t)b * T_ * ld;
  const T *kp = base + (H + kvh) * hd, *vp = base + (H + Hkv + kvh) * hd;
  Quad qf[NS], dof[NS];
  f32x4 dq[NS];
  float dlt = 0.f;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int c = s * 16 + kg * 4;
    qf[s] = row4(base + qc * ld + a * hd, c, hd, vec);
    dof[s] = row4(dO + row * H * hd + a * hd, c, hd, vec);
    const f32x4 df = S::floats(dof[s]), of = S::floats(row4(o + row * H * hd + a * hd, c, hd, vec));
#pragma unroll
    for (int e = 0; e < 4; ++e) dlt += df[e] * of[e];
    dq[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  dlt = sum4(dlt);
  if (q < T_ && kg == 0 && set == 0) delta[stat] = dlt;
  const float L = lse[stat];
  const int tiles = (min(T_, q0 + BQ) + KT - 1) / KT;
  Pair<T, HD> in;
  in.load(kp, ld, vp, ld, set * KT, T_, hd, vec, tid);   // a row past the end is zeros
  in.store(smem[0][0], smem[0][1], tid);
  __syncthreads();
  for (int i = 0; i * SETS < tiles; ++i) {   // every wavefront the same number of rounds
    const int kt = i * SETS + set, k0 = kt * KT;
    if (kt + SETS < tiles) in.load(kp, ld, vp, ld, k0 + SETS * KT, T_, hd, vec, tid);
    const T *lk = smem[i & 1][0], *lv = smem[i & 1][1];
    if (kt < tiles && k0 <= qw0 + 15) {
      f32x4 ds[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 st = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const int at = (t * 16 + lr) * LD + s * 16 + kg * 4;
          const Quad fk = *reinterpret_cast<const Quad*>(lk + at), fv = *reinterpret_cast<const Quad*>(lv + at);
          S::dot2(fk, qf[s], st, fv, dof[s], dp);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) ds[t][r] = exp_(st[r] * scale - L) * (dp[r] - dlt) * scale;
      }
      if (k0 + KT - 1 > qw0) {   // not every key is visible to every query
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (k0 + t * 16 + kg * 4 + r > q) ds[t][r] = 0.f;
      }
      S::template times<LD>(ds[0], ds[1], lk, lr, kg, dq);
    }
    if (kt + SETS < tiles) in.store(smem[(i + 1) & 1][0], smem[(i + 1) & 1][1], tid);
    __syncthreads();
  }
  if (SETS == 2) {
    if (set == 1) give<HD>(reinterpret_cast<float*>(&smem_all[0][0][0][0]), dq, tid);
    __syncthreads();
    if (set == 1) return;
    f32x4 o1[NS];
    take<HD>(reinterpret_cast<const float*>(&smem_all[0][0][0][0]), o1, tid);
#pragma unroll
    for (int c = 0; c < NS; ++c) dq[c] += o1[c];
  }
  uint32_t anew = nan_rows(dq);
  if (q < T_ && !(anew >> lr & 1)) {
#pragma unroll
    for (int c = 0; c < NS; ++c) {
      if (rope_tab) unrotate4(dq[c], rope_tab, q, c * 16 + kg * 4, hd);
      put4(dqkv + row * ld + a * hd, c * 16 + kg * 4, hd, vec, dq[c]);
    }
  }
  for (; anew; anew &= anew - 1) {
    const int i = __builtin_ctz(anew), r = qw0 + i;
    const int64_t at = (int64_t)b * T_ + r;
    if (r < T_)
      dq_row<T, HD>(base + r * ld + a * hd, dO + at * H * hd + a * hd, kp, vp, ld, r + 1, hd, scale, __shfl(L, i), __shfl(dlt, i), rope_tab,
                    dqkv + at * ld + a * hd, lane);
  }
}

// dk_j = sum_a sum_{i>=j} ds_ij q_i ; dv_j = sum_a sum_{i>=j} p_ij dO_i   (a over the q heads of this kv head)
template <class T, int HD>
__global__ __launch_bounds__(kThreads * kSets<HD>) void k_attn_bwd_dkv(const T* __restrict__ qkv, const float* __restrict__ lse,
                                                           const float* __restrict__ delta, const T* __restrict__ dO, int T_, int H,
                                                           int Hkv, int hd, bool vec, float scale, const float* __restrict__ rope_tab,
                                                           T* __restrict__ dqkv) {
  typedef Stored<T> S;
  typedef typename S::Quad Quad;
  constexpr int LD = S::template LD<HD>, NS = HD / 16, SETS = kSets<HD>;
  __shared__ __attribute__((aligned(16))) T smem_all[SETS][2][2][KT * LD];
  __shared__ __attribute__((aligned(16))) float s_lse_all[SETS][2][KT], s_dlt_all[SETS][2][KT];
  const int set = __builtin_amdgcn_readfirstlane(threadIdx.x / kThreads), tid = threadIdx.x % kThreads;
  const int lane = tid & 63, lr = lane & 15, kg = lane >> 4, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto& smem = smem_all[set];
  auto &s_lse = s_lse_all[set], &s_dlt = s_dlt_all[set];
  const int kvh = blockIdx.y, b = blockIdx.z, rep = H / Hkv;
  const int k0 = blockIdx.x * BQ, kw0 = k0 + wave * 16, key = kw0 + lr, kc = min(key, T_ - 1);
  const int64_t ld = (int64_t)(H + 2 * Hkv) * hd, ldo = (int64_t)H * hd;
  const T* base = qkv + (int64_t)b * T_ * ld;
  Quad kf[NS], vf[NS];
  f32x4 dk[NS], dv[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    kf[s] = row4(base + kc * ld + (H + kvh) * hd, s * 16 + kg * 4, hd, vec);
    vf[s] = row4(base + kc * ld + (H + Hkv + kvh) * hd, s * 16 + kg * 4, hd, vec);
    dk[s] = dv[s] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // the walk: for every query head of this kv head, the query tiles from the workgroup's first key on
  const int t0 = k0 / KT, nt = (T_ + KT - 1) / KT - t0, steps = nt * rep;
  Pair<T, HD> in;
  float in_lse = 0.f, in_dlt = 0.f;
  auto fetch = [&](int step) {
    const int a = kvh * rep + step / nt, r0 = (t0 + step % nt) * KT;
    in.load(base + a * hd, ld, dO + (int64_t)b * T_ * ldo + a * hd, ldo, r0, T_, hd, vec, tid);
    if (tid < KT && r0 + tid < T_) {
      const int64_t at = ((int64_t)b * H + a) * T_ + r0 + tid;
      in_lse = lse[at];
      in_dlt = delta[at];
    }
  };
  auto put = [&](int buf) {
    in.store(smem[buf][0], smem[buf][1], tid);
    if (tid < KT) { s_lse[buf][tid] = in_lse; s_dlt[buf][tid] = in_dlt; }
  };
  if (set < steps) fetch(set), put(0);
  __syncthreads();
  for (int i = 0; i * SETS < steps; ++i) {
    const int step = i * SETS + set, buf = i & 1;
    if (step + SETS < steps) fetch(step + SETS);
    const int qs = (t0 + step % nt) * KT;
    const T *lq = smem[buf][0], *lo = smem[buf][1];
    if (step < steps && qs + KT - 1 >= kw0) {   // some query of the tile sees a key of this wavefront
      f32x4 p[2], ds[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        f32x4 st = {0.f, 0.f, 0.f, 0.f}, dp = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const int at = (t * 16 + lr) * LD + s * 16 + kg * 4;
          const Quad fq = *reinterpret_cast<const Quad*>(lq + at), fo = *reinterpret_cast<const Quad*>(lo + at);
          S::dot2(fq, kf[s], st, fo, vf[s], dp);
        }
        const f32x4 L = *reinterpret_cast<const f32x4*>(&s_lse[buf][t * 16 + kg * 4]);
        const f32x4 D = *reinterpret_cast<const f32x4*>(&s_dlt[buf][t * 16 + kg * 4]);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          p[t][r] = exp_(st[r] * scale - L[r]);
          ds[t][r] = p[t][r] * (dp[r] - D[r]) * scale;
        }
      }
      if (qs < kw0 + 15 || qs + KT > T_) {   // not every query sees every key, or there are none
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            const int q = qs + t * 16 + kg * 4 + r;
            if (q < key || q >= T_) p[t][r] = ds[t][r] = 0.f;
          }
      }
      S::template times<LD>(p[0], p[1], lo, lr, kg, dv);
      S::template times<LD>(ds[0], ds[1], lq, lr, kg, dk);
    }
    if (step + SETS < steps) put(buf ^ 1);
    __syncthreads();
  }
  if (SETS == 2) {   // dk over in the first half of the buffers, dv in the second
    float* half = reinterpret_cast<float*>(&smem_all[SETS - 1][0][0][0]);
    if (set == 1) {
      give<HD>(reinterpret_cast<float*>(&smem_all[0][0][0][0]), dk, tid);
      give<HD>(half, dv, tid);
    }
    __syncthreads();
    if (set == 1) return;
    f32x4 o1[NS], o2[NS];
    take<HD>(reinterpret_cast<const float*>(&smem_all[0][0][0][0]), o1, tid);
    take<HD>(half, o2, tid);
#pragma unroll
    for (int c = 0; c < NS; ++c) {
      dk[c] += o1[c];
      dv[c] += o2[c];
    }
  }
  uint32_t anew = nan_rows(dk) | nan_rows(dv);
  if (key < T_ && !(anew >> lr & 1)) {
    T* row = dqkv + ((int64_t)b * T_ + key) * ld;
#pragma unroll
    for (int c = 0; c < NS; ++c) {
      if (rope_tab) unrotate4(dk[c], rope_tab, key, c * 16 + kg * 4, hd);
      put4(row + (H + kvh) * hd, c * 16 + kg * 4, hd, vec, dk[c]);
      put4(row + (H + Hkv + kvh) * hd, c * 16 + kg * 4, hd, vec, dv[c]);
    }
  }
  for (; anew; anew &= anew - 1) {
    const int r = kw0 + __builtin_ctz(anew);
    if (r >= T_) continue;
    T* row = dqkv + ((int64_t)b * T_ + r) * ld;
    const int64_t head = ((int64_t)b * H + kvh * rep) * T_;
    dkv_row<T, HD>(base + r * ld + (H + kvh) * hd, base + r * ld + (H + Hkv + kvh) * hd, base + kvh * rep * hd,
                   dO + (int64_t)b * T_ * ldo + kvh * rep * hd, lse + head, delta + head, ld, ldo, rep, r, T_, hd, scale, rope_tab,
                   row + (H + kvh) * hd, row + (H + Hkv + kvh) * hd, lane);
  }
}

// every row and head starts on a four-element boundary
template <class T>
bool rows_of_four(int hd, const void* a, const void* b, const void* c, const void* d) {
  return hd % 4 == 0 && (((uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)d) & (4 * sizeof(T) - 1)) == 0;
}

#define SP_BY_HD(GO)                                                                                        \
  do {                                                                                                      \
    if (hd <= 32) GO(32); else if (hd <= 48) GO(48); else if (hd <= 64) GO(64); else if (hd <= 96) GO(96);  \
    else if (hd <= 128) GO(128); else GO(256);                                                              \
  } while (0)

template <class T>
void fwd_t(hipStream_t s, int B, int T_, int H, int Hkv, int hd, const void* qkv, void* o, float* lse) {
  const bool vec = rows_of_four<T>(hd, qkv, o, nullptr, nullptr);
  const float scale = 1.0f / sqrtf((float)hd);
#define SP_GO(HD) hipLaunchKernelGGL((k_attn_fwd<T, HD>), dim3((T_ + BQ - 1) / BQ, H, B), dim3(kThreads * kSets<HD>), 0, s, (const T*)qkv, T_, H, Hkv, hd, vec, scale, (T*)o, lse)
  SP_BY_HD(SP_GO);
#undef SP_GO
}

template <class T>
void bwd_t(hipStream_t s, int B, int T_, int H, int Hkv, int hd, const void* qkv, const void* o, const float* lse, const void* dO,
           void* dqkv, float* delta, const float* rope_tab) {
  const bool vec = rows_of_four<T>(hd, qkv, o, dO, dqkv);
  const float scale = 1.0f / sqrtf((float)hd);
  const int nb = (T_ + BQ - 1) / BQ;
#define SP_GO(HD)                                                                                                              \
  do {                                                                                                                         \
    hipLaunchKernelGGL((k_attn_bwd_dq<T, HD>), dim3(nb, H, B), dim3(kThreads * kSets<HD>), 0, s, (const T*)qkv, (const T*)o, lse, delta,    \
                       (const T*)dO, T_, H, Hkv, hd, vec, scale, rope_tab, (T*)dqkv);                                          \
    hipLaunchKernelGGL((k_attn_bwd_dkv<T, HD>), dim3(nb, Hkv, B), dim3(kThreads * kSets<HD>), 0, s, (const T*)qkv, lse, delta, (const T*)dO, \
                       T_, H, Hkv, hd, vec, scale, rope_tab, (T*)dqkv);                                                        \
  } while (0)
  SP_BY_HD(SP_GO);
#undef SP_GO
}

int check_attn(int B, int T, int H, int Hkv, int hd) {
  if (B <= 0 || T <= 0 || H <= 0 || Hkv <= 0 || hd <= 0 || H % Hkv) return fail(SP_EINVAL, "attention: bad shape");
  if (hd > kMaxHd) return fail(SP_EINVAL, "attention: head dimension above 256");
  if (B > 65535 || H > 65535) return fail(SP_EINVAL, "attention: batch or head count above 65535");
  return SP_OK;
}

}  // namespace

int attention_fwd(hipStream_t s, int dtype, int B, int T, int H, int Hkv, int hd, const void* qkv, void* o, float* lse) {
  int rc = check_attn(B, T, H, Hkv, hd);
  if (rc) return rc;
  if (!qkv || !o || !lse) return fail(SP_EINVAL, "attention: null operand");
  const bool fast = dtype == SP_BF16 && attention_flash_supported(B, T, H, Hkv, hd);
  const int pi = prof_start(fast ? PROF_ATTN_FWD : PROF_ATTN_PLAIN, s);
  if (fast) attention_flash_fwd(s, B, T, H, Hkv, hd, qkv, o, lse);
  else if (dtype == SP_BF16) fwd_t<bf16>(s, B, T, H, Hkv, hd, qkv, o, lse);
  else fwd_t<float>(s, B, T, H, Hkv, hd, qkv, o, lse);
  prof_stop(pi, s, 2.0 * (double)B * H * (double)T * (T + 1) * hd);   // QK^T and PV over the causal half
  return SP_OK;
}

int attention_bwd(hipStream_t s, int dtype, int B, int T, int H, int Hkv, int hd, const void* qkv, const void* o,
                  const float* lse, const void* do_, void* dqkv, float* delta, const float* rope_tab) {
  int rc = check_attn(B, T, H, Hkv, hd);
  if (rc) return rc;
  if (!qkv || !o || !lse || !do_ || !dqkv || !delta) return fail(SP_EINVAL, "attention: null operand");
  if (dtype == SP_BF16 && attention_flash_supported(B, T, H, Hkv, hd)) {
    attention_flash_bwd(s, B, T, H, Hkv, hd, qkv, o, lse, do_, dqkv, delta, rope_tab);
    return SP_OK;
  }
  const int pi = prof_start(PROF_ATTN_PLAIN, s);
  if (dtype == SP_BF16) bwd_t<bf16>(s, B, T, H, Hkv, hd, qkv, o, lse, do_, dqkv, delta, rope_tab);
  else bwd_t<float>(s, B, T, H, Hkv, hd, qkv, o, lse, do_, dqkv, delta, rope_tab);
  prof_stop(pi, s, 4.0 * (double)B * H * (double)T * (T + 1) * hd);
  return SP_OK;
}

}  // namespace sp
