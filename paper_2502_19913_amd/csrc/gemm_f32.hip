// Float matrix products on the CDNA4 matrix cores (v_mfma_f32_16x16x4_f32: float operands, float sums, 1/16 of the
// bf16 rate), any shape and alignment.  They carry the float mode.
//
//   op 0  C[M,N]  = A[M,K] B[N,K]^T (+R)   A, B k-contiguous
//   op 1  C[M,N]  = A[M,K] B[K,N]          B k-strided
//   op 2  C[M,N] += A[K,M]^T B[K,N]        both k-strided; added atomically
//
// The instruction's k-slots may stand for any four k, so lane group kg = lane / 16 holds k = 4 kg .. 4 kg + 3 of a
// group of 16 and four instructions take one element each: a fragment of 16 rows x 16 k of a k-contiguous operand
// is one 16-byte read.  For ops 0 and 1 the tile of B is the instruction's row operand, so a lane ends with four
// consecutive output columns of one row (16-byte stores, and whole rotary pairs for the epilogue); for op 2 the
// tile of A is, so that a wavefront's atomics cover 64 contiguous bytes of four rows.
//
// Kernels:
//   k_gemm_f32           tiles of 128 x 128 or 64 x 64, four wavefronts, operands staged through LDS (global -> registers
//                        one step ahead -> the other of two LDS buffers, one barrier per step of 32 k).  The matrix
//                        instruction needs 32 cycles for 2 x 64 floats of operands, so LDS and memory keep up easily and
//                        the kernel is bound by the matrix cores.
//   k_gemm_f32_small     for products too small to fill the chip with those: tiles of 32 x 32, four wavefronts with a block
//                        of 16 x 16 each, eight steps in flight.  The time is one chain of latencies.
// Every entry is summed in one order (runs of 64 k), with the same instructions, in both: the tile of ops 0 and 1 follows the
// number of rows, and a microbatch's rows must not depend on how many microbatches share its group; a weight gradient is
// added with one atomic per entry and launch, so that it repeats to the bit.
// Measured against the vector-unit kernel they replaced (64 x 64 tiles, products and sums one lane at a time), us per
// launch: op 0 3072 x 3072 x 1024 424 -> 191 (101 TFLOP/s of the 157 the cores peak at), op 1 2048 x 1024 x 5632 1109 ->
// 235, op 2 864 x 288 x 4096 893 -> 31, and of the small ones op 0 128 x 288 x 768 95 -> 8.8, op 1 128 x 288 x 1536
// 191 -> 13, most others at 8 (the launch).
#include <algorithm>
#include <type_traits>

#include "devutil.h"
#include "internal.h"

namespace sp {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int BK = 32;
constexpr int kThreads = 256;

// Every kernel sums runs of 64 k and adds them up in turn: one chain of K / 4 instructions is off by 1.8e-8 sqrt(K) (2-norm,
// unit normals), 5.0e-7 at K = 768 and 1.1e-6 at 4096, the runs by 1.6e-7 and 2.1e-7 (runs of 128 2.1e-7 and 2.3e-7, of 32
// 1.4e-7 and 2.3e-7).  It takes one more set of accumulators.  With the loop written out over the two steps of a run, the first
// of which starts from zero, it costs nothing: us, one chain / runs, op 0 2048 x 288 x 768 22.7 / 21.1, 3072 x 1024 x 2816
// 168 / 161 (64-tiles), 4096 x 4096 x 1024 288 / 291, 2048 x 2048 x 2048 157 / 164 (128-tiles); 500M stage 7.18 / 7.17 ms
// (7.25 with a loop over single steps).
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

// Memory row of B that belongs at row t of a SwiGLU tile of TN rows made of shares of WN: the first half of a share
// holds gate rows, the second half the up rows of the same features (h = N / 2 features).  -1: past the end.
template <int TN, int WN>
__device__ __forceinline__ int swiglu_row(int tn, int t, int h) {
  const int w = t / WN, in = t % WN, f = tn * (TN / 2) + w * (WN / 2) + in % (WN / 2);
  return f < h ? (in < WN / 2 ? f : h + f) : -1;
}

__device__ __forceinline__ void end_run(f32x4& sum, f32x4& acc) {
  sum += acc;
  acc = f32x4{0.f, 0.f, 0.f, 0.f};
}

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

// One operand's tile of T rows (or columns) x BK: memory -> registers -> LDS -> fragments.  LDS rows are padded by
// four floats: [T][BK + 4] k-contiguous (16-byte fragment reads of 16 rows fall in different banks), [BK][T + 4]
// k-strided (the four k rows a read touches start 16 banks apart).
template <bool KS, int T, bool VEC>
struct Tile {
  static constexpr int N4 = T * BK / 4 / kThreads;
  static constexpr int kFloats = KS ? BK * (T + 4) : T * (BK + 4);
  f32x4 r[N4];
  // rows: extent of the tile's own dimension in memory; row_of maps a tile row to a memory row or -1 (k-contiguous)
  template <class RowOf>
  __device__ __forceinline__ void load(const float* X, int rows, int ld, int x0, int k0, int kend, int tid, RowOf row_of) {
#pragma unroll
    for (int j = 0; j < N4; ++j) {
      const int i = tid + kThreads * j;
      if (KS) {
        const int k = k0 + i / (T / 4), x = x0 + i % (T / 4) * 4;
        r[j] = load4<VEC>(X + (int64_t)k * ld + x, k < kend ? rows - x : 0);
      } else {
        const int row = row_of(i / (BK / 4)), k = k0 + i % (BK / 4) * 4;
        r[j] = load4<VEC>(X + (int64_t)row * ld + k, row >= 0 ? kend - k : 0);
      }
    }
  }
  __device__ __forceinline__ void store(float* lds, int tid) const {
#pragma unroll
    for (int j = 0; j < N4; ++j) {
      const int i = tid + kThreads * j;
      const int at = KS ? i / (T / 4) * (T + 4) + i % (T / 4) * 4 : i / (BK / 4) * (BK + 4) + i % (BK / 4) * 4;
      *reinterpret_cast<f32x4*>(lds + at) = r[j];
    }
  }
  // rows base .. base+15, k 16 s + 4 kg + {0..3}
  static __device__ __forceinline__ f32x4 frag(const float* lds, int base, int s, int lr, int kg) {
    if (!KS) return *reinterpret_cast<const f32x4*>(lds + (base + lr) * (BK + 4) + s * 16 + kg * 4);
    const float* p = lds + (s * 16 + kg * 4) * (T + 4) + base + lr;
    return f32x4{p[0], p[T + 4], p[2 * (T + 4)], p[3 * (T + 4)]};
  }
};

template <int OP, int EPI, int T, bool VEC>
__global__ __launch_bounds__(kThreads, 2) void k_gemm_f32(Args g) {
  constexpr bool AS = OP == 2, BS = OP != 0;
  typedef Tile<AS, T, VEC> TA;
  typedef Tile<BS, T, VEC> TB;
  constexpr int W = T / 2, NB = W / 16;   // a wavefront's share (2 x 2 wavefronts), in blocks of 16 each way
  __shared__ __attribute__((aligned(16))) float smem[2 * (TA::kFloats + TB::kFloats)];
  constexpr int kStage = TA::kFloats + TB::kFloats;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  int tm, tn;
  tile_of(g, xcd_major(blockIdx.x, gridDim.x), tm, tn);
  const int m0 = tm * T, n0 = tn * T, steps = (g.K + BK - 1) / BK;

  f32x4 acc[NB][NB], sum[NB][NB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < NB; ++i) sum[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto a_row = [&](int t) { return m0 + t < g.M ? m0 + t : -1; };
  auto b_row = [&](int t) {
    if (EPI == kEpiSwiglu) return swiglu_row<T, W>(tn, t, g.N / 2);
    return n0 + t < g.N ? n0 + t : -1;
  };
  TA ta;
  TB tb;
  auto fetch = [&](int s) {
    ta.load(g.A, g.M, AS ? g.M : g.K, m0, s * BK, g.K, tid, a_row);
    tb.load(g.B, g.N, BS ? g.N : g.K, n0, s * BK, g.K, tid, b_row);
  };
  auto put = [&](int s) {
    float* st = smem + (s & 1) * kStage;
    ta.store(st, tid);
    tb.store(st + TA::kFloats, tid);
  };
  fetch(0);
  put(0);
  __syncthreads();
  auto step = [&](int s, auto begins) {   // begins: a run, whose first products need no sum to be added to
    if (s + 1 < steps) fetch(s + 1);
    const float* la = smem + (s & 1) * kStage;
    const float* lb = la + TA::kFloats;
#pragma unroll
    for (int q = 0; q < BK / 16; ++q) {
      f32x4 fa[NB], fb[NB];
#pragma unroll
      for (int j = 0; j < NB; ++j) fa[j] = TA::frag(la, wm * W + j * 16, q, lr, kg);
#pragma unroll
      for (int i = 0; i < NB; ++i) fb[i] = TB::frag(lb, wn * W + i * 16, q, lr, kg);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const f32x4 c = decltype(begins)::value && q == 0 && e == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[j][i];
            acc[j][i] = OP == 2 ? __builtin_amdgcn_mfma_f32_16x16x4f32(fa[j][e], fb[i][e], c, 0, 0, 0)
                                : __builtin_amdgcn_mfma_f32_16x16x4f32(fb[i][e], fa[j][e], c, 0, 0, 0);
          }
    }
    if (s + 1 < steps) put(s + 1);   // into the buffer that every wavefront left before the last barrier
    if (!decltype(begins)::value || s + 1 == steps)
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < NB; ++i) sum[j][i] += acc[j][i];
    __syncthreads();
  };
  static_assert(kRun == 2, "a step that begins a run and one that ends it");
  for (int s = 0; s < steps; s += 2) {
    step(s, std::true_type());
    if (s + 1 < steps) step(s + 1, std::false_type());
  }
  if (OP == 2) {
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int n = n0 + wn * W + i * 16 + lr;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0 + wm * W + j * 16 + kg * 4 + r;
          if (m < g.M && n < g.N) unsafeAtomicAdd(g.C + (int64_t)m * g.N + n, sum[j][i][r]);
        }
      }
  } else if (EPI == kEpiSwiglu) {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int m = m0 + wm * W + j * 16 + lr;
      if (m < g.M) {
#pragma unroll
        for (int i = 0; i < NB / 2; ++i)
          emit_swiglu<VEC>(g, m, tn * (T / 2) + wn * (W / 2) + i * 16 + kg * 4, sum[j][i], sum[j][i + NB / 2]);
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int m = m0 + wm * W + j * 16 + lr;
      if (m < g.M) {
#pragma unroll
        for (int i = 0; i < NB; ++i) emit<OP, EPI, VEC>(g, m, n0 + wn * W + i * 16 + kg * 4, sum[j][i]);
      }
    }
  }
}

// One thread's quad of a step's BK x T tile for the kernel below: T = 32 rows of 8 quads (k-contiguous) or 32 k of T / 4
// quads (k-strided), on its way from memory to LDS.  A quad past an edge reads the last one inside again, so that loads
// need no branches: past the end of k `masked` makes it zeros, past the last row or column nothing of it is stored.
template <bool KS, bool VEC>
struct Quad {
  const float* p;   // start of the quad's row (k-contiguous) or of its first column (k-strided)
  int kq, dx[3];    // its first k inside a step; k-strided and element-wise: where its other columns are
  __device__ __forceinline__ void init(const float* X, int row, int ld, int k) { p = X + (int64_t)row * ld; kq = k; }
  __device__ __forceinline__ void init_cols(const float* X, int col, int cols, int k) {
    const int x = VEC ? min(col, cols - 4) : min(col, cols - 1);
    p = X + x;
    kq = k;
#pragma unroll
    for (int e = 1; e < 4; ++e) dx[e - 1] = min(col + e, cols - 1) - x;
  }
  __device__ __forceinline__ f32x4 load(int k0, int K, int ld) const {
    const int k = k0 + kq;
    if (KS) {
      const float* q = p + (int64_t)min(k, K - 1) * ld;
      if (VEC) return *reinterpret_cast<const f32x4*>(q);
      return f32x4{q[0], q[dx[0]], q[dx[1]], q[dx[2]]};
    }
    if (VEC) return *reinterpret_cast<const f32x4*>(p + min(k, K - 4));
    return f32x4{p[min(k, K - 1)], p[min(k + 1, K - 1)], p[min(k + 2, K - 1)], p[min(k + 3, K - 1)]};
  }
  __device__ __forceinline__ f32x4 masked(f32x4 v, int k0, int K) const {
    const int left = K - (k0 + kq);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if ((KS || VEC ? 0 : e) >= left) v[e] = 0.f;
    return v;
  }
};

// Tiles of 32 x 32 (SwiGLU: 32 rows x 32 features): a wavefront owns a block of 16 x 16 (SwiGLU: of gate and
// of up columns) over the whole reduction and sums it in the order and with the instructions of k_gemm_f32, so that a
// row has the same bits whatever kernel the number of rows leads to.  That chain of K / 4 dependent matrix instructions
// of 32 cycles (and the launch) bounds it: U steps of 32 k are in flight from memory (registers), one in LDS ahead of the
// one whose fragments are read, and that one ahead of the one being multiplied; one barrier per step.  Through LDS because
// fragments read straight from memory touch 16 half cache lines an instruction, about 60 cycles each: op 0, us, staged /
// straight in the order of k / straight with k divided among eight wavefronts as it was before: 128 x 288 x 1536 15.0 /
// 25.0 / 16.4, 1024 x 288 x 768 12.6 / 27.7 / 15.9, 64 x 1024 x 2816 24.9 / 40.2 / 28.2.  Op 2, one sum / the reduction cut
// over workgroups and wavefronts and added in no fixed order as it was before: 864 x 288 x 512 7.8 / 12.3, x 2048 17.4 /
// 18.0, x 4096 30.9 / 29.3, 1536 x 288 x 999 16.1 / 23.6, 4096 x 288 x 4096 112 / 165, but 288 x 288 x 4096 30.5 / 14.4.
template <int OP, int EPI, bool VEC>
__global__ __launch_bounds__(kThreads) void k_gemm_f32_small(Args g) {
  constexpr bool AS = OP == 2, BS = OP != 0;
  constexpr int T = 32, NB = EPI == kEpiSwiglu ? 2 : 1, U = 8;
  typedef Tile<AS, T, VEC> TA;
  typedef Tile<BS, T, VEC> TB;
  static_assert(TA::N4 == 1, "one quad of each tile per thread");
  constexpr int kStage = TA::kFloats + NB * TB::kFloats;
  __shared__ __attribute__((aligned(16))) float smem[2 * kStage];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 1, wn = wave & 1;
  int tm, tn;
  tile_of(g, xcd_major(blockIdx.x, gridDim.x), tm, tn);
  const int m0 = tm * T, n0 = tn * T, K = g.K, steps = (K + BK - 1) / BK;
  const int cols = EPI == kEpiSwiglu ? g.N / 2 : g.N, lda = AS ? g.M : K, ldb = BS ? g.N : K;
  f32x4 acc[NB], sum[NB];
#pragma unroll
  for (int i = 0; i < NB; ++i) acc[i] = sum[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (steps > 0) {
    Quad<AS, VEC> qa;
    Quad<BS, VEC> qb[NB];
    if (AS) qa.init_cols(g.A, m0 + tid % 8 * 4, g.M, tid / 8);
    else qa.init(g.A, min(m0 + tid / 8, g.M - 1), K, tid % 8 * 4);
#pragma unroll
    for (int i = 0; i < NB; ++i) {
      if (BS) qb[i].init_cols(g.B, n0 + tid % 8 * 4, cols, tid / 8);
      else qb[i].init(g.B, i * cols + min(n0 + tid / 8, cols - 1), K, tid % 8 * 4);
    }
    f32x4 ra[U], rb[U][NB];
    auto fetch = [&](int s, int u) {   // past the last step: the last one again
      const int k0 = min(s, steps - 1) * BK;
      ra[u] = qa.load(k0, K, lda);
#pragma unroll
      for (int i = 0; i < NB; ++i) rb[u][i] = qb[i].load(k0, K, ldb);
      __builtin_amdgcn_sched_barrier(0);   // loads stay in the order they are waited for
    };
    auto put = [&](int s, int u) {
      float* st = smem + (s & 1) * kStage;
      const int at = tid / 8 * (BK + 4) + tid % 8 * 4;   // BK = T: the same for either order
      static_assert(BK == T, "tile rows of the two orders");
      *reinterpret_cast<f32x4*>(st + at) = qa.masked(ra[u], s * BK, K);
#pragma unroll
      for (int i = 0; i < NB; ++i) *reinterpret_cast<f32x4*>(st + TA::kFloats + i * TB::kFloats + at) = qb[i].masked(rb[u][i], s * BK, K);
    };
    struct Frags { f32x4 a[BK / 16], b[BK / 16][NB]; };
    auto read = [&](int s) {
      const float* st = smem + (s & 1) * kStage;
      Frags f;
#pragma unroll
      for (int q = 0; q < BK / 16; ++q) {
        f.a[q] = TA::frag(st, wm * 16, q, lr, kg);
#pragma unroll
        for (int i = 0; i < NB; ++i) f.b[q][i] = TB::frag(st + TA::kFloats + i * TB::kFloats, wn * 16, q, lr, kg);
      }
      return f;
    };
#pragma unroll
    for (int u = 0; u < U; ++u) fetch(u, u);
    put(0, 0);
    fetch(U, 0);
    put(1, 1);
    fetch(U + 1, 1);
    __syncthreads();
    Frags now = read(0);
    __syncthreads();
    // in LDS: step s + 1 and, from the middle of the step on, s + 2; on the way: the next U
    static_assert(U % kRun == 0, "runs end at fixed places of a round of U steps");
    auto step = [&](int s, int u, bool more, bool ends) {   // u = (s + 2) % U; ends: a run
      const Frags next = read(s + 1);
#pragma unroll
      for (int q = 0; q < BK / 16; ++q) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < NB; ++i)
            acc[i] = OP == 2 ? __builtin_amdgcn_mfma_f32_16x16x4f32(now.a[q][e], now.b[q][i][e], acc[i], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_16x16x4f32(now.b[q][i][e], now.a[q][e], acc[i], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (q == 0) {
          put(s + 2, u);
          if (more) fetch(s + 2 + U, u);
        }
      }
      if (ends)
#pragma unroll
        for (int i = 0; i < NB; ++i) end_run(sum[i], acc[i]);
      now = next;
      __syncthreads();
    };
    int s = 0;
    for (; s + U <= steps; s += U)
#pragma unroll
      for (int u = 0; u < U; ++u) step(s + u, (u + 2) % U, true, u % kRun == kRun - 1);
#pragma unroll
    for (int u = 0; u < U - 1; ++u)   // the rest is on its way
      if (s + u < steps) step(s + u, (u + 2) % U, false, u % kRun == kRun - 1);
#pragma unroll
    for (int i = 0; i < NB; ++i) sum[i] += acc[i];
  }
  if (OP == 2) {
    const int n = n0 + wn * 16 + lr;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm * 16 + kg * 4 + r;
      if (m < g.M && n < g.N) unsafeAtomicAdd(g.C + (int64_t)m * g.N + n, sum[0][r]);
    }
    return;
  }
  const int m = m0 + wm * 16 + lr, n = n0 + wn * 16 + kg * 4;
  if (m >= g.M) return;
  if (EPI == kEpiSwiglu) emit_swiglu<VEC>(g, m, n, sum[0], sum[NB - 1]);
  else emit<OP, EPI, VEC>(g, m, n, sum[0]);
}

inline bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

}  // namespace

// Tile and its grid for a product.
struct F32Shape { int tile, tm, tn; };
static F32Shape choose_f32(int op, int64_t M, int64_t N, int64_t K, int epi) {
  const int64_t out = epi == kEpiSwiglu ? N / 2 : N;   // width of one stored run of columns
  auto at = [&](int t) {
    const int w = epi == kEpiSwiglu && t != 32 ? t / 2 : t;   // stored columns a tile covers of one run
    return F32Shape{t, (int)((M + t - 1) / t), (int)((out + w - 1) / w)};
  };
  auto tiles = [&](int t) { return (int64_t)at(t).tm * at(t).tn; };
  // Every CU runs its tiles at the rate of its matrix cores, so a product takes as long as the CU with the most
  // output: ceil(tiles / CUs) tiles.  Tiles of 64 divide the work more evenly; tiles of 128 read half as much per flop
  // and win where both come out alike (measured within 5 % of each other there).
  const int64_t cus = cu_count(), t128 = tiles(128), t64 = tiles(64);
  const int64_t load128 = (t128 + cus - 1) / cus * 4, load64 = (t64 + cus - 1) / cus;
  int tile = load128 * 100 <= load64 * 105 ? 128 : (t64 >= 128 ? 64 : 32);
  if (op == 2) {
    // A weight gradient is few tiles and a long reduction, and is not cut along k over workgroups: their sums would be added
    // in the order in which they end, and no two passes of the mode that gradients are checked in would agree.  Tiles of 32
    // keep their loads in flight and divide best, but read twice as much and take a tenth longer on a full chip: us, 32 / 64 /
    // 128, 4096 x 288 x 2048 59 / 83 / 162, 1536 x 1024 x 1024 38 / 44 / 85, 2048 x 1024 x 3072 133 / 127 / 242, 3072 x 1024
    // x 2048 133 / 120 / 167, 2048 x 2048 x 4096 342 / 308 / 325, 4096 x 4096 x 1024 369 / 308 / 294.  At one tile of 64 a CU
    // (1024 x 1024 x 2048 47 / 60) the stage of the 500M shape is 0.4 % faster with 64, beside the other products.
    const int64_t load32 = (tiles(32) + cus - 1) / cus;
    if (tile == 128 && t128 < 2 * cus) tile = 64;
    if (tile != 128) tile = load32 * 110 <= load64 * 400 ? 32 : 64;
  }
  return at(tile);
}

GemmShape gemm_f32_shape(int op, int64_t M, int64_t N, int64_t K, int epi) {
  const F32Shape c = choose_f32(op, M, N, K, epi);
  return {c.tile, c.tm * c.tn, c.tm * c.tn};
}

// epi as in gemm_mfma: 0 plain (R optional), 1 rotary, 2 SwiGLU (N = 2h, aux = act), 3 SwiGLU backward (N = h, R =
// gate|up, C = d(gate)|d(up)).
void gemm_f32(hipStream_t s, int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C, const void* R,
              const RopeArgs* rope, int epi, void* aux) {
  Args g{(const float*)A, (const float*)B, (const float*)R, (float*)C, (float*)aux, (int)M, (int)N, (int)K, 0, 0,
         rope ? *rope : RopeArgs{nullptr, 1, 2, 0}};
  if (rope) epi = kEpiRope;
  const int64_t out = epi == kEpiSwiglu ? N / 2 : N;   // width of one stored run of columns
  const bool vec = al16(A) && al16(B) && al16(C) && al16(R) && al16(aux) && out % 4 == 0 && (op == 2 ? M % 4 == 0 : K % 4 == 0);
  const F32Shape c = choose_f32(op, M, N, K, epi);
  const int tile = c.tile;
  g.tiles_m = c.tm;
  g.tiles_n = c.tn;
  const dim3 grid((unsigned)(c.tm * c.tn));
#define SP_GO(OP, EPI, VEC)                                                                                             \
  do {                                                                                                                  \
    if (tile == 128) hipLaunchKernelGGL((k_gemm_f32<OP, EPI, 128, VEC>), grid, dim3(kThreads), 0, s, g);                \
    else if (tile == 64) hipLaunchKernelGGL((k_gemm_f32<OP, EPI, 64, VEC>), grid, dim3(kThreads), 0, s, g);             \
    else hipLaunchKernelGGL((k_gemm_f32_small<OP, EPI, VEC>), grid, dim3(kThreads), 0, s, g);                           \
  } while (0)
#define SP_GO_V(OP, EPI) do { if (vec) SP_GO(OP, EPI, true); else SP_GO(OP, EPI, false); } while (0)
  if (op == 0 && epi == kEpiRope) SP_GO_V(0, kEpiRope);
  else if (op == 0 && epi == kEpiSwiglu) SP_GO_V(0, kEpiSwiglu);
  else if (op == 0) SP_GO_V(0, kEpiPlain);
  else if (op == 1 && epi == kEpiSwigluBwd) SP_GO_V(1, kEpiSwigluBwd);
  else if (op == 1) SP_GO_V(1, kEpiPlain);
  else SP_GO_V(2, kEpiPlain);
#undef SP_GO_V
#undef SP_GO
}

}  // namespace sp
