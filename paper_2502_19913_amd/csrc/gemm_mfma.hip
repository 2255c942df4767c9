// bf16 matrix products on the CDNA4 matrix cores, float accumulation.  v_mfma_f32_16x16x32_bf16 sustains more flops
// per watt on random data than the 32x32x16 form (the chip is power-limited here); op 2 in 256-tiles keeps
// v_mfma_f32_32x32x16_bf16, whose accumulator layout gives wider atomics.
//
// One workgroup of 8 wavefronts owns a 256x256 tile of the output (k_gemm_mfma), or a 128x128 or 64x64 tile where those
// occupy the CUs better (k_gemm_ring; choose_shape decides), and walks the reduction dimension in steps of 64.  Operand
// tiles go from memory straight into LDS (buffer loads with the LDS modifier: no staging registers, no LDS stores; the
// hardware range check returns zero past the end of an operand, so ragged edges need no branches).  The
// 256-tile fills the CU's 160 KB of LDS alone (two tiles of A, three of B) and
// runs the alternating-phase loop described where it stands: the two wavefronts of a SIMD take turns between
// reading fragments and issuing MFMAs, half a step apart.  The small tiles go through a ring of four or five steps.
//
// LDS layouts.  A load instruction fills 1 KiB of LDS in lane order, so tiles are unpadded and the
// 16-byte chunks of a row are permuted by an XOR with bits of the row number (see Operand), which
// makes every fragment read conflict free while every global access stays a full 16-byte chunk of a
// contiguous run:
//   k-contiguous operand (memory [row][k]): LDS [256 rows][64 k]; a lane's MFMA fragment (8 consecutive
//     k of one row) is one ds_read_b128.
//   k-strided operand (memory [k][x]):      LDS [64 k][256 x]; the fragment is gathered by two
//     ds_read_b64_tr_b16 (the LDS transpose read: within 16 lanes, lane i receives element i%4 of the
//     8-byte pieces addressed by lanes i/4, i/4+4, i/4+8, i/4+12).
//
//   op 0  C[M,N]  = A[M,K] B[N,K]^T (+R)   A, B k-contiguous
//   op 1  C[M,N]  = A[M,K] B[K,N]          B k-strided
//   op 2  C[M,N] += A[K,M]^T B[K,N]        both k-strided; float output, added atomically: the k-steps
//                                          of every tile are cut into a whole number of equal runs, one
//                                          workgroup each, so that the rounds of workgroups are full (a
//                                          weight gradient has few tiles and a long reduction)
//
// For bf16 outputs the MFMA is issued with the tile of B as its row operand and the tile of A as its
// column operand, so a lane's accumulator holds 4 consecutive output columns of one output row; they go
// through LDS ([256][256] padded to 528 B) and leave as coalesced 16-byte stores, the optional
// added matrix R is read the same way.  Wavefront layout inside the tile: 2 (M) x 4 (N), each
// wavefront 128x64.  Workgroup ids are regrouped so that the ids that land on one XCD (id mod 8)
// cover neighbouring tiles and share operand panels in that XCD's L2.
#include "devutil.h"
#include "internal.h"

#include <type_traits>

namespace sp {

int cu_count() {
  static int n = 0;
  if (!n) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0) n = v;
    else n = 256;
  }
  return n;
}

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;

constexpr int BK = 64;
constexpr int kThreads = 512;
// Geometry of a TILE x TILE output tile: 256 (k_gemm_mfma), 128 or 64 (k_gemm_ring)
template <int TILE>
struct Geo {
  static constexpr int kTileBytes = TILE * BK * 2;        // one operand tile, either layout, unpadded
  static constexpr int kStageBytes = 2 * kTileBytes;      // A and B of one step
  static constexpr int kCRowBytes = TILE * 2 + 16;        // output staging row: TILE bf16 + 16 bytes
  static constexpr int kLdsBytesPP = 5 * kTileBytes;     // alternating-phase loop: two tiles of A, three of B
  static constexpr int XCH = TILE / 8;                    // 16-byte chunks per k row of a k-strided tile
};

constexpr uint32_t kPastEnd = 0x80000000u;      // no descriptor is this large

// Permutation of a k-strided tile's 16-byte chunks: position p of k row k holds chunk p ^ kkey(k).
//   16-wide fragments: the 8 k rows x 32 bytes that 32 lanes of a transpose read touch (rows k0 .. k0+3 and
//     k0+8 .. k0+11) fall in 8 different 32-byte bank groups; two rows of a 64-wide tile fill the banks together, so
//     there the parity of k separates them already and the key has the other two bits.
//   32-wide fragments (W32, the 256-tile of the weight-gradient product): the 4 k rows x 4 chunks that 32 lanes
//     touch fall in 16 different bank groups.
template <bool W32, int TILE>
__device__ __forceinline__ int kkey(int k) {
  if (W32) return (k & 3) << 2;
  if (TILE == 64) return (((k >> 1) & 1) | (((k >> 3) & 1) << 1)) << 1;
  return ((k & 3) | (((k >> 3) & 1) << 2)) << 1;
}

// Byte offset, from the tile's first row (k-contiguous) or first x (k-strided) at the step's first k, of the
// 16-byte chunk that belongs at position q of the tile in LDS (layouts above); kc8: for k-contiguous tiles, the
// first k of that chunk inside the step.
// split (k-contiguous only): the second half of the tile's rows lies `split` rows further on in memory (the gate
// and up rows of a SwiGLU projection that share one tile).
template <bool KSTRIDED, bool W32, int TILE>
__device__ __forceinline__ uint32_t chunk_offset(int q, int ld, int& kc8, int split = 0) {
  constexpr int XCH = Geo<TILE>::XCH;
  if (KSTRIDED) {
    const int krow = q / XCH, pos = q % XCH;
    const int c = pos ^ kkey<W32, TILE>(krow);
    return ((uint32_t)krow * ld + c * 8) * 2u;
  }
  const int row = q >> 3, pos = q & 7, c = pos ^ ((row >> 1) & 7);
  kc8 = c * 8;
  return ((uint32_t)(row + (row >= TILE / 2 ? split : 0)) * ld + c * 8) * 2u;
}

// The loads of one wavefront when a workgroup's halves divide the operands between them (the alternating-phase
// loop): wavefronts 0-3 load the tiles of A, wavefronts 4-7 those of B, so a wavefront issues a quarter of one
// operand's tile, instruction j filling chunks (4 j + w4) * 64 + lane.  One set of offsets serves either role.
template <bool AS, bool BS, bool W32, int TILE>
struct HalfLoader {
  static constexpr int NJ = Geo<TILE>::kTileBytes / 1024 / 4;
  const char* base;
  int64_t left;
  uint32_t voff[NJ];
  uint32_t k_step;
  int kc8;
  bool strided;
  __device__ __forceinline__ void init(bool late, const bf16* A, int64_t a_rows, int a_ld, int a_origin, const bf16* B,
                                       int64_t b_rows, int b_ld, int b_origin, int w4, int lane, int b_split = 0) {
    const bf16* X = late ? B : A;
    const int64_t rows = late ? b_rows : a_rows;
    const int ld = late ? b_ld : a_ld, origin = late ? b_origin : a_origin;
    strided = late ? BS : AS;
    const int64_t first = strided ? (int64_t)origin : (int64_t)origin * ld;
    base = reinterpret_cast<const char*>(X + first);
    left = (rows * ld - first) * 2;
    kc8 = 0;
    // two instructions further on: 64 rows (k-contiguous) or 16 k rows (k-strided) on, under the same permutation
    const uint32_t two_on = (uint32_t)ld * (strided ? 16 * 2u : 64 * 2u);
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      if (j < 2) {
        const int q = (4 * j + w4) * 64 + lane;
        int kc_a = 0, kc_b = 0;
        const uint32_t oa = chunk_offset<AS, W32, TILE>(q, ld, kc_a);
        const uint32_t ob = AS == BS ? oa : chunk_offset<BS, W32, TILE>(q, ld, kc_b);
        voff[j] = late ? ob : oa;
        kc8 = late && AS != BS ? kc_b : kc_a;
      } else {
        voff[j] = voff[j - 2] + two_on;
        if (!BS && j / 2 == NJ / 4 && late) voff[j] += (uint32_t)b_split * ld * 2u;   // second half of the rows
      }
    }
    k_step = strided ? (uint32_t)ld * 2u : 2u;
  }
  template <bool KMASK>
  __device__ __forceinline__ void load(int k0, int kend, char* tile, int w4) const {
    const bool dead = KMASK && !strided && (k0 + kc8 >= kend);
    const int64_t skip = (int64_t)k0 * k_step;
    const int64_t rest = left - skip;
    const u32x4 desc = make_desc(base + skip, (uint32_t)(rest < 0 ? 0 : (rest > 0x7fffffff ? 0x7fffffff : rest)));
#pragma unroll
    for (int j = 0; j < NJ; ++j) load_to_lds16(desc, (lds_ptr)(tile + (4 * j + w4) * 1024), dead ? kPastEnd : voff[j]);
  }
};

// MFMA operand fragment (v_mfma_f32_16x16x32_bf16: lane l holds row l % 16, k = (l / 16) * 8 .. + 7) of tile rows
// row_base .. row_base + 15 for the k32-th group of 32 k of the step.  row_base is a multiple of 16.
template <bool KSTRIDED, int TILE>
__device__ __forceinline__ bf16x8 read_frag(const char* tile, int row_base, int k32, int lane) {
  constexpr int KR = TILE * 2;   // bytes per k row of a k-strided tile
  if (!KSTRIDED) {
    const int lr = lane & 15, kg = lane >> 4;
    // chunk 4 k32 + kg permuted by the row's key; k32 enters by XOR with k32 * 64
    const int lane_off = lr * 128 + ((kg ^ ((lr >> 1) & 7)) << 4);
    return *reinterpret_cast<const bf16x8*>(tile + row_base * 128 + (lane_off ^ (k32 * 64)));
  } else {
    // Two transpose reads.  Within a group of 16 lanes, lane s addresses k row s/4 and the 8-byte piece s%4 of
    // the group's 32 bytes (16 x), and receives x = s, 4 consecutive k.  Group g = lane/16 takes k rows
    // 8g .. 8g+3, then 8g+4 .. 8g+7; both have the same kkey.
    const int g = lane >> 4, s = lane & 15;
    const int key = TILE == 64 ? kkey<false, TILE>((s >> 2) + (g & 1) * 8) : ((s >> 2) | ((g & 1) << 2)) << 1;
    const int lane_off = (g * 8 + (s >> 2)) * KR + (key << 4) + (((s & 3) >> 1) << 4) + (s & 1) * 8;
    const char* p = tile + k32 * 32 * KR + (lane_off ^ (row_base * 2));   // row_base * 2: a multiple of 32 bytes
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * KR));
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
}

// The same for v_mfma_f32_32x32x16_bf16 (the weight-gradient product keeps this form: its accumulator layout
// gives atomics that cover 128 contiguous bytes).  Fragment of tile row `row_base + lane % 32` for k-step ks (16 k): 8 consecutive k, starting at
// ks*16 + (lane/32)*8.  row_base is a multiple of 32.
template <bool KSTRIDED, int TILE>
__device__ __forceinline__ bf16x8 read_frag32(const char* tile, int row_base, int ks, int lane) {
  constexpr int KR = TILE * 2;
  if (!KSTRIDED) {
    const int lr = lane & 31, hh = lane >> 5;
    // chunk 2 ks + hh permuted by the row's key; ks enters by XOR with ks * 32
    const int lane_off = lr * 128 + ((hh ^ ((lr >> 1) & 7)) << 4);
    return *reinterpret_cast<const bf16x8*>(tile + row_base * 128 + (lane_off ^ (ks * 32)));
  } else {
    // group of 16 lanes = 16 consecutive x; lane s of the group addresses k row s/4, x piece s%4:
    // k row ks*16 + hh*8 + i (and + 4), chunk row_base/8 + 2 g16 + (s%4)/2, permuted by i << 2
    const int g16 = (lane >> 4) & 1, hh = lane >> 5, s = lane & 15, i = s >> 2;
    const int lane_off = (hh * 8 + i) * KR + (((i << 2) | (g16 * 2 + ((s & 3) >> 1))) << 4) + (s & 1) * 8;
    const char* p = tile + ks * 16 * KR + (lane_off ^ (row_base * 2));   // row_base * 2 = chunk bits 2.. : multiple of 64
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + 4 * KR));
    typedef __attribute__((ext_vector_type(8))) short s16x8;
    s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
  }
}

// What happens to a bf16 output tile on its way out (EPI):
//   kEpiPlain      stored, plus the matrix R if given (op 0)
//   kEpiRope       op 0: the leading rope.rot_cols columns are rotated
//   kEpiSwiglu     op 0, N = 2h, B = [gate rows | up rows]: a tile holds TILE/2 gate columns and the TILE/2 up
//                  columns of the same features (tiles_n = h / (TILE/2)); C receives both at their places and
//                  aux[M, h] receives silu(gate) * up, formed from the rounded values C holds
//   kEpiSwigluBwd  op 1, N = h: the product is d(act); with gate|up read from R[M, 2h], C[M, 2h] receives
//                  d(gate) | d(up); d(act) itself is not stored
enum { kEpiPlain = 0, kEpiRope = 1, kEpiSwiglu = 2, kEpiSwigluBwd = 3 };

// A finished bf16 tile from its LDS staging area ([TILE][TILE], rows of kCRowBytes) to memory; all 512 threads.
// m0, n0: the tile's first output row and column; the rest as in k_gemm_mfma.
template <int OP, int EPI, int TILE>
__device__ __forceinline__ void store_tile(const char* smem, bf16* C, const bf16* Rr, bf16* aux, const RopeArgs& rope, int M, int N,
                                           int m0, int n0, int tid) {
  constexpr int kCRowBytes = Geo<TILE>::kCRowBytes;
  const int hN = N / 2;
  asm volatile("" : "+v"(tid));   // keeps what follows from tid out of the registers of the loop over tiles (30 spills)
  const bool add = OP == 0 && EPI == kEpiPlain && Rr != nullptr;
  if (EPI == kEpiSwiglu) {
    // chunk nc < TILE/16 of a staged row is 8 gate values, chunk nc + TILE/16 the up values of the same features
#pragma unroll 4
    for (int c = tid; c < TILE * TILE / 16; c += kThreads) {
      const int row = c / (TILE / 16), nc = c % (TILE / 16);
      const int grow = m0 + row, gcol = n0 + nc * 8;
      if (grow < M) {
        const uint4 vg = *reinterpret_cast<const uint4*>(smem + row * kCRowBytes + nc * 16);
        const uint4 vu = *reinterpret_cast<const uint4*>(smem + row * kCRowBytes + (nc + TILE / 16) * 16);
        float g[8], u[8], o[8];
        unpack8(vg, g);
        unpack8(vu, u);
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = g[e] / (1.0f + expf(-g[e])) * u[e];
        store16_stream(C + (int64_t)grow * N + gcol, vg);
        store16_stream(C + (int64_t)grow * N + hN + gcol, vu);
        store8_stream(aux + (int64_t)grow * hN + gcol, o);
      }
    }
  } else if (EPI == kEpiSwigluBwd || add) {
    // A second operand comes from memory: its loads for kBatch chunks are issued together (where a chunk is outside the matrix, of
    // the nearest one inside), so that a thread waits for memory once or twice and not for every chunk.  Measured against one
    // load and one wait per chunk, in us: sum with R of 8192x1024 over k = 1024 29.4 -> 27.4, over k = 2816 53.5 -> 51.8; d(gate) |
    // d(up) of 16384x2816 over k = 1024 141.7 -> 140.5, of 2048x1408 over k = 512 12.9 -> 12.5.  Loads issued before the tile goes
    // to its staging area gave no more and spilled (4096 cubed with R 98.3 -> 99.8).
    constexpr int kIts = TILE * TILE / 8 / kThreads, kBatch = kIts < 8 ? kIts : 8;
    const int64_t ld = EPI == kEpiSwigluBwd ? 2 * N : N;
#pragma unroll 1
    for (int it0 = 0; it0 < kIts; it0 += kBatch) {
      uint4 r0[kBatch], r1[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int c = tid + kThreads * (it0 + b);
        const bf16* r = Rr + min(m0 + c / (TILE / 8), M - 1) * ld + min(n0 + c % (TILE / 8) * 8, N - 8);
        r0[b] = *reinterpret_cast<const uint4*>(r);
        if (EPI == kEpiSwigluBwd) r1[b] = *reinterpret_cast<const uint4*>(r + N);
      }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int c = tid + kThreads * (it0 + b);
        const int row = c / (TILE / 8), nc = c % (TILE / 8);
        const int grow = m0 + row, gcol = n0 + nc * 8;
        if (grow < M && gcol < N) {   // N is a multiple of 8: a chunk is inside or outside as a whole
          float d[8], g[8];
          unpack8(*reinterpret_cast<const uint4*>(smem + row * kCRowBytes + nc * 16), d);
          unpack8(r0[b], g);
          const int64_t at = grow * ld + gcol;
          if (EPI == kEpiSwigluBwd) {
            float u[8], og[8], ou[8];
            unpack8(r1[b], u);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float sg = 1.0f / (1.0f + expf(-g[e]));
              og[e] = d[e] * u[e] * sg * (1.0f + g[e] * (1.0f - sg));
              ou[e] = d[e] * g[e] * sg;
            }
            store8_stream(C + at, og);
            store8_stream(C + at + N, ou);
          } else {
            // the sum is formed in float from the accumulator's bf16 rounding; one more rounding on the way out
#pragma unroll
            for (int e = 0; e < 8; ++e) d[e] += g[e];
            store8_stream(C + at, d);
          }
        }
      }
    }
  } else if (EPI == kEpiRope && n0 < rope.rot_cols) {
    // A thread's chunks lie in one column of chunks, its rows kStep apart: the position follows from the one before, and the
    // table's loads for kBatch chunks are issued together.  A division by T, one by the head dimension and a wait for every chunk
    // took 3 us of every tile: the QKV products of the 500M shape's evaluation 89.9 -> 80.0 us a launch, of the 1.5B shape on
    // 1777 tokens 58.3 -> 54.3, of the 50M shape on 3 x 333 tokens (64-tiles) 7.55 -> 7.4.
    constexpr int kIts = TILE * TILE / 8 / kThreads, kBatch = kIts < 8 ? kIts : 8, kStep = kThreads / (TILE / 8);
    const int row0 = tid / (TILE / 8), nc = tid % (TILE / 8), gcol = n0 + nc * 8;
    // 8 columns = 4 pairs of one head (hd is a multiple of 8); their cos, sin are 32 contiguous bytes
    const float4* cs = reinterpret_cast<const float4*>(rope.table) + (gcol % rope.hd) / 4;
    int pos = (m0 + row0) % rope.T;
#pragma unroll 1
    for (int it0 = 0; it0 < kIts; it0 += kBatch) {
      float4 c01[kBatch], c23[kBatch];
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const float4* at = cs + (int64_t)pos * (rope.hd / 4);
        c01[b] = at[0];
        c23[b] = at[1];
        pos += kStep;
        while (pos >= rope.T) pos -= rope.T;
      }
#pragma unroll
      for (int b = 0; b < kBatch; ++b) {
        const int row = row0 + kStep * (it0 + b), grow = m0 + row;
        if (grow < M && gcol < N) {
          const uint4 v = *reinterpret_cast<const uint4*>(smem + row * kCRowBytes + nc * 16);
          const int64_t at = (int64_t)grow * N + gcol;
          if (gcol < rope.rot_cols) {
            float x[8];
            unpack8(v, x);
            const float c[4] = {c01[b].x, c01[b].z, c23[b].x, c23[b].z}, sn[4] = {c01[b].y, c01[b].w, c23[b].y, c23[b].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float p = x[2 * e], q = x[2 * e + 1];
              x[2 * e] = __builtin_fmaf(p, c[e], -(q * sn[e]));   // written out: which product is rounded is the compiler's
              x[2 * e + 1] = __builtin_fmaf(q, c[e], p * sn[e]);  // choice otherwise, and bf16 results move with it
            }
            store8_stream(C + at, x);
          } else {
            store16_stream(C + at, v);
          }
        }
      }
    }
  } else
#pragma unroll 4
  for (int it = 0; it < TILE * TILE / 8 / kThreads; ++it) {
    const int c = tid + kThreads * it;
    const int row = c / (TILE / 8), nc = c % (TILE / 8);
    const int grow = m0 + row, gcol = n0 + nc * 8;
    if (grow < M && gcol < N)   // N is a multiple of 8: a chunk is inside or outside as a whole
      store16_stream(C + (int64_t)grow * N + gcol, *reinterpret_cast<const uint4*>(smem + row * kCRowBytes + nc * 16));
  }
}

// wg of n_wgs: the workgroup's number among those of the product
template <int OP, bool KMASK, int EPI>
__device__ __forceinline__ void gemm_256(const bf16* __restrict__ A, const bf16* __restrict__ B, void* __restrict__ Cv,
                                         const bf16* __restrict__ Rr, int M, int N, int K, int tiles_m, int tiles_n,
                                         const RopeArgs& rope, bf16* __restrict__ aux, int wg, int n_wgs) {
  constexpr int TILE = 256;
  static_assert(EPI == kEpiPlain || (EPI == kEpiSwigluBwd ? OP == 1 : OP == 0), "epilogue and product do not match");
  constexpr bool AS = OP == 2, BS = OP != 0;   // which operands are k-strided
  typedef Geo<TILE> G;
  constexpr int kTileBytes = G::kTileBytes, kCRowBytes = G::kCRowBytes;
  constexpr int WM = TILE / 2, WN = TILE / 4, BM = TILE, BN = TILE;   // a wavefront's share: 2 x 4 wavefronts
  __shared__ __attribute__((aligned(1024))) char smem[G::kLdsBytesPP];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 2, wn = wave & 3;

  // ---- the work of this workgroup: tiles of the output, or a range of the k-steps of one.
  // OP 0/1: whole tiles id, id + n_wgs, ...: the launch has as many workgroups as make its rounds of
  // tiles equally full.  OP 2: one of n_wgs / tiles equal runs of the k-steps of one tile, added to the output
  // atomically.
  // Ids that share an XCD (id mod 8) get consecutive tiles (runs); tiles run down M first inside bands
  // of 8 tile columns so that neighbours share B panels and reuse A panels.
  const int tiles = tiles_m * tiles_n;
  int id = wg;
  {
    const int n_ids = n_wgs, per = n_ids / 8, rem = n_ids % 8, x = id % 8;
    id = x * per + min(x, rem) + id / 8;
  }
  const int ksteps = (K + BK - 1) / BK;
  // OP 2: n_wgs = tiles x s; id -> run id / tiles of tile id % tiles, so that the ids that share an XCD (a
  // contiguous range) work on neighbouring tiles over the same k range and share their operand panels
  const int s_runs = OP == 2 ? n_wgs / tiles : 1;
  const int run = OP == 2 ? id / tiles : 0;
  const int ks0 = OP == 2 ? (int)((int64_t)run * ksteps / s_runs) : 0;
  const int ks1 = OP == 2 ? (int)((int64_t)(run + 1) * ksteps / s_runs) : ksteps;
  for (int tile = OP == 2 ? id % tiles : id; tile < tiles; tile += OP == 2 ? tiles : n_wgs) {
  constexpr int kBand = 8;
  const int band = tile / (kBand * tiles_m);
  const int band_w = min(kBand, tiles_n - band * kBand);
  const int in_band = tile - band * kBand * tiles_m;
  const int tm = in_band / band_w, tn = band * kBand + in_band % band_w;
  // n0: first output column of the tile (kEpiSwiglu: first gate column; the up columns start at hN + n0)
  const int hN = N / 2;
  const int m0 = tm * BM, n0 = EPI == kEpiSwiglu ? tn * (BN / 2) : tn * BN;
  const int b_split = EPI == kEpiSwiglu ? hN - BN / 2 : 0;
  const int kb = ks0 * BK, kend = min(K, ks1 * BK);
  const int nk = ks1 - ks0;

  constexpr bool W32 = OP == 2;   // which MFMA form (see read_frag32)

  // OP 0/1: acc[j][i] = 16 output rows m x 16 output columns n of the wavefront's WM x WN share.
  // OP 2: acc32[j][i] = 32 rows x 32 columns of it.
  constexpr int NJ16 = WM / 16, NI16 = WN / 16, NJ32 = WM / 32, NI32 = WN / 32;
  f32x4 acc[W32 ? 1 : NJ16][W32 ? 1 : NI16];
  f32x16 acc32[W32 ? NJ32 : 1][W32 ? NI32 : 1];
  if (W32) {
#pragma unroll
    for (int j = 0; j < NJ32; ++j)
#pragma unroll
      for (int i = 0; i < NI32; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc32[W32 ? j : 0][W32 ? i : 0][r] = 0.f;
  } else {
#pragma unroll
    for (int j = 0; j < NJ16; ++j)
#pragma unroll
      for (int i = 0; i < NI16; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[W32 ? 0 : j][W32 ? 0 : i][r] = 0.f;
  }

  {
    // Two wavefronts share a SIMD (w and w + 4).  They alternate between a memory phase (all fragments of one
    // k-step from LDS into registers, loads of a later step issued) and a compute phase (the step's MFMAs, back
    // to back from registers), half a step apart, so that a SIMD's matrix core always has one wavefront
    // feeding it while the other waits for LDS and for the load queue.  Every phase ends at a workgroup
    // barrier; the late half executes one more barrier before its first phase and the early half one more
    // after its last.  The early half loads the tiles of A one step ahead into two buffers, the late half the
    // tiles of B two steps ahead into three, so every load has two phases to land before anyone waits for it
    // and the load unit sees the same number of instructions in every phase.
    const bool late = wave >= 4;
    const int w4 = wave & 3;
    constexpr int kLgkm0 = 0xC07F, kVm0 = 0x0F70;
    char* const a_ring = smem;                       // 2 tiles
    char* const b_ring = smem + 2 * kTileBytes;      // 3 tiles
    HalfLoader<AS, BS, W32, TILE> mine;
    int at = lane;
    asm volatile("" : "+v"(at));   // as in store_tile
    mine.init(late, A, AS ? K : M, AS ? M : K, m0, B, BS ? K : N, BS ? N : K, n0, w4, at, b_split);
    auto issue_a = [&](int t) { mine.template load<KMASK>(kb + t * BK, kend, a_ring + (t & 1) * kTileBytes, w4); };
    auto issue_b = [&](int t, int slot) { mine.template load<KMASK>(kb + t * BK, kend, b_ring + slot * kTileBytes, w4); };
    if (!late) issue_a(0);
    else { issue_b(0, 0); if (nk > 1) issue_b(1, 1); }
    __builtin_amdgcn_s_waitcnt(kVm0);
    __builtin_amdgcn_s_barrier();
    if (late) __builtin_amdgcn_s_barrier();
    int bs = 0;   // kt mod 3
    for (int kt = 0; kt < nk; ++kt) {
      const char* ta = a_ring + (kt & 1) * kTileBytes;
      const char* tb = b_ring + bs * kTileBytes;
      if (W32) {
        bf16x8 fa[BK / 16][NJ32], fb[BK / 16][NI32];
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
#pragma unroll
          for (int j = 0; j < NJ32; ++j) fa[ks][j] = read_frag32<AS, TILE>(ta, wm * WM + j * 32, ks, lane);
#pragma unroll
          for (int i = 0; i < NI32; ++i) fb[ks][i] = read_frag32<BS, TILE>(tb, wn * WN + i * 32, ks, lane);
        }
        if (!late) { if (kt + 1 < nk) issue_a(kt + 1); }
        else if (kt + 2 < nk) issue_b(kt + 2, bs == 0 ? 2 : bs - 1);
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks)
#pragma unroll
          for (int j = 0; j < NJ32; ++j)
#pragma unroll
            for (int i = 0; i < NI32; ++i)
              acc32[W32 ? j : 0][W32 ? i : 0] =
                  __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[ks][j], fb[ks][i], acc32[W32 ? j : 0][W32 ? i : 0], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
      } else {
        bf16x8 fa[BK / 32][NJ16], fb[BK / 32][NI16];
#pragma unroll
        for (int k32 = 0; k32 < BK / 32; ++k32) {
#pragma unroll
          for (int j = 0; j < NJ16; ++j) fa[k32][j] = read_frag<AS, TILE>(ta, wm * WM + j * 16, k32, lane);
#pragma unroll
          for (int i = 0; i < NI16; ++i) fb[k32][i] = read_frag<BS, TILE>(tb, wn * WN + i * 16, k32, lane);
        }
        if (!late) { if (kt + 1 < nk) issue_a(kt + 1); }
        else if (kt + 2 < nk) issue_b(kt + 2, bs == 0 ? 2 : bs - 1);
        __builtin_amdgcn_s_waitcnt(kLgkm0);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(1);
#pragma unroll
        for (int k32 = 0; k32 < BK / 32; ++k32)
#pragma unroll
          for (int j = 0; j < NJ16; ++j)
#pragma unroll
            for (int i = 0; i < NI16; ++i)
              acc[W32 ? 0 : j][W32 ? 0 : i] =
                  __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[k32][i], fa[k32][j], acc[W32 ? 0 : j][W32 ? 0 : i], 0, 0, 0);
        __builtin_amdgcn_s_setprio(0);
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(kVm0);   // issued two phases ago
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_sched_barrier(0);
      bs = bs == 2 ? 0 : bs + 1;
    }
    if (!late) __builtin_amdgcn_s_barrier();
  }

  // ---- epilogue.  With the tile of B as the MFMA's row operand (OP 0/1), accumulator r of lane l is output
  // row m = l % 16, output column n = (l / 16) * 4 + r of its 16x16 block: 4 consecutive columns.
  const int lm = lane & 15, kg = lane >> 4;
  if (OP == 2) {
    // float output, accumulated in place.  Here the tile of A is the MFMA's row operand: accumulator r of
    // lane l is output row (r/4)*8 + (l/32)*4 + r%4, column l%32, so a wavefront's atomic covers 128
    // contiguous bytes of two rows.
    float* C = reinterpret_cast<float*>(Cv);
#pragma unroll
    for (int j = 0; j < NJ32; ++j)
#pragma unroll
      for (int i = 0; i < NI32; ++i) {
        const int col = n0 + wn * WN + i * 32 + (lane & 31);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = m0 + wm * WM + j * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
          if (row < M && col < N) {
            float* p = C + (int64_t)row * N + col;
            unsafeAtomicAdd(p, acc32[W32 ? j : 0][W32 ? i : 0][r]);
          }
        }
      }
  } else {
    // all wavefronts are past the last barrier of the loop: the operand buffers are free
#pragma unroll
    for (int j = 0; j < NJ16; ++j)
#pragma unroll
      for (int i = 0; i < NI16; ++i) {
        uint2 w;
        w.x = pack_bf16(acc[W32 ? 0 : j][W32 ? 0 : i][0], acc[W32 ? 0 : j][W32 ? 0 : i][1]);
        w.y = pack_bf16(acc[W32 ? 0 : j][W32 ? 0 : i][2], acc[W32 ? 0 : j][W32 ? 0 : i][3]);
        *reinterpret_cast<uint2*>(smem + (wm * WM + j * 16 + lm) * kCRowBytes + (wn * WN + i * 16 + kg * 4) * 2) = w;
      }
    __syncthreads();
    store_tile<OP, EPI, TILE>(smem, reinterpret_cast<bf16*>(Cv), Rr, aux, rope, M, N, m0, n0, tid);
    __syncthreads();   // the staging area becomes the next tile's operand ring
  }
  }  // next tile
}

// ---- tiles of 128 or 64 for products that leave the chip partly idle in 256-tiles (a single microbatch, narrow
// layers, the weight gradient of a small matrix).
//
// One workgroup per CU is then the rule, so nothing but its own loads in flight hides the memory's latency: operand
// tiles go through a ring of S steps in LDS, a slot is loaded again as soon as its fragments are in registers, S - 1
// steps before it is waited for, and the fragments of step t + 1 are read while the MFMAs of step t run.  One
// barrier per step.  The eight wavefronts are a 2 x 2 grid over the tile twice.  Weight gradients: wavefronts 0-3 take
// the first 32 k of every step, 4-7 the other 32 (a wavefront's share is as square as the tile, so LDS reads stay level
// with the MFMAs: 64 KB against 512 matrix cycles a step at TILE = 128), and the two halves' accumulators meet in LDS at
// the end.  Forward and input-gradient products: the two sets divide the rows of a share instead (96 KB of reads), so
// that every output is summed in the order of k as in a 256-tile: their results are rounded to bf16, and a
// microbatch's must not depend on the tile that the size of its group leads to.
// A step of a 128-tile takes 0.51 us (op 0), 0.54 (op 1), 0.46 (op 2) with every CU busy; with the loads delivering zeros
// 0.32, 0.36 and 0.36: in ops 0 and 1 that is the fragment reads (96 KB at 128 bytes a cycle 0.32 us at 2.4 GHz), against
// 0.21 of MFMAs, and the rest is the way from the L2s.  Against the two-slot loop of 128-tiles with one wait per step that
// stood here before: NT 4096 x 1024 x 2816 34 -> 27 us, NN 1777 x 2048 x 11264 127 -> 92 us; TN (256-tiles before) 1024 x
// 1024 x 4096 37 -> 26 us, 288 x 768 x 999 19 -> 8 us (64-tiles).
template <int TILE>
struct RingGeo {
  static constexpr int S = TILE == 128 ? 4 : 5;            // 128 KB; 80 KB, so that two workgroups of 64-tiles share a CU
  static constexpr int kLdsBytes = S * Geo<TILE>::kStageBytes;
  static constexpr int NL = Geo<TILE>::kTileBytes / 1024 / 8;   // load instructions per wavefront and operand tile
  static constexpr int W = TILE / 2, NF = W / 16;          // a wavefront's share of the tile: NF x NF blocks of 16 x 16
  static constexpr int kRowFloats = TILE + 4;              // float staging row (weight gradients)
};

// One operand's share of the loads of one wavefront: instruction j fills chunks (8 j + wave) * 64 + lane of the tile.
template <bool KSTRIDED, int TILE>
struct RingOperand {
  static constexpr int NL = RingGeo<TILE>::NL;
  const char* base;    // first byte of the tile's rows (k-contiguous) or of its first x (k-strided), at k = 0
  int64_t left;        // bytes from base to the end of the operand
  uint32_t voff[NL];
  uint32_t k_step;     // byte distance of one k element
  int kc8;             // k-contiguous: first k of the lane's chunk inside a step
  __device__ __forceinline__ void init(const bf16* X, int64_t rows, int ld, int origin, int wave, int lane, int split = 0) {
    const int64_t first = KSTRIDED ? (int64_t)origin : (int64_t)origin * ld;
    base = reinterpret_cast<const char*>(X + first);
    left = (rows * ld - first) * 2;
    kc8 = 0;
#pragma unroll
    for (int j = 0; j < NL; ++j) voff[j] = chunk_offset<KSTRIDED, false, TILE>((8 * j + wave) * 64 + lane, ld, kc8, split);
    k_step = KSTRIDED ? (uint32_t)ld * 2u : 2u;
  }
  // live = false: zeros, without touching memory
  __device__ __forceinline__ u32x4 desc(bool live, int k0) const {
    const int64_t skip = (int64_t)k0 * k_step;
    const int64_t rest = live ? left - skip : 0;
    return make_desc(base + skip, (uint32_t)(rest < 0 ? 0 : (rest > 0x7fffffff ? 0x7fffffff : rest)));
  }
  template <bool KMASK>
  __device__ __forceinline__ void load(int j, const u32x4& desc, int k0, int kend, char* tile, int wave) const {
    const bool dead = KMASK && !KSTRIDED && (k0 + kc8 >= kend);
    load_to_lds16(desc, (lds_ptr)(tile + (8 * j + wave) * 1024), dead ? kPastEnd : voff[j]);
  }
};

template <int OP, bool KMASK, int EPI, int TILE>
__device__ __forceinline__ void gemm_ring(const bf16* __restrict__ A, const bf16* __restrict__ B, void* __restrict__ Cv,
                                          const bf16* __restrict__ Rr, int M, int N, int K, int tiles_m, int tiles_n,
                                          const RopeArgs& rope, bf16* __restrict__ aux, int wg, int n_wgs) {
  static_assert(EPI == kEpiPlain || (EPI == kEpiSwigluBwd ? OP == 1 : OP == 0), "epilogue and product do not match");
  constexpr bool AS = OP == 2, BS = OP != 0;
  typedef Geo<TILE> G;
  typedef RingGeo<TILE> RG;
  constexpr int S = RG::S, NF = RG::NF, W = RG::W;
  constexpr bool KH = OP == 2;                           // the sets divide k (else rows)
  constexpr int Q = KH ? 1 : 2, NA = KH ? NF : NF / 2;   // k halves and row blocks of a wavefront
  __shared__ __attribute__((aligned(1024))) char smem[RG::kLdsBytes];
  static_assert(TILE * RG::kRowFloats * 4 <= RG::kLdsBytes && TILE * G::kCRowBytes <= RG::kLdsBytes, "staging fits");
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = wave >> 2, wm = (wave >> 1) & 1, wn = wave & 1;

  // the tiles of this workgroup, numbered as in k_gemm_mfma
  const int tiles = tiles_m * tiles_n;
  int id = wg;
  {
    const int n_ids = n_wgs, per = n_ids / 8, rem = n_ids % 8, x = id % 8;
    id = x * per + min(x, rem) + id / 8;
  }
  const int ksteps = (K + BK - 1) / BK;
  const int s_runs = OP == 2 ? n_wgs / tiles : 1;
  const int run = OP == 2 ? id / tiles : 0;
  const int ks0 = OP == 2 ? (int)((int64_t)run * ksteps / s_runs) : 0;
  const int ks1 = OP == 2 ? (int)((int64_t)(run + 1) * ksteps / s_runs) : ksteps;
  const int kb = ks0 * BK, kend = min(K, ks1 * BK), nk = ks1 - ks0;
  for (int tile = OP == 2 ? id % tiles : id; tile < tiles; tile += OP == 2 ? tiles : n_wgs) {
    constexpr int kBand = 8;
    const int band = tile / (kBand * tiles_m);
    const int band_w = min(kBand, tiles_n - band * kBand);
    const int in_band = tile - band * kBand * tiles_m;
    const int tm = in_band / band_w, tn = band * kBand + in_band % band_w;
    const int hN = N / 2;
    const int m0 = tm * TILE, n0 = EPI == kEpiSwiglu ? tn * (TILE / 2) : tn * TILE;
    const int b_split = EPI == kEpiSwiglu ? hN - TILE / 2 : 0;

    RingOperand<AS, TILE> opa;
    RingOperand<BS, TILE> opb;
    opa.init(A, AS ? K : M, AS ? M : K, m0, wave, lane);
    opb.init(B, BS ? K : N, BS ? N : K, n0, wave, lane, b_split);
    // every step issues 2 NL loads per wavefront, past the last one too (they deliver zeros), so that one wait fits all
    auto issue = [&](int p, const u32x4& da, const u32x4& db, int t, int slot) {   // load p of the step's 2 NL
      char* st = smem + slot * G::kStageBytes;
      if (p < RG::NL) opa.template load<KMASK>(p, da, kb + t * BK, kend, st, wave);
      else opb.template load<KMASK>(p - RG::NL, db, kb + t * BK, kend, st + G::kTileBytes, wave);
    };
    // this wavefront's LDS reads are done and all but its newest n loads have landed
    auto wait = [](auto n) {
      constexpr int v = decltype(n)::value;
      __builtin_amdgcn_s_waitcnt((v & 15) | (7 << 4) | (0 << 8) | ((v >> 4) << 14));
    };
    struct Frags { bf16x8 a[Q * NA], b[Q][NF]; };   // a: by k half, then row block; Q NA = NF
    auto read = [&](int j, int slot, Frags& f) {
      const char* ta = smem + slot * G::kStageBytes;
      f.a[j] = read_frag<AS, TILE>(ta, wm * W + (KH ? j : hh * NA + j % NA) * 16, KH ? hh : j / NA, lane);
#pragma unroll
      for (int q = 0; q < Q; ++q) f.b[q][j] = read_frag<BS, TILE>(ta + G::kTileBytes, wn * W + j * 16, KH ? hh : q, lane);
    };

    f32x4 acc[NA][NF];
#pragma unroll
    for (int j = 0; j < NA; ++j)
#pragma unroll
      for (int i = 0; i < NF; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[j][i][r] = 0.f;

#pragma unroll
    for (int t = 0; t < S; ++t) {
      const u32x4 da = opa.desc(t < nk, kb + t * BK), db = opb.desc(t < nk, kb + t * BK);
#pragma unroll
      for (int p = 0; p < 2 * RG::NL; ++p) issue(p, da, db, t, t);
    }
    wait(std::integral_constant<int, (S - 1) * 2 * RG::NL>());
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    Frags f0, f1;
#pragma unroll
    for (int j = 0; j < NF; ++j) read(j, 0, f0);
    int slot = 0;   // kt mod S
    auto step = [&](int kt, Frags& now, Frags& next) {
      wait(std::integral_constant<int, (S - 2) * 2 * RG::NL>());   // `now` is in registers, step kt + 1 in LDS
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();                                // the same for every wavefront: the slot is free
      __builtin_amdgcn_sched_barrier(0);
      const int after = slot + 1 == S ? 0 : slot + 1;
      const u32x4 da = opa.desc(kt + S < nk, kb + (kt + S) * BK), db = opb.desc(kt + S < nk, kb + (kt + S) * BK);
      static_assert(2 * RG::NL == NF, "one load per row of blocks");
      // the matrix core starts at once; reads and loads are issued behind each row of blocks
#pragma unroll
      for (int j = 0; j < NF; ++j) {
#pragma unroll
        for (int i = 0; i < NF; ++i) acc[j % NA][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(now.b[j / NA][i], now.a[j], acc[j % NA][i], 0, 0, 0);
        read(j, after, next);
        issue(j, da, db, kt + S, slot);
        __builtin_amdgcn_sched_barrier(0);
      }
      slot = after;
    };
    for (int kt = 0; kt < nk; kt += 2) {
      step(kt, f0, f1);
      if (kt + 1 < nk) step(kt + 1, f1, f0);
    }

    // ---- k halves: the two halves' sums meet: a wavefront gives its partner (wave ^ 4) the row blocks the partner finishes and
    // finishes the others, blocks hh * NF / 2 .. of the share
    wait(std::integral_constant<int, 0>());
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    f32x4 sum[NF / 2][NF];
    if constexpr (KH) {
      f32x4* const swap = reinterpret_cast<f32x4*>(smem);
#pragma unroll
      for (int j = 0; j < NF / 2; ++j)
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          swap[((wave * (NF / 2) + j) * NF + i) * 64 + lane] = hh ? acc[j][i] : acc[j + NF / 2][i];
          sum[j][i] = hh ? acc[j + NF / 2][i] : acc[j][i];
        }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < NF / 2; ++j)
#pragma unroll
        for (int i = 0; i < NF; ++i) {
          const f32x4 o = swap[(((wave ^ 4) * (NF / 2) + j) * NF + i) * 64 + lane];
#pragma unroll
          for (int r = 0; r < 4; ++r) sum[j][i][r] += o[r];
        }
      __syncthreads();
    } else {
#pragma unroll
      for (int j = 0; j < NF / 2; ++j)
#pragma unroll
        for (int i = 0; i < NF; ++i) sum[j][i] = acc[j][i];
    }
    // lane: row lane % 16 of a block, columns (lane / 16) * 4 .. + 3
    const int lm = lane & 15, kg = lane >> 4;
#pragma unroll
    for (int j = 0; j < NF / 2; ++j)
#pragma unroll
      for (int i = 0; i < NF; ++i) {
        const int row = wm * W + (hh * (NF / 2) + j) * 16 + lm, col = wn * W + i * 16 + kg * 4;
        if (OP == 2) {
          *reinterpret_cast<f32x4*>(smem + (row * RG::kRowFloats + col) * 4) = sum[j][i];
        } else {
          uint2 w;
          w.x = pack_bf16(sum[j][i][0], sum[j][i][1]);
          w.y = pack_bf16(sum[j][i][2], sum[j][i][3]);
          *reinterpret_cast<uint2*>(smem + row * G::kCRowBytes + col * 2) = w;
        }
      }
    __syncthreads();
    if (OP == 2) {
      // a wavefront's atomics cover 256 contiguous bytes of one row
      float* C = reinterpret_cast<float*>(Cv);
#pragma unroll 8
      for (int it = 0; it < TILE * TILE / kThreads; ++it) {
        const int c = tid + kThreads * it, row = c / TILE, col = c % TILE;
        if (m0 + row < M && n0 + col < N)
          unsafeAtomicAdd(C + (int64_t)(m0 + row) * N + n0 + col, reinterpret_cast<const float*>(smem)[row * RG::kRowFloats + col]);
      }
    } else {
      store_tile<OP, EPI, TILE>(smem, reinterpret_cast<bf16*>(Cv), Rr, aux, rope, M, N, m0, n0, tid);
    }
    __syncthreads();   // the staging area becomes the next tile's ring
  }
}

template <int OP, bool KMASK, int EPI>
__global__ __launch_bounds__(kThreads) void k_gemm_mfma(const bf16* __restrict__ A, const bf16* __restrict__ B,
                                                        void* __restrict__ Cv, const bf16* __restrict__ Rr, int M,
                                                        int N, int K, int tiles_m, int tiles_n, RopeArgs rope,
                                                        bf16* __restrict__ aux) {
  gemm_256<OP, KMASK, EPI>(A, B, Cv, Rr, M, N, K, tiles_m, tiles_n, rope, aux, blockIdx.x, gridDim.x);
}
template <int OP, bool KMASK, int EPI, int TILE>
__global__ __launch_bounds__(kThreads) void k_gemm_ring(const bf16* __restrict__ A, const bf16* __restrict__ B,
                                                        void* __restrict__ Cv, const bf16* __restrict__ Rr, int M,
                                                        int N, int K, int tiles_m, int tiles_n, RopeArgs rope,
                                                        bf16* __restrict__ aux) {
  gemm_ring<OP, KMASK, EPI, TILE>(A, B, Cv, Rr, M, N, K, tiles_m, tiles_n, rope, aux, blockIdx.x, gridDim.x);
}

// The weight gradients of a layer in one launch: its four products together fill the chip where one of them leaves it partly
// idle or has to be cut into many runs.
template <int TILE>
__global__ __launch_bounds__(kThreads) void k_gemm_grads(GradGroup g) {
  int i = 0;
  while (i + 1 < kGrads && (int)blockIdx.x >= g.first[i + 1]) ++i;
  const int wg = (int)blockIdx.x - g.first[i], n = g.first[i + 1] - g.first[i];
  const RopeArgs none{nullptr, 1, 8, 0};
  if constexpr (TILE == 256)
    gemm_256<2, false, kEpiPlain>((const bf16*)g.A[i], (const bf16*)g.B[i], g.C[i], nullptr, g.M[i], g.N[i], g.K, g.tm[i], g.tn[i], none, nullptr, wg, n);
  else
    gemm_ring<2, false, kEpiPlain, TILE>((const bf16*)g.A[i], (const bf16*)g.B[i], g.C[i], nullptr, g.M[i], g.N[i], g.K, g.tm[i], g.tn[i], none, nullptr, wg, n);
}

inline bool al16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// Tile, tile grid and workgroups of a launch: the least of what each choice is expected to take, in microseconds,
//   rounds of workgroups x (k-steps x step + ends)  +  op 2: runs x output bytes / atomics rate
// step and ends are fits to measured products of 4 to 344 steps over grids of 24 to 1400 tiles: a 256-tile takes 0.9 to
// 1.3 us a step (the clock falls as CUs fill), a 128-tile 0.5 (its operand traffic per flop is twice as large), a
// 64-tile 0.3 alone on its CU and 0.37 beside another.  (Taken again over one full round: 256-tiles 1.30 / 1.33 / 1.44 for
// ops 0 / 1 / 2, 128-tiles 0.51 / 0.54 / 0.46, 64-tiles 0.25 / 0.27 / 0.27 alone and 0.42 / 0.47 / 0.43 beside another; the
// choices at the examples stay the faster ones or within 3 %.)  Float atomics reach 1.4 TB/s over the whole chip whatever the
// tile, so that further runs per tile cost most where the reduction is short.  Examples, us, 256- / 128- / 64-tile:
// NT 4096 x 1024 x 2816 47 / 27 / 46, NT 1777 x 6144 x 2048 42 / 53 / 91, NN 8192 x 1024 x 1024 24 / 23 / 41, NT 8192 x
// 6144 x 2048 148 / 219 / 369, NN 1777 x 2048 x 11264 178 / 92 / 168, TN 1024 x 1024 x 4096 32 / 26 / 26, TN 2048 x 2048
// x 8192 90 / 79 / 126, TN 5632 x 1024 x 8192 108 / 126 / 183, TN 288 x 768 x 999 15 / 9 / 8.
struct Shape { int tile, tm, tn, wgs; };
Shape choose_shape(int op, int64_t M, int64_t N, int64_t K, int epi) {
  const int64_t cus = cu_count(), ksteps = (K + BK - 1) / BK;
  Shape best{};
  double best_us = 0;
  for (int t : {256, 128, 64}) {
    if (epi == kEpiSwiglu && (N / 2) % (t / 2)) continue;   // a tile covers t/2 gate and the matching t/2 up columns
    const int64_t tm = (M + t - 1) / t, tn = (N + t - 1) / t, tiles = tm * tn;
    // op 2, 256-tiles: the smallest number of runs whose last round is at least 0.65 full; another number has to
    // promise 7 %, which is as good as the fits are
    int usual = 0;
    for (int runs = 1; op == 2 && t == 256 && runs <= 8 && (runs == 1 || ksteps / runs >= 8); ++runs) {
      usual = runs;
      const int64_t wgs = tiles * runs, last = wgs % cus;
      if (last == 0 || last * 100 >= cus * 65 || wgs >= 6 * cus) break;
    }
    // an op 2 run of fewer than 4 steps would be mostly start and end
    for (int runs = 1; runs <= (op == 2 ? 16 : 1) && (runs == 1 || ksteps / runs >= 4); ++runs) {
      const int64_t wgs = tiles * runs, slots = t == 64 && wgs > cus ? 2 * cus : cus, rounds = (wgs + slots - 1) / slots;
      const double step = t == 256 ? 0.85 + 0.45 * (double)wgs / (double)(rounds * cus) : t == 128 ? 0.5 : slots > cus ? 0.37 : 0.3;
      const double ends = t == 256 ? 5 : t == 128 ? 4 : 3;
      double us = (double)rounds * ((double)((ksteps + runs - 1) / runs) * step + ends) +
                  (op == 2 ? runs * 4.0 * (double)M * (double)N / 1.4e6 : 0.0);
      if (runs == usual) us *= 0.93;
      if (best.tile && us >= best_us) continue;
      best_us = us;
      // op 0/1: equally full rounds, every workgroup taking every wgs-th tile
      best = {t, (int)tm, (int)tn, (int)(op == 2 ? wgs : (tiles + rounds - 1) / rounds)};
    }
  }
  return best;
}

}  // namespace

GemmShape gemm_mfma_shape(int op, int64_t M, int64_t N, int64_t K, int epi) {
  const Shape s = choose_shape(op, M, N, K, epi);
  return {s.tile, s.tm * s.tn, s.wgs};
}

bool gemm_mfma_supported(int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, const void* C,
                         const void* R) {
  if (M < 1 || N < 1 || K < 1) return false;
  // tile-relative byte offsets (up to 256 rows of the leading dimension) stay below 2^31
  if (M >= (1 << 21) || N >= (1 << 21) || K >= (1 << 21)) return false;
  if (!al16(A) || !al16(B) || !al16(C) || (R && !al16(R))) return false;
  if (((M + 127) / 128) * ((N + 127) / 128) > (1 << 24)) return false;
  if (N % 8) return false;                      // 16-byte output chunks
  switch (op) {
    case 0: return K % 8 == 0;
    case 1: return K % 8 == 0;
    case 2: return M % 8 == 0;
  }
  return false;
}

// epi: kEpiPlain (R optional), kEpiRope (rope given), kEpiSwiglu (N = 2h, aux = act out), kEpiSwigluBwd (N = h,
// R = gate|up in, C = d(gate)|d(up) out)
void gemm_mfma(hipStream_t s, int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C,
               const void* R, const RopeArgs* rope, int epi, void* aux) {
  if (rope) epi = kEpiRope;
  const Shape sh = choose_shape(op, M, N, K, epi);
  const int tile = sh.tile, tm = sh.tm, tn = sh.tn, wgs = sh.wgs;
  dim3 grid(wgs);
  const bf16* a = (const bf16*)A;
  const bf16* b = (const bf16*)B;
  const bf16* r = (const bf16*)R;
  const bool kmask = K % BK != 0;
  const RopeArgs ra = rope ? *rope : RopeArgs{nullptr, 1, 8, 0};
#define SP_LAUNCH(KERNEL) \
  hipLaunchKernelGGL(KERNEL, grid, dim3(kThreads), 0, s, a, b, C, r, (int)M, (int)N, (int)K, tm, tn, ra, (bf16*)aux)
#define SP_LAUNCH_K(OP, KM, EP)                            \
  do {                                                     \
    if (tile == 256) SP_LAUNCH((k_gemm_mfma<OP, KM, EP>)); \
    else if (tile == 128) SP_LAUNCH((k_gemm_ring<OP, KM, EP, 128>)); \
    else SP_LAUNCH((k_gemm_ring<OP, KM, EP, 64>));         \
  } while (0)
#define SP_LAUNCH_T(OP, EP) \
  do { if (kmask) SP_LAUNCH_K(OP, true, EP); else SP_LAUNCH_K(OP, false, EP); } while (0)
  if (op == 0 && epi == kEpiRope) SP_LAUNCH_T(0, kEpiRope);
  else if (op == 0 && epi == kEpiSwiglu) SP_LAUNCH_T(0, kEpiSwiglu);
  else if (op == 0) SP_LAUNCH_T(0, kEpiPlain);
  else if (op == 1 && epi == kEpiSwigluBwd) SP_LAUNCH_T(1, kEpiSwigluBwd);
  else if (op == 1) SP_LAUNCH_T(1, kEpiPlain);
  else SP_LAUNCH_K(2, false, kEpiPlain);
#undef SP_LAUNCH_T
#undef SP_LAUNCH_K
#undef SP_LAUNCH
}

// One tile and one number of runs for all of them, by the costs of choose_shape.
void gemm_mfma_grads(hipStream_t s, int64_t K, const GradItem (&items)[kGrads]) {
  const int64_t cus = cu_count(), ksteps = (K + BK - 1) / BK;
  GradGroup g{};
  int tile = 0, best_runs = 0;
  double best_us = 0;
  for (int t : {256, 128, 64}) {
    int64_t tiles = 0;
    double bytes = 0;
    for (const GradItem& i : items) {
      tiles += ((i.M + t - 1) / t) * ((i.N + t - 1) / t);
      bytes += 4.0 * (double)i.M * (double)i.N;
    }
    for (int runs = 1; runs <= 16 && (runs == 1 || ksteps / runs >= 4); ++runs) {
      const int64_t wgs = tiles * runs, slots = t == 64 && wgs > cus ? 2 * cus : cus, rounds = (wgs + slots - 1) / slots;
      const double step = t == 256 ? 0.85 + 0.45 * (double)wgs / (double)(rounds * cus) : t == 128 ? 0.5 : slots > cus ? 0.37 : 0.3;
      const double us = (double)rounds * ((double)((ksteps + runs - 1) / runs) * step + (t == 256 ? 5 : t == 128 ? 4 : 3)) + runs * bytes / 1.4e6;
      if (tile && us >= best_us) continue;
      best_us = us;
      tile = t;
      best_runs = runs;
    }
  }
  for (int i = 0; i < kGrads; ++i) {
    const GradItem& x = items[i];
    g.A[i] = x.A; g.B[i] = x.B; g.C[i] = x.C;
    g.M[i] = (int)x.M; g.N[i] = (int)x.N;
    g.tm[i] = (int)((x.M + tile - 1) / tile); g.tn[i] = (int)((x.N + tile - 1) / tile);
    g.first[i + 1] = g.first[i] + g.tm[i] * g.tn[i] * best_runs;
  }
  g.K = (int)K;
  const dim3 grid(g.first[kGrads]);
  if (tile == 256) hipLaunchKernelGGL(k_gemm_grads<256>, grid, dim3(kThreads), 0, s, g);
  else if (tile == 128) hipLaunchKernelGGL(k_gemm_grads<128>, grid, dim3(kThreads), 0, s, g);
  else hipLaunchKernelGGL(k_gemm_grads<64>, grid, dim3(kThreads), 0, s, g);
}

bool gemm_swiglu_supported(bool bwd, int64_t R, int64_t h, int64_t d, const void* X, const void* W, const void* gu,
                           const void* other) {
  if (h % 64) return false;   // forward: a tile of 64, 128 or 256 columns holds whole halves of gate and up
  if (bwd) return gemm_mfma_supported(1, R, h, d, X, W, other, gu);
  return gemm_mfma_supported(0, R, 2 * h, d, X, W, gu, other);
}

void gemm_mfma_swiglu_fwd(hipStream_t s, int64_t R, int64_t h, int64_t d, const void* hn, const void* wgu, void* gu, void* act) {
  gemm_mfma(s, 0, R, 2 * h, d, hn, wgu, gu, nullptr, nullptr, kEpiSwiglu, act);
}

void gemm_mfma_swiglu_bwd(hipStream_t s, int64_t R, int64_t h, int64_t d, const void* dy, const void* wd, const void* gu, void* dgu) {
  gemm_mfma(s, 1, R, h, d, dy, wd, dgu, gu, nullptr, kEpiSwigluBwd, nullptr);
}

}  // namespace sp
