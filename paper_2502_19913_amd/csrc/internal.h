// Declarations shared by the library's translation units (not part of the public boundary).
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/skippipe.h"

typedef struct ihipStream_t* hipStream_t;

namespace sp {

// ---- error plumbing
int fail(int code, const std::string& msg);
int check_cfg(const sp_cfg* c);
int hip_fail(int hip_error, const char* what);  // records the HIP message, returns SP_EHIP

// ---- flat parameter layout
struct LayerOff { int64_t g1, wqkv, wo, g2, wgu, wd; };
struct Layout {
  int64_t embed = 0, gf = 0, whead = 0, total = 0;
  std::vector<LayerOff> layers;  // local layers, stage-major
  std::vector<sp_tensor_desc> tensors;
};
Layout make_layout(const sp_cfg& c);

// ---- routing
struct Group { int pos, stage; std::vector<int> mb; };
int check_one_path(const sp_cfg& c, const int32_t* p, int len, int mb);
int build_plan(const sp_cfg& c, const int32_t* paths, const int32_t* len, int n_mb, std::vector<Group>& out);

inline int64_t elt_size(int dtype) { return dtype == SP_BF16 ? 2 : 4; }

// Up to this many microbatches may share one group (slot numbers travel as a kernel argument).
constexpr int kMaxGroup = 64;
struct SlotList { int32_t n; int32_t slot[kMaxGroup]; };

// ---- kernel launchers (all asynchronous on `s`; dtype is SP_F32 or SP_BF16)
// A token outside [0, V) sets *bad (device int32) to 1; its row reads as zeros / adds nothing.
void embed_fwd(hipStream_t s, int dtype, const void* E, const int32_t* tok, int64_t rows, int d, int V, void* x,
               int32_t* bad);
void embed_bwd(hipStream_t s, int dtype, const void* dx, const int32_t* tok, int64_t rows, int d, int V, float* dE,
               int32_t* bad);
// dst[g*rows_per_slot + r, :] = pool[slot[g]*rows_per_slot + r, :]   (and the reverse)
void gather_slots(hipStream_t s, int dtype, const void* pool, const SlotList& sl, int64_t rows_per_slot, int d, void* dst);
void scatter_slots(hipStream_t s, int dtype, const void* src, const SlotList& sl, int64_t rows_per_slot, int d, void* pool);
void fill_zero(hipStream_t s, void* p, int64_t bytes);

void rmsnorm_fwd(hipStream_t s, int dtype, const void* x, const void* g, int64_t R, int d, float eps, void* y, float* rstd);
// dx = (dres ? dres : 0) + rmsnorm'(dy) ; dg += sum_rows dy * x * rstd
// part (may be null): scratch of part_floats floats for the per-block partial sums of dg (kRmsPartRows x d is
// enough); where the call leaves sums there it notes them in *fold, and dg is complete after rmsnorm_bwd_fold, which
// adds up all that is noted (norms of the same width d) and empties the list
constexpr int kRmsPartRows = 1024;
// Two norms of each layer of a four-layer stage wait for one fold.  One launch instead of eight: 50M shapes (d = 288) 3.65 ->
// 3.60 ms a pass in bf16, 5.72 -> 5.64 in float, 500M shape (d = 1024) 64.6 -> 64.4, 1.5B stage (d = 2048) on 300 to 2500
// rows 0.2 to 1 % (2.65 -> 2.62 on 700), 7B stage (d = 4096) 6.30 -> 6.17 on 500 rows, 10.05 -> 10.0 on 1500; large groups
// even.  It costs 8 x 1024 x d floats of workspace (128 MiB at d = 4096).
constexpr int kRmsFoldMax = 8;
struct RmsFold {
  const float* part[kRmsFoldMax];
  float* dg[kRmsFoldMax];
  int rows[kRmsFoldMax];
  int n;
  void add(const float* p, float* g, int r) { part[n] = p; dg[n] = g; rows[n++] = r; }
};
void rmsnorm_bwd_fold(hipStream_t s, RmsFold* fold, int d);
void rmsnorm_bwd(hipStream_t s, int dtype, const void* dy, const void* x, const void* g, const float* rstd,
                 const void* dres, int64_t R, int d, void* dx, float* dg, float* part, int64_t part_floats, RmsFold* fold);
// bf16: rotates the first nheads*hd columns of every row (row_stride elements apart); position = row % T
void rope(hipStream_t s, void* qk, int64_t R, int T, int nheads, int hd, int row_stride, float theta);
// table[(p * hd/2 + i) * 2 + {0, 1}] = cos, sin of p * theta^(-2i/hd), the angles rope() uses, for p < T
void rope_table(hipStream_t s, int T, int hd, float theta, float* table);
// Rotation fused into a producer: the leading rot_cols columns of a row are heads of hd columns whose pairs
// (2i, 2i+1) turn by the angle of position (row % T); table as written by rope_table
struct RopeArgs {
  const float* table;
  int T, hd, rot_cols;
};
// bf16; a = silu(gate) * up and its gradient as passes of their own
void swiglu_fwd(hipStream_t s, const void* gu, int64_t R, int h, void* a);
void swiglu_bwd(hipStream_t s, const void* da, const void* gu, int64_t R, int h, void* dgu);
// counts[mb] = number of targets in [0, V) among the rows of microbatch mb; a target below -1 or >= V sets *bad
void count_targets(hipStream_t s, const int32_t* tgt, int n_mb, int64_t rows_per_mb, int V, int32_t* counts,
                   int32_t* bad);
// rows [row0, row0+R) of the iteration: logits -> dlogits in place, loss_mb[mb] += rowloss / counts[mb]
void cross_entropy(hipStream_t s, int dtype, void* logits, const int32_t* tgt, int64_t row0, int64_t R, int V,
                   int64_t rows_per_mb, const int32_t* counts, float inv_n_mb, float* loss_mb);

// C = A*B^T (+R) | C = A*B | C += A^T*B  (see sp_gemm); returns SP_EINVAL for bad arguments
int gemm(hipStream_t s, int dtype, int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C,
         const void* R);

// The weight gradients of a layer: C[i] (float) += A[i]^T B[i] over K rows, in one launch where the matrix-core kernels take all of them.
constexpr int kGrads = 4;
struct GradItem { int64_t M, N; const void *A, *B; float* C; };
int gemm_grads(hipStream_t s, int dtype, int64_t K, const GradItem (&items)[kGrads]);
// What such a launch needs on the device; item i has the workgroups first[i] .. first[i + 1] - 1
struct GradGroup {
  const void *A[kGrads], *B[kGrads];
  float* C[kGrads];
  int M[kGrads], N[kGrads], tm[kGrads], tn[kGrads], first[kGrads + 1], K;
};
void gemm_mfma_grads(hipStream_t s, int64_t K, const GradItem (&items)[kGrads]);
void gemm_f32_grads(hipStream_t s, int64_t K, const GradItem (&items)[kGrads]);

int attention_fwd(hipStream_t s, int dtype, int B, int T, int H, int Hkv, int hd, const void* qkv, void* o, float* lse);
// rope_tab (may be null): if given, q and k in qkv are rotated vectors and dqkv is returned with respect to
// the vectors before the rotation
int attention_bwd(hipStream_t s, int dtype, int B, int T, int H, int Hkv, int hd, const void* qkv, const void* o,
                  const float* lse, const void* do_, void* dqkv, float* delta, const float* rope_tab = nullptr);
// C = A*B^T with the rotation applied to C on the way out (same result as gemm op 0 followed by rope)
int gemm_rope(hipStream_t s, int dtype, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C,
              const RopeArgs& ra, float rope_theta);

int cu_count();   // compute units of the current device
// How a product is divided: edge of its tiles (0: the plain kernel), their number, workgroups
struct GemmShape { int tile, tiles, workgroups; };
GemmShape gemm_mfma_shape(int op, int64_t M, int64_t N, int64_t K, int epi);
bool gemm_f32_far(int op, int64_t M, int64_t N, int64_t K, int epi);   // not for gemm_f32_grads
GemmShape gemm_f32_shape(int op, int64_t M, int64_t N, int64_t K, int epi);   // of 128 x 64 the shorter edge
// building blocks the dispatchers choose between
void gemm_simple(hipStream_t s, int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C, const void* R);
// float, any shape; rope / epi / aux as for gemm_mfma
void gemm_f32(hipStream_t s, int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C, const void* R,
              const RopeArgs* rope, int epi, void* aux);
bool gemm_mfma_supported(int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, const void* C,
                         const void* R);
void gemm_mfma(hipStream_t s, int op, int64_t M, int64_t N, int64_t K, const void* A, const void* B, void* C,
               const void* R, const RopeArgs* rope = nullptr, int epi = 0, void* aux = nullptr);
// the feed-forward projections with the SwiGLU arithmetic in their epilogues (bf16, matrix cores):
//   forward   gu[R, 2h] = hn[R, d] wgu[2h, d]^T  and  act[R, h] = silu(gate) * up
//   backward  dgu[R, 2h] = swiglu'(dy[R, d] wd[d, h]; gu)            (d(act) is never stored)
bool gemm_swiglu_supported(bool bwd, int64_t R, int64_t h, int64_t d, const void* X, const void* W, const void* gu,
                           const void* other);
void gemm_mfma_swiglu_fwd(hipStream_t s, int64_t R, int64_t h, int64_t d, const void* hn, const void* wgu, void* gu, void* act);
void gemm_mfma_swiglu_bwd(hipStream_t s, int64_t R, int64_t h, int64_t d, const void* dy, const void* wd, const void* gu, void* dgu);
// the same two steps whatever the dtype and shape: fused where the matrix-core path takes them, else the plain
// product with the pointwise kernel after it; da_tmp [R, h]: scratch for the unfused backward path
int ffn_up_fwd(hipStream_t s, int dtype, int64_t R, int64_t h, int64_t d, const void* hn, const void* wgu, void* gu, void* act);
int ffn_down_bwd(hipStream_t s, int dtype, int64_t R, int64_t h, int64_t d, const void* dy, const void* wd, const void* gu,
                 void* dgu, void* da_tmp);
bool attention_flash_supported(int B, int T, int H, int Hkv, int hd);
void attention_flash_fwd(hipStream_t s, int B, int T, int H, int Hkv, int hd, const void* qkv, void* o, float* lse);
void attention_flash_bwd(hipStream_t s, int B, int T, int H, int Hkv, int hd, const void* qkv, const void* o,
                         const float* lse, const void* do_, void* dqkv, float* delta, const float* rope_tab);

// ---- optional per-launch timing (see sp_prof_begin); classes:
enum { PROF_GEMM_NT = 0, PROF_GEMM_NN = 1, PROF_GEMM_TN = 2, PROF_ATTN_FWD = 3, PROF_ATTN_DELTA = 4, PROF_ATTN_DQ = 5,
       PROF_ATTN_DKV = 6, PROF_GEMM_PLAIN = 7, PROF_ATTN_PLAIN = 8,
       // bandwidth-bound kernels: the work recorded is algorithmic bytes, not flops
       PROF_RMSNORM_FWD = 9, PROF_RMSNORM_BWD = 10, PROF_CROSS_ENTROPY = 11, PROF_COPY_ROWS = 12, PROF_SWIGLU = 13,
       PROF_CLASSES = 14 };
int prof_start(int cls, hipStream_t s);
void prof_stop(int idx, hipStream_t s, double flops);

}  // namespace sp
