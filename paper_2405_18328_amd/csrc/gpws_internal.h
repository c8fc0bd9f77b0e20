// Internal declarations shared by the translation units of libgpws (gfx950 only).
#ifndef GPWS_INTERNAL_H
#define GPWS_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/gpws.h"

// ---------------------------------------------------------------------------
// Geometry of the fp32 tile pass.  A wavefront (64 lanes) owns MI sub-tiles of 32
// rows i and walks over the columns j in chunks of 32; one 32x32 tile of
// pairs is one v_mfma_f32_32x32x2_f32 accumulator (16 VGPRs per lane).
// ---------------------------------------------------------------------------
constexpr int GP_CHUNK = 32;          // rows per packed operand chunk
constexpr int GP_WAVES = 4;           // wavefronts per workgroup
constexpr int GP_THREADS = 64 * GP_WAVES;
constexpr int GP_ROW_ALIGN = 512;     // packed operand arrays are padded to this many rows
constexpr int GP_VEC_PAD = 4;         // solver arrays are padded to a multiple of 4 rows (float4 streams)
constexpr float GP_PAD_NORM = 1.0e30f; // squared norm given to padding rows of XA (phi underflows to 0)
constexpr int GP_PACK_SLACK = 256;    // floats allocated past the packed arrays: staging loads overrun by < 256
constexpr float GP_PAD_NORM_H = 60000.0f;  // same for the fp16 operands (must fit fp16)
enum { GP_PATH_PENDING = -1, GP_PATH_FP32 = 0, GP_PATH_F16X2 = 1, GP_PATH_F16X3 = 2 };
// fp16 distance pieces: two pieces carry 22 bits, so r^2 has an absolute error ~2^-22 (|xs_i|^2+|xs_j|^2);
// past this squared norm three pieces (33 bits) are used, and past fp16's range the fp32 MFMA path
constexpr float GP_NORM_X2_MAX = 64.0f;
constexpr float GP_NORM_X3_MAX = 16000.0f;
constexpr int GP_FLUSH_CHUNKS = 1024; // tile kernels add their fp32 accumulators into OUT every this many column chunks (power of 2)
constexpr int GP_PROF_MAX = 8192;     // event pairs available to gp_profile
// Regions of the context's pinned host block (64 KB).  A region the host writes before an asynchronous
// host-to-device copy must not be written again until that copy has run, so gp_set_theta has one no
// other call touches (it waits for the stream before writing it); the solvers stage their tolerances
// and read results back in the first region and synchronise before they return.
constexpr size_t GP_PIN_SOLVER = 0;       // flags, tolerances in, residuals / gradient sums out
constexpr size_t GP_PIN_THETA = 16384;    // gp_set_theta: 1/ell, a, sigma staged for the device copy
constexpr size_t GP_PIN_NORM = 24576;     // largest scaled squared norm read back
constexpr size_t GP_PIN_POST = 32768;     // flags the solvers' finalise kernels post for the host loop

// Operands of the distance contraction, packed so that one wave-wide dword
// load is one MFMA operand: P[(chunk*KS + ks)*64 + lane] holds, for row
// 32*chunk + lane%32, the component k = 2*ks + lane/32 of
//   XA (column side j): [ xs_j(0..d-1), |xs_j|^2, 1, 0.. ]
//   XB (row side i)   : g * [ -2 xs_i(0..d-1), 1, |xs_i|^2, 0.. ]
// with xs = (x - mean)/ell and g = -log2(e)/2 (SE) or 3 (Matern-3/2), so that
// XA_j . XB_i = g * r^2_ij comes straight out of the MFMA chain.
// Column splits already worked out for a shape of product: a solver asks for the same few thousands of times.
struct SplitMemo {
  int64_t rows, chunks;
  int t, XP, JS, CG;
  bool wide;
};

struct gp_ctx {
  int kernel;
  int64_t n;
  int d;
  int KS;                 // k-steps (of 2) of the distance chain, bucketed
  int64_t n_pad;          // n rounded up to GP_ROW_ALIGN
  hipStream_t stream;
  const float* dX;        // caller-owned
  unsigned packed;        // bit 1 << GP_PATH_*: what that path reads is packed for the current theta
  float* dXA;             // fp32 path: n_pad/32 * KS * 64; one block with dXB, NULL until a theta or a prediction asks for that path
  float* dXB;
  float* dXs;             // scaled centred inputs, row-major n x d (gradient pass)
  unsigned long long* dMaxNorm;   // a tag and below it the bit pattern of the largest |xs_i|^2 packed under it (device)
  unsigned norm_seq;      // the latest tag
  // split-fp16 operands of the tile pass on two and three pieces (dist_f16.h), column and row side, 16-byte units
  // [(16 points)*groups + group]*64 + lane: lane l holds slots 8 (l/16) .. + 7 of point l % 16
  void* dDist;            // one block: those on two pieces, dDistSlots and dCI
  void* dDA[2];           // [1]: NULL until a theta or a prediction asks for three pieces; one block with dDB[1], dXAh[2] and dXBh[2]
  void* dDB[2];
  void* dDistSlots;       // what stands where in them (gp_dist_slots)
  float* dCI;             // gamma |xs_i|^2, [n_pad]
  // split-fp16 operands of the gradient pass: two or three pieces (hi, mid, lo) per side, 16-byte units
  // [(chunk*KH + kh)*64 + lane], element e of a unit = component 16 kh + 8 (lane/32) + e
  void* dXAh[3];
  void* dXBh[3];
  int grad_pieces;        // how many of them are packed for the current theta
  int KH;                 // 16-wide k-steps of the fp16 distance chain, bucketed
  int XP;                 // pieces used per operand of the distance chain (2 or 3)
  int path;               // GP_PATH_* chosen by gp_set_theta
  int path_forced;        // -1, or a GP_PATH_* forced through the GPWS_PATH environment variable
  bool f16_ok;            // false when d + 3 components do not fit the widest fp16 operand bucket (SE, d = 126)
  float max_norm;         // host copy of max_i |xs_i|^2
  unsigned* dColmax;      // GP_MAX_T words, zero between calls: column maxima of gp_kmv in accumulation
  int colmax_dirty;       // how many of them may be set: a call ended with an error, or was a prediction that turned to the fp32 path
  double* dMean;          // d column means of X
  double* dTheta;         // device copy: 1/ell (d), then a, sigma
  bool created, theta_set;
  double xabs[GP_MAX_D];  // max_i |x_ik - mean_k| per dimension (host copy, fixed at gp_create)
  double xvar[GP_MAX_D];  // mean_i (x_ik - mean_k)^2
  double ell[GP_MAX_D];
  double a, sigma;
  // lazily grown scratch for split-column partial sums of gp_kmv / gp_mll_grad
  void* dScratch;
  size_t scratch_bytes;
  bool grad_tight;        // the scratch of gp_mll_grad did not fit once: it makes do with less
  void* static_scratch;   // this device's address of the file-scope scratch gp_kmv_static uses (never freed)
  // small device + pinned host blocks for scalars
  double* dRed;           // reduction partials
  size_t red_bytes;
  void* hPinned;          // pinned host staging for scalar read-back
  void* dPinned;          // the same block as the device addresses it (kernels post small results there)
  size_t pinned_bytes;
  int num_cu;
  // event pairs bracketing kernel launches while profiling is on (gp_profile): prof_mask has bit k set
  // when launches of kind k (GP_PROF_* of gpws.h) are bracketed
  unsigned prof_mask;
  int prof_count;
  hipEvent_t* prof_ev;    // 2 * GP_PROF_MAX events, created on first enable
  unsigned char* prof_kind;   // kind of every recorded pair
  SplitMemo split_memo[4];
  int split_next;         // entry to overwrite next
  char err[256];
};

// Row side of a rectangular product K(X*, X) V: m other points packed like the context's own rows
// (same centring, lengthscales and scaling).  NULL everywhere below means the square product.
struct KmvRows {
  int64_t m;
  const float* XB;        // fp32 packed row operands, [m_pad/32][KS][64]
  const void* DB[2];      // fp16 row operands on two and three pieces, as in the context
  const float* X;         // the points themselves, and whether a launch that reads them is behind the one their norm was posted by
  bool reads_X;
  bool v_prepared;        // the column maxima of V are in the context's words, or its one column is in the scratch
  const float* CI;
  const int* gather;      // fp16 paths: row i is the row gather[i] of DB and CI, which hold the context's n points; NULL: i
  int path;               // GP_PATH_* to use (covers the norms of both point sets); GP_PATH_PENDING: gp_rows_path will tell
};

// Column-split partial results of a product whose final sum the caller takes over (the CG dot-product
// kernel adds the partials while it reads H P anyway): OUT_ic = sum_k part[k stride + i t + c].
// JS == 1 means the launcher wrote OUT itself.
struct KmvDeferred {
  const float* part;
  int64_t stride;
  int JS;
};

// Contraction restricted to the context's points 32 chunk0 .. min(n, 32 (chunk0 + nchunks)) - 1 (a
// column block of K): OUT = K[:, window] V[window, :].  V is still the full-height n x t array; only
// the window's rows are read.  Coincident pairs get no special treatment (as in a rectangular product)
// and no noise term can be asked for.
struct KmvWindow {
  int chunk0;
  int nchunks;
};

int gp_fail(gp_ctx* ctx, int code, const char* fmt, ...);
#define GP_HIP(ctx, call)                                                              \
  do {                                                                                 \
    hipError_t e__ = (call);                                                           \
    if (e__ != hipSuccess)                                                             \
      return gp_fail(ctx, GP_ERR_HIP, "%s failed: %s", #call, hipGetErrorString(e__)); \
  } while (0)

// Bracket one kernel launch of the given kind with an event pair when that kind is being profiled:
//   const bool pr = gp_prof_begin(ctx, kind);  launch;  gp_prof_end(ctx, pr);
inline bool gp_prof_begin(gp_ctx* ctx, int kind) {
  if (!((ctx->prof_mask >> kind) & 1u) || ctx->prof_count >= GP_PROF_MAX) return false;
  if (hipEventRecord(ctx->prof_ev[2 * ctx->prof_count], ctx->stream) != hipSuccess) return false;
  ctx->prof_kind[ctx->prof_count] = (unsigned char)kind;
  return true;
}
inline void gp_prof_end(gp_ctx* ctx, bool begun) {
  if (!begun) return;
  if (hipEventRecord(ctx->prof_ev[2 * ctx->prof_count + 1], ctx->stream) == hipSuccess) ++ctx->prof_count;
}

int gp_ks_bucket(int d);   // -1 if d is out of range
int gp_ensure_scratch(gp_ctx* ctx, size_t bytes);

// ---- prep_kernels.hip
int gp_launch_column_means(gp_ctx* ctx);
int gp_launch_pack(gp_ctx* ctx, int path, bool want_norm);     // for a new theta: what `path` reads
int gp_need_path(gp_ctx* ctx, int path);                       // and another one too, unless it is there
// waits for the largest scaled squared norm of the latest packing that was asked for it
int gp_wait_norm(gp_ctx* ctx, const char* who, float* norm);
// packs m other points (device, row-major m x d) against the context's centring and theta into
// caller-provided buffers sized by gp_pack_rows_bytes; fills rows.  The path follows from the larger of the two sets' scaled
// norms: it stays pending until gp_rows_path waits for that norm, so that launches which do not depend on it go first
size_t gp_pack_rows_bytes(const gp_ctx* ctx, int64_t m);
constexpr int GP_DIST_LIST_EXTRA = 6;
int gp_dist_slots(const gp_ctx* ctx, unsigned short* slots);     // fills (or NULL: counts) the table the packing kernel works from
size_t gp_dist_bytes(const gp_ctx* ctx, int XP, int64_t rows);   // of one side's operands of the tile pass, rows a multiple of 32
size_t gp_grad_piece_bytes(const gp_ctx* ctx);                   // of one piece of one side's operands of the gradient pass
// dV, kmv_scratch: as gp_kmv_launch will get them; what V needs first is prepared in the same launch (rows->v_prepared)
int gp_pack_rows(gp_ctx* ctx, const float* dXstar, int64_t m, void* buf, KmvRows* rows, const float* dV, int64_t ldv, int t, void* kmv_scratch);
int gp_rows_path(gp_ctx* ctx, KmvRows* rows);
int gp_rows_x3(gp_ctx* ctx, KmvRows* rows);      // operands on three pieces, of both sides

// ---- tile_pass.hip
struct KmvPlan {
  int MI;        // 32-row sub-tiles per wave
  int JS;        // column-range splits
  int row_blocks;
  int cps;       // chunks per split
};
KmvPlan gp_plan_kmv(const gp_ctx* ctx, int64_t rows, int64_t col_chunks = 0);   // col_chunks = 0: all of the context's
size_t gp_kmv_scratch_bytes(const gp_ctx* ctx, int t);   // square product, worst case over the paths gp_set_theta may choose
size_t gp_kmv_least_scratch_bytes(const gp_ctx* ctx, int t);   // the least the square product can run with (its rows in panels)
size_t gp_kmv_rect_scratch_bytes(const gp_ctx* ctx, int t, int64_t rows);
size_t gp_kmv_window_scratch_bytes(const gp_ctx* ctx, int t, int col_chunks);   // product over any column window of at most that many chunks
// OUT = K V (+ sigma^2 V).  colmax: optional device array of t bit patterns of max_i |V_ic| that the
// caller already holds (the split-fp16 path then skips its own reduction over V); NULL otherwise.
// rows: NULL, or the row side of a rectangular product (add_noise must then be 0).
// defer: NULL, or where to report column-split partials instead of summing them into OUT.
int gp_kmv_launch(gp_ctx* ctx, const float* dV, int64_t ldv, int t, float* dOut, int64_t ldo,
                  int add_noise, void* scratch, size_t scratch_bytes, const unsigned* colmax,
                  KmvRows* rows = nullptr, KmvDeferred* defer = nullptr, const KmvWindow* win = nullptr);

// ---- tile_pass_f16.hip
int gp_kh_bucket(int d, int kernel);
// Number of equal ranges the column chunks are cut into, given the row blocks, the workgroups a compute unit holds and the
// waves that share a workgroup's rows (see the definition); *cost: about what the launch takes, in us.
int gp_column_splits(int64_t row_blocks, int64_t chunks, int num_cu, int per_cu, int cg, double chunk_us, double stream_us, double image_us,
                     int max_splits, double* cost);
size_t gp_kmv_f16_scratch_bytes(const gp_ctx* ctx, int t, int64_t rows, int64_t col_chunks = 0);
size_t gp_kmv_f16_least_scratch_bytes(const gp_ctx* ctx, int t);   // square product with its rows in panels
// GP_OK, an error, or GP_TO_FP32: the rows' path was pending and turned out to be the fp32 one (nothing is in OUT yet)
constexpr int GP_TO_FP32 = 1000;
int gp_kmv_launch_f16(gp_ctx* ctx, const float* dV, int64_t ldv, int t, float* dOut, int64_t ldo,
                      int add_noise, void* scratch, size_t scratch_bytes, const unsigned* colmax,
                      KmvRows* rows, KmvDeferred* defer, const KmvWindow* win);

// The tile passes alone, for solvers that keep their vectors column by column and pack operands themselves: the
// sums of image k, column c lie at images[(k t + c) ld + i], a^2 included, no noise term; rows from n up to the next
// multiple of 32 hold nothing of meaning.  f16 paths only.
struct KmvPacked {
  const void* VP;          // operands of every column pass, one after the other (gp_packed_units 16-byte units)
  const float* VY;         // the vector-ALU column (column 0 where vec_columns(t)), zero up to the next multiple of 32 rows
  const unsigned* colmax;  // bit patterns of the column maxima the operands were scaled by
  float* images;
  int64_t ld;              // rows per column, a multiple of 32
  const int* done;         // device flag that turns the launch into a no-op, or NULL
};
// Contraction over the columns of one block of consecutive points, chosen on the device: points sel block ..
// sel block + block - 1.  Operands and the vector-ALU column are counted from the chunk the block starts in, zero for
// the points of its first and last chunk that are not the block's.
struct KmvBlock {
  const int* sel;
  int block;
  int nchunks;   // chunks a block can touch
};
int64_t gp_packed_units(int t, int64_t nchunks);
int gp_packed_images(const gp_ctx* ctx, int t, int64_t rows, int64_t col_chunks = 0);   // most images such a product leaves
// gather: device, nrows indices of the context's points that are the rows of the product (NULL: all n, in order)
int gp_kmv_packed(gp_ctx* ctx, int t, const KmvPacked& pk, const int* gather, int64_t nrows, const KmvBlock* win, int* images);

int gp_colmax_blocks(const gp_ctx* ctx, int t);
int gp_clear_maxima(gp_ctx* ctx, int t);
bool gp_short_pack(const gp_ctx* ctx, int t);
size_t gp_vec_column_offset(const gp_ctx* ctx, int t);     // of the vector-ALU column in the scratch of a product
// colmax[c] = bit pattern of max_i |V_ic| for c < t, stream-ordered; optionally the same for a second
// n x t matrix in the same launch.  cleared = true: the caller has already zeroed the output words.
int gp_launch_colmax(gp_ctx* ctx, const float* dV, int64_t ldv, int t, unsigned* colmax, const float* dV2 = nullptr,
                     int64_t ldv2 = 0, unsigned* colmax2 = nullptr, bool cleared = false);

// ---- ap_kernels.hip
size_t gp_ap_workspace_bytes_impl(const gp_ctx* ctx, int t, int block);
int gp_ap_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv, int t,
              const float* h_tol, int block, int max_iters, void* dWork, size_t work_bytes, int* h_iters,
              int* h_kmv_count, float* h_relres, int* h_picks);

// the inverse of every diagonal block of H (fp32, layout of ap_inverse.h), for the current theta; scratch: batch blocks of BP^2 doubles
// (A, W, T) and batch BP 64 doubles (DI); *breakdown is raised when a block is not positive definite
int gp_ap_inverses(gp_ctx* ctx, int block, int nb, int BP, int batch, float* Hinv, double* A, double* W, double* T, double* DI,
                   int* breakdown);

// ---- ap_columns.hip: the same solve for problems up to this size and this many blocks on the f16 product paths
constexpr int64_t AP_COLUMNS_MAX_N = 65536;
constexpr int AP_COLUMNS_MAX_BLOCKS = 256;
bool gp_ap_by_columns(const gp_ctx* ctx, int block);
size_t gp_ap_columns_workspace_bytes(const gp_ctx* ctx, int t, int block);
int gp_ap_columns_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv, int t,
                      const float* h_tol, int block, int max_iters, void* dWork, int* h_iters, int* h_kmv_count,
                      float* h_relres, int* h_picks);

// ---- sgd_kernels.hip
size_t gp_sgd_workspace_bytes_impl(const gp_ctx* ctx, int t, int batch);
int gp_sgd_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv, int t,
               const float* h_tol, const int* dBatches, int batch, int max_iters, double lr, double momentum,
               void* dWork, size_t work_bytes, int* h_iters, int* h_kmv_count, float* h_relres);

// ---- sgd_columns.hip: the same solve for problems up to this size on the f16 product paths
// Its vector work takes one compute unit per column, a time that grows with n but not with t up to 256, the streaming
// kernels' with n t.  Per step with batches of 1000, Matern-3/2, d = 26, streaming -> columns:
//   n = 65536   t = 1  83 -> 50 us, t = 17  76 -> 72, t = 33  84 -> 79, t = 65  116 -> 97
//   n = 81920   t = 1  92 -> 59,    t = 17  84 -> 84, t = 33  94 -> 94, t = 48 109 -> 103
//   n = 131072  t = 1 114 -> 83,    t = 17 109 -> 126, t = 48 142 -> 153, t = 65 170 -> 164, t = 97 267 -> 255
// (for a single column the streaming kernels have too few workgroups).
constexpr int64_t SGD_COLUMNS_MAX_N = 131072, SGD_COLUMNS_FEW_N = 81920;
bool gp_sgd_by_columns(const gp_ctx* ctx, int t);
size_t gp_sgd_columns_workspace_bytes(const gp_ctx* ctx, int t, int batch);
int gp_sgd_columns_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv, int t,
                       const float* h_tol, const int* dBatches, int batch, int max_iters, double lr, double momentum,
                       void* dWork, int* h_iters, int* h_kmv_count, float* h_relres);

// ---- cg_kernels.hip
int gp_cg_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv,
              int t, const float* h_tol, int max_iters, void* dWork, size_t work_bytes,
              int* h_iters, int* h_kmv_count, float* h_relres);
size_t gp_cg_workspace_bytes(const gp_ctx* ctx, int t);

// ---- cg_columns.hip: the same solve for problems up to this size on the f16 product paths
constexpr int64_t CG_COLUMNS_MAX_N = 65536;
bool gp_cg_by_columns(const gp_ctx* ctx);
size_t gp_cg_columns_workspace_bytes(const gp_ctx* ctx, int t);
int gp_cg_columns_run(gp_ctx* ctx, const float* dB, int64_t ldb, const float* dX0, float* dV, int64_t ldv, int t,
                      const float* h_tol, int max_iters, void* dWork, int* h_iters, int* h_kmv_count, float* h_relres);

// ---- grad_pass.hip
int gp_grad_run(gp_ctx* ctx, const float* dV, int64_t ldv, const float* dB, int64_t ldb, int t,
                double* h_grad);
// Row blocks of W chunks (the first ones) whose columns, from the block's own first chunk on, have more than js pieces of cps
// chunks: row block rb has nchunks - rb W chunks.  W is 4 or 8.
__host__ __device__ inline int gp_grad_rows_with_piece(int js, int nchunks, int cps, int W) {
  return (nchunks - js * cps + W - 1) >> (W == 8 ? 3 : 2);
}
// fp64 reduction of one right-hand-side block's tile-pass output OUT into acc[d + 2] (part: G x (d + 2) workgroup
// partials); first_block adds the sigma component sum_i w_ii.  tri_W = 0: OUT[JS][n][nq].  Else only the tiles on and
// above the diagonal were worked on, the columns of a row block of tri_W chunks in pieces of at most tri_cps chunks, and
// image k of OUT has the rows of the row blocks with that piece alone
int gp_grad_reduce_launch(gp_ctx* ctx, const float* OUT, int JS, int nq, const float* dV,
                          int64_t ldv, const float* dB, int64_t ldb, int t, float half_w, float probe_w,
                          int first_block, double* part, int G, double* acc, int tri_W = 0, int tri_cps = 0);

// ---- grad_pass_f16.hip
int gp_grad_run_f16(gp_ctx* ctx, const float* dV, int64_t ldv, const float* dB, int64_t ldb, int t,
                    double* h_grad);

#endif
