// Internal declarations shared by the translation units of the library
// (host launchers only; kernels stay private to their .hip file).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

struct abs_ctx;

namespace absk {

typedef uint16_t bf16_t;   // raw bfloat16 bits in memory

enum { ACT_NONE = 0, ACT_RELU = 1, ACT_GELU = 2 };
enum { OPT_SGD = 0, OPT_SHB = 1, OPT_ADAMW = 2, OPT_ADAGRAD = 3 };

// Epilogues of the grouped GEMM  C[g][m][n] = sum_k A[g][m][k] * B[g][n][k].
enum {
  EPI_FWD_ACT = 0,  // C = bf16/f32 phi(acc + bias[n]); C2 = phi'(acc + bias[n]) if C2 != null
  EPI_LOGITS = 1,   // C(f32) = acc + bias[n]
  EPI_BWD = 2,      // C = acc * E[m][n]   (act == RELU: E > 0 ? 1 : 0 ; GELU: E itself)
  EPI_WGRAD = 3,    // C(f32) = alpha * acc ; C2(bf16) = same, rounded, if C2 != null
  EPI_IPDOT = 4,    // part[tile_n][m] = sum_{n in tile} E[m][n] * (acc + bias[n])
  EPI_WGRAD_UPD = 5 // internal to the bf16 family: EPI_WGRAD with the optimizer step in the epilogue (GemmP::upd_x)
};

// The softmax cross-entropy head in the epilogue of an EPI_LOGITS launch (gemm_head_fits): instead of the logits the launch
// stores delta = p - e_y (rows of ldd elements, pad columns zero), dn[g][i] = ||stored delta_i||^2 and loss[g][i].
struct HeadP {
  const int32_t *y, *idx;      // labels [N]; row i of group g carries label y[idx[g * ldi + i]] (null y: no head)
  int N, ldi, ldd;
  void *D; long long sDg;
  float *dn, *loss; long long sNg;
};

struct GatherP {
  const void *X; int d, N;               // dataset: N rows of d elements
  const int32_t *idx; int ldi, b, groups;
  void *A0; long long sA0g; int ldo;
  float *an0; long long sNg;
  const int *rows;                       // ragged groups (optional): rows[g] <= b of them
};
inline long long gather_blocks(const GatherP &p) { return (long long)((p.b + 3) / 4) * p.groups; }
constexpr long long GATHER_RIDES = 1024;       // blocks that may ride with another launch
inline bool gather_ok(const GatherP &p) {
  return p.X && p.idx && p.A0 && p.an0 && p.N > 0 && p.d > 0 && p.ldo >= p.d && p.ldi >= p.b && gather_blocks(p) <= GATHER_RIDES;
}
// Which launch of the step takes the gather along (GemmP::gather), the first layer's contraction (1) or the logits (2), or none (0);
// the first layer then reads its rows from the dataset (GemmP::aidx).
int gather_rides(int is_bf16, int L, int b, const int *dims, int groups, long long N, const int *rows_host);

struct GemmP {
  const void *A, *B;           // operands (bf16 bits or float, by kernel family)
  long long sAg, sBg;          // group (replica) strides in elements
  int lda, ldb;                // leading dimensions in elements
  int a_trans, b_trans;        // 0: memory is [row][k] (k contiguous); 1: memory is [k][row]
  int Md, Nd, Kd, groups;
  void *C;  long long sCg;  int ldc;     // main output
  void *C2; long long sC2g; int ldc2;    // optional second output
  const float *bias; long long sBiasg;   // per-column vector (may be null)
  const void *E; long long sEg; int lde; // elementwise operand of the epilogue
  HeadP head;                  // EPI_LOGITS (optional)
  const GatherP *gather;       // EPI_FWD_ACT, EPI_LOGITS (optional, host): the gather's blocks ride behind the tiles (bf16: gemm_small.hip)
  const int32_t *aidx;         // EPI_FWD_ACT, EPI_LOGITS (optional): row i of group g is row aidx[g * aldi + i], clamped, of the
  int aN, aldi;                //   aN rows at A (sAg 0; bf16: lda a multiple of 8, gemm_small.hip or 64 x 128 tiles)
  float *part; long long sPartg; long long sPartTile; // row partials: part[g][tile_n][m]
                               //   EPI_IPDOT: the row dots; EPI_FWD_ACT / EPI_BWD (bf16 family, optional):
                               //   sum over the tile's columns of the squared stored outputs
  float *part2;                // EPI_IPDOT (optional): likewise the sum over the tile's columns of E[m][n]^2
  float *cpart; long long sCpartg;   // EPI_BWD (bf16 family, optional): column partials
                               //   cpart[g][tile_m * WM + wave_m][n] = sum over the wave's rows of the stored outputs
  float alpha;
  int act;
  int pad_to_ld;               // also write zeros to columns [Nd, ldc) of C (and C2)
  // Ragged groups (optional): rows[g] (device) replaces Md (rows_is_k == 0) or Kd (rows_is_k == 1,
  // where alpha becomes 1 / rows[g]) for group g; Md / Kd then hold the largest count, which sizes
  // the grid of the fp32 and of the 32-row kernels.  Memory beyond a group's own rows is neither read nor written.
  const int *rows;
  int rows_is_k;
  const int *rows_host;        // the same counts on the host (bf16 family): the tile shape goes by them (weight gradients: optional) and, rows_is_k == 0, the grid
  // Optional (device, EPI_WGRAD of the bf16 family): the order in which the launch walks the groups.  Work-group ids are dealt
  // to the XCDs in contiguous ranges of groups, so with ragged groups the host orders them such that every
  // XCD gets about the same number of rows to reduce over.
  const int *gperm;
  int accumulate;              // EPI_WGRAD: C = alpha * acc + C  (micro-batch accumulation)
  // Split reduction (EPI_WGRAD of the bf16 family, optional): ksplit > 1 cuts k into ksplit slices of
  // kchunk elements; slice sp of group g writes its raw partial product to
  // kpart[(g * ksplit + sp) * Md * Nd] (row-major, ld = Nd) and C / C2 are left to launch_splitk_finish.
  int ksplit, kchunk;
  float *kpart;
  int fine;                    // bf16 family, EPI_WGRAD launches of tile shape 1: 1: 64 x 128 tiles instead of 128 x 128 (two stages); 2: 256 x 256, ksplit > 1
  int f32_tile;                // fp32 family, EPI_WGRAD: extent of the tile, 16, 32 or 64 (0: by the number of outputs)
  // fp32 family, EPI_WGRAD without a split (optional): rowsum[g * sRowsumg + m] = alpha * sum_k A[m][k] (+ the old value
  // if accumulate): the bias gradient beside the weight gradient
  float *rowsum; long long sRowsumg;
  // Optimizer step inside the epilogue (EPI_WGRAD of the bf16 family, optional: upd_x != null; needs ksplit <= 1,
  // accumulate == 0 and ldc, the layer offsets and the group stride multiples of 4).  The finished gradient entry
  // g = alpha * acc is not stored in C; instead the parameter at the same offset of upd_x (and its state in
  // upd_v / upd_m, its bf16 shadow in upd_shadow; all laid out like C: group stride sCg, leading dimension ldc)
  // takes its step.  C2 (the bf16 copy of the gradient) is still written.  Every wavefront leaves the sum of its
  // squared gradient entries in upd_sq[g * upd_sSqg + upd_slot0 + tile * waves + wave] (tile = tm * tilesN + tn):
  // the layer's share of ||gbar||^2, added up later in index order.
  float *upd_x, *upd_v, *upd_m;
  bf16_t *upd_shadow;
  int upd_opt;
  float upd_lr, upd_momentum, upd_beta1, upd_beta2, upd_eps, upd_wd, upd_c1, upd_c2;
  const float *upd_scal;       // optional (device): {lr, c1, c2} read from memory (replayable launches)
  float *upd_sq; long long upd_sSqg; int upd_slot0;
  // EPI_WGRAD of the bf16 family without a split or a step (optional): the sum of the squared entries of every wavefront's
  // part of the output in sq64[g * sSq64g + tile * waves + wave].  C may then be null: only C2 and these sums are written.
  double *sq64; long long sSq64g;
};

// bf16 MFMA family (gemm_bf16.hip).  Returns the number of column partials that
// EPI_IPDOT writes per row (tiles along n) for the tile shape it picks.
hipError_t launch_gemm_bf16(const GemmP &p, int epi, hipStream_t s);
// EPI_WGRAD of n layers whose tile shape (gemm_bf16_wgrad_shape) is `shape`, 1 or 3, in one launch per eight layers: all of
// them with the optimizer step in the epilogue or none
struct StepTail;
hipError_t launch_wgrad_many(const GemmP *p, int n, int shape, hipStream_t s, const StepTail *tail = nullptr);
int gemm_bf16_ipdot_parts(int Nd);
// Exact number of row partials (tiles along n) and of column-partial rows (tiles along m times
// wave rows) that launch_gemm_bf16 writes for epilogue epi (forward, logits, backward-data, inner products) of an
// Md x Nd output; the rows of a column partial's tile and the partials per tile.
int gemm_bf16_row_parts(int epi, int Md, int Nd, int groups, const int *rows_host);
int gemm_bf16_col_parts(int epi, int Md, int Nd, int groups, const int *rows_host);
void gemm_bf16_col_part_shape(int epi, int Md, int Nd, int groups, const int *rows_host, int *tile_m, int *parts_per_tile);
// Floats per group that hold the row partials of forward / backward-data launches over any b <= cap rows when
// partials lie b (rounded up to 64) apart.
size_t gemm_bf16_row_part_floats(int Nd, int groups, int cap);
// Tile shape the bf16 family uses for an Md x Nd output over `groups` replicas: 0 = 128x64, 1 = 128x128, 2 = 256x256,
// 4 = 64x128 with a six-stage ring (outputs of at most 64 rows; 3 is a weight-gradient shape, see below),
// 5 = 32-row tiles of gemm_small.hip (forward, logits and backward-data launches that would leave most CUs idle).
// rows_host (here and below): the rows of ragged groups, at most Md (weight gradients: Kd) each, or null.
int gemm_bf16_tile_shape(int epi, int Md, int Nd, int groups, const int *rows_host);
hipError_t launch_gemm_small(const GemmP &p, int epi, hipStream_t s);
// Passes of a step whose launches are all of them 32-row tiles, in one launch: forward of layers 1 .. L - 1 (the first with GemmP::aidx),
// logits with the head, backward-data of layers L .. 2, and the gather.  count: `words` ints (small_chain_words) for each replica and 32
// rows, zero before the first launch and after each.
struct SmallChain {
  enum { MAXL = 4, MAX_CHAINS = 224 };
  enum { POLLS = 1 << 22 };                      // of a tile's wait, at about a microsecond each: only a mistake in here lets it last that long
  int L, words, polls;
  int *count, *failed;                           // failed (pinned host memory, as the device sees it): set to 1 if a wait gave up
  int end[2 * MAXL - 2], chains;                 // set by the launcher: tiles of a chain up to and with each pass (logits with layer L's backward-data)
  GatherP gather;
  GemmP p[2 * MAXL - 1];
};
static_assert(sizeof(SmallChain) <= 4096, "kernel arguments");
int small_chain_words(int L, const int *dims);
void set_chain_polls(abs_ctx *c, int polls);       // (for tests of a wait that gives up)
bool small_chain_fits(int L, const int *dims, int b, int groups, long long N, const int *rows_host);       // (bf16) where that is the way
hipError_t launch_small_chain(SmallChain &c, hipStream_t s);
// ---- mlp_rows.hip ------------------------------------------------------------
// The same passes with a block of `rows` rows of one replica to a work-group, which walks all layers (p, gather as in SmallChain; one row
// partial and one column partial to a block).  mlp_rows_block: the rows to a block where that is the faster way, else 0.
struct MlpRows {
  enum { MAXL = 4, MAX_CLASSES = 128, MAX_INPUTS = 896 };
  int L, rows;
  int per, blocks, share, weight_bytes;          // set by the launcher: blocks to a replica, in all, to an XCD; from the first layer's weights to the last's end
  GatherP gather;
  GemmP p[2 * MAXL - 1];
};
static_assert(sizeof(MlpRows) <= 4096, "kernel arguments");
int mlp_rows_block(int L, const int *dims, int b, int groups, long long N);
hipError_t launch_mlp_rows(MlpRows &c, hipStream_t s);

// ---- gemm_bf16.hip -----------------------------------------------------------
bool gemm_bf16_operands_ok(const GemmP &p, int epi);       // what every launch of the family relies on
// Whether an EPI_LOGITS launch can carry the softmax head: a row's classes lie in one tile, eight or sixteen lanes to the row.
bool gemm_head_fits(int is_bf16, int Md, int Nd, int groups);
// Tile shape of an EPI_WGRAD launch whose reduction runs over Kd samples: as above, or 3 = 64x256 with a k-step of
// 32 and several work-groups per CU while the batch is short and the launch is bound by its epilogue's memory traffic;
// fused != 0: the launch carries the optimizer step in its epilogue (GemmP::upd_x), which keeps medium batches on
// 128x128 tiles, or 5 = 128x256 tiles of eight wavefronts.
int gemm_bf16_wgrad_shape(int Md, int Nd, int Kd, int groups, int fused, const int *rows_host);
// The tile that such a launch takes with GemmP::fine: the shape, or of shape 1 also 4 = 64x128 (1) and 2 = 256x256 (2).
inline int gemm_bf16_wgrad_tile(int shape, int fine) { return shape != 1 || !fine ? shape : fine == 2 ? 2 : 4; }
// Number of upd_sq slots (fused: with the optimizer step in the epilogue) or sq64 slots an EPI_WGRAD launch writes per group.
int gemm_bf16_upd_slots(int Md, int Nd, int Kd, int groups, int fused, int fine, const int *rows_host);
// fp32 SIMT family (gemm_f32.hip); EPI_IPDOT is not offered (U is materialised instead).
hipError_t launch_gemm_f32(const GemmP &p, int epi, hipStream_t s);
// Its EPI_WGRAD takes the optimizer step as well (GemmP::upd_x; the gradient is stored in C all the same, rowsum's entries take
// theirs with it: rowsum and C point into the same vectors as upd_x); one upd_sq slot per block.
int gemm_f32_upd_slots(int Md, int Nd, int tile);
// Tile extent and number of slices (of a multiple of 256 samples each) of an EPI_WGRAD launch over Kd samples; floats of
// kpart scratch, over all groups, that its slices take at most.
struct F32WgradPlan { int tile, ksplit; };
F32WgradPlan gemm_f32_wgrad_plan(int Md, int Nd, int Kd, int groups, size_t kpart_floats);
size_t gemm_f32_kpart_floats(int Md, int Nd, int groups);

// ---- softmax_step.hip --------------------------------------------------------
// One local step of a net without hidden layers in fp32 (weights [K][d] at 0 and biases at offB of every vector of stride sPg): gradient,
// optimizer step, n_i, and the sums n, ||gbar||^2, loss (with do_q also q^2 and q, and q_i) in stats and its mirror, as StatsP has them.
struct SoftmaxStepP {
  const float *X; const int32_t *y, *idx; int N, ldi, d, K, b, groups, has_bias;
  const int *rows;                       // ragged groups (optional): rows[g] <= b
  float *upd_x, *upd_v, *upd_m, *grad; long long sPg, offB;
  float alpha;                           // 1 / b
  int opt; float lr, momentum, beta1, beta2, eps, wd, c1, c2;
  const float *scal;                     // optional (device): {lr, c1, c2}
  int do_q;
  float *n_out, *q_out; long long sNg;   // [g][i]
  float *D; long long sDg; int ldd;      // scratch: signals [g][i][ldd], ldd >= K (do_q over several chunks)
  float *part; double *csums; int *count;   // scratch of several chunks: [g][chunk][part_ld], [g][chunk][4], and 16 ints per group that
                                            //   are zero before the first launch and after each
  int max_chunks;                           // chunks to a group that part and csums hold
  double *stats, *stats_host, ticket;
  int chunks, part_ld;                   // set by the launcher
};
enum { SOFTMAX_STEP_CHUNKS = 32, SOFTMAX_STEP_PARTS = 1 << 19 };     // chunks, and floats of partial gradients, to a group
inline int softmax_step_part_floats(int K, int d) { return (K * d + K + 63) / 64 * 64; }
int softmax_step_chunks(int d, int b);
// The most chunks that a step of up to cap samples takes (a longer batch may take fewer: chunk_of), 0 where none is taken
int softmax_step_max_chunks(int K, int d, int cap, int groups);
bool softmax_step_fits(int K, int d, int b, int groups);
bool softmax_step_taken(int K, int d, int b, int groups, int ip);        // and where it is the faster way (ip: with inner products)
hipError_t launch_softmax_step(SoftmaxStepP p, hipStream_t s);

// ---- gram_ip.hip -----------------------------------------------------------
// q[g][i] = (1 / b_g) sum_l sum_j (D_l D_l^T)[i][j] ((A_l A_l^T)[i][j] + [has_bias]),  i, j < b_g: the inner products
// <g_i, gbar> of a short batch from the Gram matrices of the layer inputs A_l = a^{l-1} and backprop signals
// D_l = delta^l (bf16, rows = samples, K[.] features at leading dimension ld[.], a multiple of 8).  Matrices come
// in pairs: X[2 l] = A_l, X[2 l + 1] = D_l.  part: scratch of gram_ip_scratch_floats(n, groups) floats.  The
// launcher fills in the slicing fields.  b <= GRAM_MAX_B.
enum { GRAM_MAX_B = 256, GRAM_SLICE_ELEMS = 2 * GRAM_MAX_B * GRAM_MAX_B };
struct GramP {
  enum { MAXL = 16 };
  int n;                                   // matrices (two per layer)
  const bf16_t *X[2 * MAXL];
  long long sXg[2 * MAXL];                 // group strides in elements
  int ld[2 * MAXL], K[2 * MAXL];
  int b, groups;
  const int *rows;                         // optional per-group sample counts (device) replacing b
  float *part;                             // [g][matrix][slice][bp][bp] partial Gram matrices
  int bp, S, kslice[2 * MAXL], nsl[2 * MAXL];   // set by the launcher: padded b, slices, features per slice, slices in use
};
long long gram_ip_scratch_floats(int n, int groups);
hipError_t launch_gram_ip(GramP p, int has_bias, float *q, long long sQg, hipStream_t s);

// ---- elementwise.hip -------------------------------------------------------
// T = activation element type: 0 float, 1 bf16
hipError_t launch_convert_f32_to_bf16(const float *src, bf16_t *dst, long long n, hipStream_t s);
// A0[g][i][:] = X[idx[g][i]][:]  and  an0[g][i] = ||row||^2
// Every launcher below takes `rows` (device, may be null): per-group row counts that replace b
// (then b is the largest count and sizes the grid).  `ldi` is the row stride of idx.
hipError_t launch_gather_rows(int is_bf16, const GatherP &p, hipStream_t s);
// softmax cross-entropy head: delta = p - e_y (stored in T, pad columns zeroed),
// dn[g][i] = ||stored delta_i||^2, loss[g][i] = f_i
hipError_t launch_softmax_ce(int is_bf16, const float *Z, long long sZg, int ldz, int K,
                             const int32_t *y, int N, const int32_t *idx, int ldi, int groups, int b,
                             void *D, long long sDg, int ldd, float *dn, float *loss,
                             long long sNg, const int *rows, hipStream_t s);
// out[g][i] = sum_j X[g][i][j]^2
hipError_t launch_row_sqnorm(int is_bf16, const void *X, long long sXg, int ld, int cols,
                             int groups, int b, float *out, long long sOg, const int *rows, hipStream_t s);
// out[g][j] = alpha * sum_i X[g][i][j]   (bias gradients); scratch: groups * ceil(b / COLSUM_ROWS)
// * cols floats of partial sums
enum { COLSUM_ROWS = 128 };
hipError_t launch_col_sum(int is_bf16, const void *X, long long sXg, int ld, int cols, int groups,
                          int b, float alpha, float *out, long long sOg, float *scratch, const int *rows,
                          int accumulate, hipStream_t s);
// First stage of launch_col_sum alone (partials into scratch, nsplit = ceil(b / COLSUM_ROWS) rows per group).
hipError_t launch_col_sum_partials(int is_bf16, const void *X, long long sXg, int ld, int cols, int groups, int b,
                                   float *scratch, const int *rows, hipStream_t s);
// Second stage alone, for several layers in one launch (the bias gradients of a whole step):
// out[g][out_off_l + j] = alpha * sum_r part_l[g][r][j], r < nsplit_l (partials from a GEMM epilogue or from
// launch_col_sum_partials).  With rows: alpha = 1 / rows[g] and, where tile_m_l > 0, only the first
// ceil(rows[g] / tile_m_l) * parts_per_tile_l partials of group g exist.
// A layer with src_l set has no partials: its b signals src_l[g][i][j] (bf16, group stride sXg_l, row stride
// ldx_l) are added up directly.
// With upd_x the biases take their optimizer step in the same launch (accumulate == 0): parameters, state and shadow lie at
// out_off_l + j of every group's vector (group stride sOg), and block (x, layer l) of group g leaves its squared gradient
// entries' sum in sq[g * sSqg + slot0 + l * gridDim.x + x] (col_finish_slots of them).  A block owns cb columns, 64 or 256.
struct ColFinishMany {
  enum { MAXN = 16 };
  int n, cb;                     // layers; columns to a block
  const bf16_t *src[MAXN];
  long long sXg[MAXN];
  int ldx[MAXN], b;
  float *upd_x, *upd_v, *upd_m;
  bf16_t *upd_shadow;
  int upd_opt;
  float upd_lr, upd_momentum, upd_beta1, upd_beta2, upd_eps, upd_wd, upd_c1, upd_c2;
  const float *upd_scal;
  float *sq; long long sSqg; int slot0;
  const float *part[MAXN];       // partials [groups][nsplit][cols]
  int cols[MAXN], nsplit[MAXN], tile_m[MAXN], parts_per_tile[MAXN];
  long long out_off[MAXN];       // offset of the layer's sums inside a group's output vector
  float alpha;
  float *out; long long sOg;
  const int *rows;
  int accumulate;
};
hipError_t launch_col_sum_finish_many(const ColFinishMany &p, int groups, hipStream_t s);
inline int col_finish_slots(int layers, int max_cols, int cb) { return layers * ((max_cols + cb - 1) / cb); }
// q[g][i] += sum_j D[g][i][j] * U[g][i][j]  (fp32 path of the inner products)
hipError_t launch_rowdot_f32(const float *D, long long sDg, int ldd, const float *U,
                             long long sUg, int ldu, int cols, int groups, int b, float *q,
                             long long sQg, int accumulate, const int *rows, hipStream_t s);

struct StatsP {
  int L, has_bias, groups, b, want_ip;
  const float *an[16];      // layer-input squared norms as an_parts[l] partial vectors:
  const float *dn[16];      //   an[l][g * an_sg[l] + part * sPart + i]; likewise the backprop-signal norms
  int an_parts[16], dn_parts[16];
  long long an_sg[16], dn_sg[16];
  long long sPart;          // distance between two partial vectors of the norms
  long long sNg;
  const float *qpart[16];   // per layer: [g][part][i]
  int nparts[16];
  long long sQg[16], sQpart[16];
  const float *loss;        // [g][i] (null: zeros)
  float *n_out, *q_out;     // [g][i] (stride sNg)
  const float *grad;        // [g][Ppad]
  long long Ppad;
  double *partials;         // scratch: [groups][5][PBLK]
  double *stats;            // out: [groups][8] = S1, S2, S3, S4, loss, 0,0,0
  double ticket;            // with stats_host: written to stats_host[g * 8 + 7] after group g's sums have been
                            //   made visible to the host (a host that polls that word needs no stream synchronisation)
  double *stats_host;       // optional mirror in device-visible pinned host memory (same layout): the host then
                            //   needs a stream synchronisation only, no copy
  const float *sq_wave;     // alternative source of S2 (grad must be null): per-wavefront sums of g^2 left by the
  long long n_sq_wave;      //   update kernel, n_sq_wave per group (one per 256 consecutive parameters)
  long long sq_stride;      //   distance between two groups' sums (0: n_sq_wave)
  const double *sq_wave64;  // the same in double (one of the two; n_sq_wave and sq_stride count these)
  const int *rows;          // optional per-group sample counts (device) replacing b
  // which sums this launch produces: S1 and the loss (do_n), S3 and S4 (do_q; needs want_ip),
  // S2 (grad != null); acc_n / acc_q add to the stored sums instead of replacing them
  int do_n, do_q, acc_n, acc_q;
  int nb_done;              // do_n without do_q: the sample blocks (stats_sample_blocks) have run already (StepTail)
};
enum { STATS_PBLK = 256 };
inline int stats_sample_blocks(int b) { return (b + 63) / 64 < STATS_PBLK ? (b + 63) / 64 : (int)STATS_PBLK; }
// What of a step's end needs nothing but the signals and rides in front of a weight-gradient launch (launch_wgrad_many), one
// block of 256 threads each: the bias gradients (cf.n > 0; with the weights' step if the launch carries it) and the per-sample
// part of the statistics (st.nb_done > 0 blocks per group, which leave their sums in st.partials).
struct StepTail { int groups, blocks, cf_x; ColFinishMany cf; StatsP st; };
hipError_t launch_stats(const StatsP &p, hipStream_t s);

struct UpdateP {
  float *x; const float *g; float *v; float *m; bf16_t *shadow;
  long long n;              // total elements (groups * Ppad)
  float *sq_wave;           // optional: sq_wave[i / 256] = sum of g^2 over parameters [256 i', 256 i' + 256)
  int opt; float lr, momentum, beta1, beta2, eps, wd, c1, c2;  // c = 1/(1-beta^t)
  const float *scal;        // optional (device): {lr, c1, c2} read from memory instead of the fields above, so
                            //   that a captured launch can be replayed with new values
};
hipError_t launch_update(const UpdateP &p, hipStream_t s);
hipError_t launch_average_f32(float *x, bf16_t *shadow, float *mean, int groups, long long Ppad, hipStream_t s);
hipError_t launch_average_bf16(bf16_t *x, bf16_t *mean, int groups, long long n, hipStream_t s);
// cross-worker statistics: out[0] = sum_m ||g^m||^2, out[1] = ||mean_m g^m||^2;
// partials: 2 * cross_worker_blocks(Ppad) doubles of scratch
int cross_worker_blocks(long long Ppad);
hipError_t launch_cross_worker(const float *g, int groups, long long Ppad, double *partials,
                               double *out, hipStream_t s);
hipError_t launch_fill_zero(void *p, long long bytes, hipStream_t s);
// Finish of split reductions, the layers of a step in one launch: for layer l and group g
//   C[g][c_off_l + e] = alpha * sum_sp kpart_l[(g * ksplit_l + sp) * mn_l + e]  (+ the old value if accumulate),
// slices added in order; C2 (bf16, may be null) gets the rounded result at the same offsets; rows (may be null):
// alpha = 1 / rows[g].  mn_l and c_off_l are multiples of 4.
struct SplitKFinishMany {
  enum { MAXN = 16 };
  int n;
  const float *kpart[MAXN];
  int ksplit[MAXN];
  long long mn[MAXN], c_off[MAXN];
  float alpha;
  const int *rows;
  float *C; long long sCg;
  bf16_t *C2; long long sC2g;
  int accumulate;
  // Optional (upd_x != null, accumulate == 0): the optimizer step in place of the store to C, as in the
  // weight-gradient epilogue (GemmP::upd_*): parameters, state and shadow at upd_* + g * sCg + c_off_l + e; block j of
  // layer l leaves the sum of its squared gradient entries in upd_sq[g * upd_sSqg + upd_slot0[l] + j]
  // (launch_splitk_finish_slots(mn_l) blocks per layer).
  float *upd_x, *upd_v, *upd_m;
  bf16_t *upd_shadow;
  int upd_opt;
  float upd_lr, upd_momentum, upd_beta1, upd_beta2, upd_eps, upd_wd, upd_c1, upd_c2;
  const float *upd_scal;
  float *upd_sq; long long upd_sSqg; int upd_slot0[MAXN];
};
hipError_t launch_splitk_finish(const SplitKFinishMany &p, int groups, hipStream_t s);
inline int splitk_finish_slots(long long mn) { return (int)((mn / 4 + 255) / 256); }
// Inputs of a replayed step: idx_dst[0..n) = idx_src[0..n), scal[0..3) = {lr, c1, c2}
hipError_t launch_stage_step_inputs(const int32_t *idx_src, int32_t *idx_dst, long long n, float lr, float c1, float c2,
                                    float *scal, hipStream_t s);
// dst[0..n) = v[0..n): the values travel as kernel arguments, so the host array may be reused at once
enum { SET_INTS_MAX = 64 };
hipError_t launch_set_ints(const int *v_host, int n, int *dst, hipStream_t s);
hipError_t launch_copy_probe(const void *src, void *dst, long long bytes, hipStream_t s);

}  // namespace absk
