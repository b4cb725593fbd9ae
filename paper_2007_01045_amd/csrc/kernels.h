// Internal launcher interface between the host-side stage sequencer and the
// gfx950 kernels.  Plain structs and pointers; every launcher enqueues on the
// given stream and returns the hipError_t of the launch.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dapple {

enum Dtype { DT_F32 = 0, DT_BF16 = 1 };

// ---------------------------------------------------------------- GEMM
// C[m,n] = epilogue( sum_k A(m,k) * B(n,k) ),  m < M, n < N, k < K.
// Operand addressing: a "k-contiguous" operand X(r,k) = X[r*ld + k]; a
// "k-strided" operand X(r,k) = X[k*ld + r].
// K may be cut in segments of kseg_len: segment s reads A + s*segA, B + s*segB
// with k running inside the segment (used to contract over [dq|dk|dv] held in
// three separate buffers).  batch: grid.z instances at strides sA, sB, sC, sBias.
enum GemmEpi {
  EPI_BIAS = 1,   // t = acc + bias[n]
  EPI_ADD = 2,    // t += aux[m,n]
  EPI_MUL = 4,    // t *= aux[m,n]
  EPI_GELU = 8,   // C = gelu(t), C2 = gelu'(t)
  EPI_ACC32 = 16,  // C is fp32 and C += t (weight-gradient accumulation)
  EPI_OUT32 = 32,  // C is fp32 and C = t
  EPI_AUX32 = 64,  // aux is fp32 (residual stream of a bf16 stage)
  EPI_BSUM = 128,  // bsum[n] += sum_k B(n,k): the bias gradient rides along with the weight gradient
  // rowdot[j*M + m] = sum over the 32 columns n of block j of C[m,n] (as stored, rounded to bf16) * aux[m,n];
  // aux is neither added nor multiplied in.  MFMA kernel only, bf16 output, batch 1.  (The attention
  // backward's delta = rowsum(dctx o ctx) per head leaves the product that makes dctx this way.)
  EPI_ROWDOT = 256,
  // with EPI_ACC32, both operands k-strided: every K segment's sum is added to C (and with EPI_BSUM to bsum) on its
  // own, in segment order -- the bits of one accumulating product per segment.
  EPI_SEGACC = 512,
  // with EPI_ADD | EPI_AUX32: what is added is the LayerNorm of aux, (aux[m,n] - mean[m]) rstd[m] gamma[n] + beta[n] --
  // the residual input of a bf16 stage, unrounded, from the sums it was normalised from.  Batch 1.
  EPI_AUXLN = 1024
};

struct GemmArgs {
  const void* A;
  const void* B;
  void* C;
  void* C2;
  const void* bias;
  const void* aux;
  int M, N, K;
  int lda, ldb, ldc, ldaux;
  int a_kstrided, b_kstrided;
  int kseg_len;
  long segA, segB;
  int batch;
  long sA, sB, sC, sBias;
  float* bsum;    // EPI_BSUM: fp32 [N], of instance 0; both operands k-strided
  const float* ln_stats;               // EPI_AUXLN: mean and rstd of every row, gamma and beta in the product's type
  const void *ln_gamma, *ln_beta;
  float* rowdot;  // EPI_ROWDOT: fp32 [ceil(N/32)][M]
  int k_valid;  // k-strided operands: rows k >= k_valid read as zero (K itself is padded)
  int m_valid, n_valid;  // rows of A / B that exist in memory (0 = M / N); rows beyond read as zero
  int epi;
  int tile;  // 0 = automatic choice; 1..10, 12 = a specific tile shape / ring depth (see choose_tile)
  // for the automatic choice: compute units the stream may use (0 = all 256); shared: a data gradient beside the stream of
  // the weight gradients, so a workgroup should leave room on its unit
  int units;
  bool shared;
  // fp32: rows of one micro-batch, where M holds those of several (0 = M).  The fp32 kernels add in one of two orders,
  // and which one follows from a micro-batch's rows alone, so that no bit depends on how many share a launch.
  int rows1;
};

// a launch of the MFMA kernel: its tile, the depth of a k-tile, the k-tiles a workgroup runs, those of zeros that fill
// the ring's last turn among them, its waves and the stages of its ring
struct GemmPlan {
  int rows, cols, depth, k_tiles, waves, stages;
};
// plan: filled in instead of launching anything (MFMA kernel only)
hipError_t launch_gemm(Dtype dt, const GemmArgs& g, hipStream_t st, GemmPlan* plan = nullptr);
// the MFMA kernel's launches per operand layout (a = A k-strided, b = B k-strided: nn, nt, tn, tt); tile: see
// choose_tile; short_k: K segments that are no multiple of 64
struct GemmLaunch {
  int tile;
  bool short_k;
  hipStream_t st;
  GemmPlan* plan;   // filled in instead of launching anything, if given
};
typedef hipError_t (*LaunchMfma)(const GemmArgs& g, const GemmLaunch& l);
hipError_t launch_mfma_nn(const GemmArgs& g, const GemmLaunch& l);
hipError_t launch_mfma_nt(const GemmArgs& g, const GemmLaunch& l);
hipError_t launch_mfma_tn(const GemmArgs& g, const GemmLaunch& l);
hipError_t launch_mfma_tt(const GemmArgs& g, const GemmLaunch& l);
// ... for products of several K segments that follow each other without a gap in the ring (packs, gemm_mfma.h)
hipError_t launch_mfma_nn_pack(const GemmArgs& g, const GemmLaunch& l);
hipError_t launch_mfma_nt_pack(const GemmArgs& g, const GemmLaunch& l);
hipError_t launch_mfma_tn_pack(const GemmArgs& g, const GemmLaunch& l);
hipError_t launch_mfma_tt_pack(const GemmArgs& g, const GemmLaunch& l);
// out[c] += sum over blk (ascending, in the order of launch_partial_reduce) of partial[blk*stride + c], c < cols,
// for up to 12 such jobs in one launch.  nmb > 1: the same for partial + mb_stride, partial + 2 mb_stride, ..., one
// micro-batch's sum after the other
struct ReduceJob {
  const float* partial;
  float* out;
  int nblk, cols;
  long stride;
};
struct ReduceJobs {
  ReduceJob j[12];
  int n;
  int nmb;          // 0 counts as 1
  long mb_stride;
};
// Several weight-gradient products over the same rows in one launch: for each problem C += sum over the micro-batches'
// rows of A^T B, both operands [rows][...] with the rows of the micro-batches one behind the other; K = rows in all,
// kseg = rows of a micro-batch; each one's sum is added to C -- and its column sums of B to bsum, if given -- on its
// own, in order (EPI_SEGACC).
struct WgradProblem {
  const void *A, *B;
  float *C, *bsum;
  int M, N, lda, ldb, ldc;
};
struct WgradGroup {
  static constexpr int MAX = 6;
  WgradProblem p[MAX];
  int n, K, kseg;
  int units;   // as in GemmArgs
  // fp32: 64x64 tiles of the whole list that this one is part of (0 = of this one): the order of the sums follows from
  // them, and must not change where a caller cuts its list in two
  long list_tiles64;
  // sums that go out with the products, as workgroups behind theirs (the LayerNorm parameter gradients of the layer): a
  // launch of their own is 3 to 8 us of waiting for memory with most of the chip idle, here they fill a tail.  nmb >= 1
  ReduceJobs jobs;
  int job_blocks() const { return jobs.n > 0 ? jobs.n * ((jobs.j[0].cols + 63) / 64) : 0; }   // (all of one width)
};
// the same as one accumulating product
GemmArgs wgrad_args(const WgradGroup& w, int i);
bool wgrad_group_takes(Dtype dt, const WgradGroup& w);
hipError_t launch_wgrad_group(Dtype dt, const WgradGroup& w, hipStream_t st);
hipError_t launch_wgrad_group_mfma(const WgradGroup& w, hipStream_t st);
hipError_t launch_wgrad_group_f32(const WgradGroup& w, hipStream_t st);

// fp32 products on the fp32 matrix instructions (gemm_f32.hip): whether they take this problem (else the plain
// kernel does), and the launch
bool gemm_f32_takes(const GemmArgs& g);
hipError_t launch_gemm_f32(const GemmArgs& g, hipStream_t st);
// true when the MFMA kernel takes this problem (else the plain ALU kernel does)
bool gemm_uses_mfma(Dtype dt, const GemmArgs& g);

// ---------------------------------------------------------------- attention
// q,k,v,ctx,dq,dk,dv,dctx: [b*s, H] row-major, head h in columns [h*d, (h+1)*d).
// lse: [b, A, s] fp32, log2-domain logsumexp of the scaled logits.
// delta: [b, A, s] fp32 scratch, rowsum(dctx * ctx) per head.
// delta_blocks (may be NULL): fp32 [H/32][b*s], the same sums per block of 32 columns as EPI_ROWDOT
// of the product that made dctx leaves them; when set, the MFMA backward reads delta from there
// (a head's d/32 blocks added in ascending order) and `delta` is not touched.
// ctx32 (may be NULL): unrounded fp32 copy of ctx, written by the forward and used by the
// backward for delta -- an error in delta shifts a whole row of dS coherently, so a bf16 ctx
// there costs percents of accuracy in dq and dk although ctx itself is accurate to 2^-9.
struct AttnArgs {
  const void *q, *k, *v;
  void* ctx;
  float* ctx32;
  float* lse;
  const void* dctx;
  void *dq, *dk, *dv;
  float* delta;
  const float* delta_blocks;
  int b, s, A, d, H;
  int head0;   // first head of the launch, counted over all sequences (attn_launches)
  int units;   // as in GemmArgs
};
// f(args, heads) for each launch of an attention kernel: its grid's y dimension counts the heads of all sequences and ends
// at 65535, which short sequences in a large batch exceed.  (Runs of heads in the z dimension instead, and an exit for
// those past the last, cost every launch half a microsecond: the kernel's pointers are fetched behind that branch.)
template <typename F>
hipError_t attn_launches(const AttnArgs& a, F&& f) {
  AttnArgs b = a;
  for (b.head0 = 0; b.head0 < a.b * a.A; b.head0 += 65535) {
    const int left = a.b * a.A - b.head0;
    const hipError_t e = f(b, left < 65535 ? left : 65535);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}
hipError_t launch_attn_fwd(Dtype dt, const AttnArgs& a, hipStream_t st);
hipError_t launch_attn_bwd(Dtype dt, const AttnArgs& a, hipStream_t st);
bool attn_uses_mfma(Dtype dt, const AttnArgs& a);
// fp32 stages (attention_f32.hip; ctx32, delta and delta_blocks are not used there)
bool attn_f32_takes(const AttnArgs& a);
hipError_t launch_attn_fwd_f32(const AttnArgs& a, hipStream_t st);
hipError_t launch_attn_bwd_f32(const AttnArgs& a, hipStream_t st);
// true when its backward can take delta_blocks (a head is a whole number of 32-column blocks)
bool attn_takes_delta_blocks(Dtype dt, const AttnArgs& a);

// ---------------------------------------------------------------- row kernels
// y = LN(z) over the last dim (H), stats[2*r] = mean, stats[2*r+1] = rstd.  z_f32: z is fp32
// although the stage is bf16 (the residual stream is kept unrounded); y32 (may be NULL): an
// fp32 copy of y for the next residual add (after the embedding; elsewhere EPI_AUXLN takes it from z).
hipError_t launch_ln_fwd(Dtype dt, const void* z, bool z_f32, const void* gamma, const void* beta, void* y,
                         float* y32, float* stats, int rows, int H, float eps, hipStream_t st);
// dz = LN backward; partial[(blk*3 + {0,1,2})*H + c] = block partial sums of
// dy*xhat (dgamma), dy (dbeta), dz (bias of the linear that produced z).
// Returns the number of partial blocks through *nblk.  nmb micro-batches of `rows` rows each lie one behind the
// other; each has its own *nblk blocks.
int ln_bwd_blocks(int rows);   // *nblk for that many rows
hipError_t launch_ln_bwd(Dtype dt, const void* dy, const void* z, bool z_f32, const float* stats,
                         const void* gamma, void* dz, float* partial, int* nblk, int rows, int H, int nmb,
                         hipStream_t st);
// o_v[c] += sum over blk (ascending) of partial[(blk*nvec + v)*H + c], v < nvec <= 3;
// a NULL o_v is skipped
hipError_t launch_partial_reduce(const float* partial, int nblk, int nvec, int H, float* o0,
                                 float* o1, float* o2, hipStream_t st);
// out[c] += sum_r X[r*ld + c]  (two fixed-order stages through `partial`); nb instances at
// element strides zs_x (X) and zs_out (out); partial needs nb * ceil(rows/64) * cols floats
hipError_t launch_colsum(Dtype dt, const void* X, int rows, int cols, int ld, float* partial,
                         float* out, int nb, long zs_x, long zs_out, hipStream_t st);
// first stage of launch_colsum alone: partial[(z*nblk + blk)*PS + c], blk < *nblk = ceil(rows/64) blocks of 64 rows
hipError_t launch_colsum_partials(Dtype dt, const void* X, int rows, int cols, int ld, float* partial, int nb, long zs_x,
                                  int* nblk, int* PS_out, hipStream_t st);
// (see ReduceJobs)
hipError_t launch_reduce_jobs(const ReduceJobs& J, hipStream_t st);
hipError_t launch_copy(void* dst, const void* src, size_t bytes, hipStream_t st);
hipError_t launch_zero(void* dst, size_t bytes, hipStream_t st);

// ---------------------------------------------------------------- embedding / head
// e[r] = E_w[ids[r]] + E_p[r % s]
hipError_t launch_embed_gather(Dtype dt, const int32_t* ids, const void* Ew, const void* Ep, void* e, int rows, int s,
                               int H, int vocab, hipStream_t st);
// for each of the nmb micro-batches of b sequences, one after the other:
// dEw[id] += sum over rows r with ids[r] == id (ascending r) of de[r];
// dEp[p] += sum over the b sequences of de[bi*s + p]
hipError_t launch_embed_bwd(Dtype dt, const int32_t* ids, const void* de, float* dEw, float* dEp, int b, int s, int H,
                            int vocab, int nmb, hipStream_t st);
// rows_idx / tgt [np], np >= cap: the rows with target >= 0 in ascending order, at most cap of them
// (-1 / 0 in every other entry); info[0] = count, info[1] set to 1 if more than cap rows are predicted
// (nmb micro-batches: targets T apart, rows_idx and tgt np apart; the indices count within a micro-batch)
hipError_t launch_mlm_compact(const int32_t* targets, int T, int nmb, int cap, int np, int vocab, int32_t* rows_idx,
                              int32_t* tgt, int32_t* info, hipStream_t st);
// dst[i] = src[idx[i]] (zero row if idx[i] is outside [0, nsrc)); dst[idx[i]] = src[i]
// (for nmb micro-batches of n gathered and nsrc / ndst full rows)
hipError_t launch_gather_rows(Dtype dt, const void* src, const int32_t* idx, void* dst, int n, int H, int nsrc, int nmb,
                              hipStream_t st);
hipError_t launch_scatter_rows(Dtype dt, const void* src, const int32_t* idx, void* dst, int n, int H, int ndst, int nmb,
                               hipStream_t st);
// logits fp32 [n, VP] (+ bias over v < V) -> dz [n, VP], row_loss [n]
hipError_t launch_mlm_ce(Dtype dt, const float* logits, const void* bias, const int32_t* rows_idx, const int32_t* tgt,
                         int n, int V, int VP, float loss_scale, void* dz, float* row_loss, hipStream_t st);
// loss_out[i] = scale * (sum of row_loss[i*n .. i*n + n - 1]), i < nmb
hipError_t launch_loss_sum(const float* row_loss, int n, int nmb, float scale, float* loss_out, hipStream_t st);
hipError_t launch_mul(Dtype dt, const void* a, const void* b, void* c, long n, hipStream_t st);

// ---------------------------------------------------------------- weight update
// One Adam step over n parameters: g = grad_scale * G; m, v, w32 updated in fp32 (c1, c2: the
// reciprocal bias corrections 1/(1-beta1^step), 1/(1-beta2^step)); w = w32 in the stage's dtype;
// G is zeroed when zero_grads is set.  All fp32 pointers 16-byte aligned.
hipError_t launch_adam(Dtype dt, float* G, float* w32, float* m, float* v, void* w, size_t n, float lr, float beta1,
                       float beta2, float eps, float c1, float c2, float grad_scale, int zero_grads, hipStream_t st);

// ---------------------------------------------------------------- host-side plumbing shared by the C-ABI files
// records the message stage_last_error() returns and hands the code back
int set_error(int code, const char* fmt, ...);
// the compute-unit mask of a stream made by pipeline_partition_stream_create (NULL for any other stream);
// n_words receives its length in 32-bit words
const uint32_t* partition_mask_of(hipStream_t st, int* n_words);

}  // namespace dapple
