// Internal launchers of the dllm HIP kernels (not part of the C ABI).
#pragma once
#include "common.h"

namespace dllm {

// ---- k_misc.hip ------------------------------------------------------------
// Bits of the workspace's error word, set by kernels that meet an input they
// cannot represent and reported (then cleared) by the commit kernel.
enum { ERR_TOKEN_RANGE = 1, ERR_V_RANGE = 2 };
// h[b*rows + i, :] = float(E[x[b*L + row0 + i], :]) for b < B, i < rows.  An id
// outside [0, V) gathers a zero row; *err is set to ERR_TOKEN_RANGE if there is
// one and to 0 otherwise.  The nzero ints at zero (the forward's attention
// tickets) are set to 0.  With rope the same launch writes cos/sin [L, hd/2] of
// pos * base^(-2j/hd), evaluated in float64, stored float32.
struct RopeTable {
  float* cosb;
  float* sinb;
  int hd;
  double base;
};
void launch_embed(const int32_t* x, const void* E, int dtype, float* h, int B, int rows, int L, int row0, int d,
                  int V, int* err, hipStream_t s, int* zero = nullptr, int nzero = 0, const RopeTable* rope = nullptr);
// out[b*rows + i, :] = act(RMSNorm(h[b*L + row0 + i, :]) * g) for b < B, i < rows.
void launch_rmsnorm(const float* h, const void* g, void* out, int dtype, int B, int rows, int L, int row0,
                    int d, float eps, hipStream_t s);
// Decoding state initialisation (see dllm_state_init); a non-null err word is
// cleared as well.
void launch_state_init(const int32_t* prompt, int32_t* x, int32_t* commit_step, int8_t* reason, float* sv,
                       int32_t* budget, int32_t* ell, int32_t* done, int B, int P, int G, int mask_id,
                       int* err, hipStream_t s);

// ---- fp32 path (k_f32.hip) -------------------------------------------------
// C = A W^T of an fp32 model (all float32 row-major, float64 accumulation), by epi:
//   F32_QKV    W0/W1/W2 = wq/wk/wv; RoPE on q and k; row m = b Lq + i holds
//              position pos0 + i of sequence b: q [B, Hq, Lq, hd], k [B, Hkv, L,
//              hd] and v^T [B, Hkv, hd, L] (N = the three tensors' rows)
//   F32_SWIGLU W0/W1 = gate/up [N, K]: C[M, N] = silu(gate) * up
//   F32_RESID  C[M, N] += A W0^T          F32_STORE  C[M, N] = A W0^T
// With rows > 0 row m of A is row (m / rows) Ls + r0 + m % rows.  With gain set
// (gemm_f32_fuses_norm; not F32_RESID) the rows of A are RMS-normalised first,
// and the normed rows [M, K] stored at `normed`.
enum { F32_QKV = 0, F32_SWIGLU = 1, F32_RESID = 2, F32_STORE = 3 };
struct GemmF32 {
  int epi;
  int M, N, K;
  const float* A;
  const float* W0; const float* W1; const float* W2;
  float* C;
  int rows, Ls, r0;
  const float* gain; float* normed; float eps;
  float* q; float* k; float* vt; const float* cosb; const float* sinb;
  int Lq, L, pos0, Hq, Hkv, hd;
};
bool gemm_f32_fuses_norm(const GemmF32& g);
void launch_gemm_f32(GemmF32 g, hipStream_t s);
// Non-causal attention, float32, of Lq queries per sequence (q [B, Hq, Lq, hd])
// over L keys (k [B, Hkv, L, hd], v^T [B, Hkv, hd, L]): out[b*Lq + l, h*hd + j].
void launch_attn_f32(const float* q, const float* k, const float* vt, float* out, int B, int Lq, int L, int Hq,
                     int Hkv, int hd, hipStream_t s);
// Per row of logits [R, V]: conf = 1 / sum exp(l - max), argmax (lowest index), mask_id excluded.
void launch_vocab_reduce_f32(const float* logits, int R, int V, int mask_id, float* conf, int32_t* argmax,
                             hipStream_t s);

// ---- bf16 path -------------------------------------------------------------
enum GemmEpi { EPI_QKV_ROPE = 0, EPI_RESID = 1, EPI_SWIGLU = 2 };

struct GemmArgs {
  int epi;
  int M, N, K;              // N counts output columns of the virtual B (gate and up both counted)
  const bf16_t* A;          // [M, K]
  // launches of at most GEMM_ROWS_MAX rows with Wp set: A in operand order
  // (frag_at), and for EPI_SWIGLU a second, operand-order output
  const bf16_t* Af; bf16_t* outf;
  const bf16_t* W0;         // q / gate / plain weight [*, K]
  const bf16_t* W1;         // k / up
  const bf16_t* W2;         // v
  int n0, n1;               // rows of W0 and W1 (QKV: Hq*hd, Hkv*hd)
  // epilogue targets
  float* resid;             // EPI_RESID: [M, N] float32, += result
  bf16_t* out;              // EPI_SWIGLU: [M, N/2]
  bf16_t* q; bf16_t* k; f16_t* vt;   // EPI_QKV_ROPE (v^T holds the bf16 values as IEEE half)
  const float* cosb; const float* sinb;
  // EPI_QKV_ROPE: row m = b Lq + i holds position pos0 + i of sequence b; q is
  // [B, Hq, Lq, hd], k [B, Hkv, L, hd] and v^T [B, Hkv, hd, L] are written at
  // that position (a full forward: Lq = L, pos0 = 0)
  int B, L, Hq, Hkv, Lq, pos0;
  // split-K scratch (float32 partials [split, M, N]) from the workspace
  float* splitk_buf;
  // optional packed copy of Bv (launch_pack_gemm_weights)
  const bf16_t* Wp;
  // EPI_QKV_ROPE: error word; a v value beyond IEEE half's range is stored as
  // +-65504 and sets ERR_V_RANGE
  int* err;
};
// Rows up to which a GEMM with packed weights streams them register-direct; its
// producers then also write A in MFMA operand order: element (m, k) of [M, K] at
// frag_at(MB, m, k), MB = 32-row blocks (rows past M are never stored from).
constexpr int GEMM_ROWS_MAX = 64;
bool gemm_rows_path(int M);
__host__ __device__ inline size_t frag_at(int MB, int m, int k) {
  return ((size_t)(k >> 4) * MB + (m >> 5)) * 512 + ((m & 31) + 32 * ((k >> 3) & 1)) * 8 + (k & 7);
}
int device_cu_count();  // compute units of the current device (256 if it cannot be queried)
// Split-K partial tiles of a residual GEMM whose reduction into the residual
// has been left to the next RMSNorm (split 0: nothing pending).
struct PendingResid {
  const float* part = nullptr;  // [split, M, N] float32
  int split = 0;
};
// With defer non-null, a split-K residual GEMM of more than 128 rows, or of the
// few-row path, leaves its partials pending there instead of launching the
// reduction (defer->split = 0 otherwise).
void launch_gemm_bf16(const GemmArgs& a, hipStream_t s, PendingResid* defer = nullptr);
// Completes a deferred residual update and normalises in one pass, for every
// row m < M (bf16 model, d % 4 == 0, d <= 8192):
//   h[m, :] += sum_z part[z, m, :]   (z in order, as the split-K reduction does)
//   out[m, :] = bf16(RMSNorm(h[m, :]) * g)
// With outf (M <= GEMM_ROWS_MAX) the normed rows also go there in operand order;
// such launches run one 1024-thread workgroup per row, and pend may be empty:
// then d and the alignment of g are free.
void launch_resid_rmsnorm(float* h, const PendingResid& pend, const bf16_t* g, bf16_t* out, bf16_t* outf, int M, int d,
                          float eps, hipStream_t s);
// Packed copy of a GEMM's virtual weight matrix (g's W0/W1/W2, n0, n1, N, K,
// epi) in the LM head's tiled operand order, rows padded to 256.
size_t gemm_packed_bytes(int N, int K);
void launch_pack_gemm_weights(const GemmArgs& g, bf16_t* out, hipStream_t s);
// Bytes of split-K scratch a launch of this shape needs (0 if it does not split).
size_t gemm_bf16_splitk_bytes(int M, int N, int K, int epi);

// Non-causal attention of Lq queries per sequence (q [B, Hq, Lq, 128]) over L
// keys (k [B, Hkv, L, 128], v^T [B, Hkv, 128, L] as IEEE half):
// out[b*Lq + l, h*128 + j] (bf16).  With split_part (attn_split_bytes(B, Hq)
// bytes) and split_ticket (B * Hq ints, zero; left zero) a launch of at most 32
// queries per sequence splits the keys of each head over several workgroups.
// With outf (B * Lq <= GEMM_ROWS_MAX) the rows also go there in operand order.
// Launches of more queries at an L that is no multiple of 8 need pad
// (attn_pad_bytes(B, Hkv, L) bytes of scratch).
size_t attn_split_bytes(int B, int Hq);
size_t attn_pad_bytes(int B, int Hkv, int L);
void launch_attn_bf16(const bf16_t* q, const bf16_t* k, const f16_t* vt, bf16_t* out, bf16_t* outf, int B, int Lq,
                      int L, int Hq, int Hkv, hipStream_t s, float* split_part = nullptr, int* split_ticket = nullptr,
                      f16_t* pad = nullptr);

// The bf16 LM head is read from a tiled copy: vocabulary tiles of HEAD_TILE rows,
// each stored as d/64 consecutive [HEAD_TILE, 64] blocks, rows past V zero;
// inside a block, each 32-row x 16-k MFMA A operand is 1 KiB in lane order.
constexpr int HEAD_TILE = 256;
// Head-row counts up to HEAD_FRAG_ROWS use the streaming LM-head kernel, which
// reads the normed rows from a copy in MFMA B-operand order: for 16-k slice s,
// lane l = row + 32 * ((k / 8) % 2) holds bf16 k = 16 s + 8 (l / 32) .. +7
// (rows >= R unused), 1 KiB per slice.
constexpr int HEAD_FRAG_ROWS = 32;
// Final RMSNorm of the head rows (bf16 model, d % 4 == 0, d <= 8192): out[B*rows,
// d] row-major as launch_rmsnorm, and, when outf is non-null (B * rows <=
// HEAD_FRAG_ROWS), the same values in the operand order above.  Split-K
// partials still pending from the last layer's down projection (pend->split >
// 0, partials [S, B*L, d]) are added to the head rows of h first, as the fused
// residual norm does; the other rows of h are left without them.  A non-null
// ticket (the LM head's) is set to zero for the head kernel that follows.
void launch_rmsnorm_head(float* h, const PendingResid* pend, const bf16_t* g, bf16_t* out, bf16_t* outf, int B,
                         int rows, int L, int row0, int d, float eps, int* ticket, hipStream_t s);
size_t head_bf16_packed_bytes(int V, int d);
void launch_pack_head_bf16(const bf16_t* W, bf16_t* Wt, int V, int d, hipStream_t s);

struct HeadArgs {
  const bf16_t* hb;   // [R, d]
  const bf16_t* hbf;  // R <= HEAD_FRAG_ROWS: the same rows in MFMA operand order (launch_rmsnorm_head)
  const bf16_t* W;    // tiled copy of the [V, d] LM head (launch_pack_head_bf16)
  int R, V, d, mask_id;
  float* conf; int32_t* argmax; float* logits;  // logits optional
  float* part_m; float* part_s; int32_t* part_i;  // [head_bf16_tiles(V), R]: one slot per workgroup
  int* ticket;                                    // zero before the first launch; left zero
};
void launch_head_bf16(const HeadArgs& a, hipStream_t s);
int head_bf16_tiles(int V);
int head_bf16_max_rows();

// ---- controller (k_commit.hip) ---------------------------------------------
struct CommitArgs {
  int32_t* x; int32_t* commit_step; int8_t* reason; float* sv; int32_t* budget; int32_t* ell; int32_t* done;
  const float* conf; const int32_t* argmax; int32_t* all_done;
  int B, L, P, G, bl, g0, t, T, mask_id;
  float thr[4];        // theta_i(t) per position band (float32)
  int edge[3];         // band edges
  int budget_on, grind_on;
  float s_easy, s_hard; int p_easy, p_hard, b_easy, b_mid, b_hard;
  double eta_bar; int patience; float theta_fb;
  int fixed;           // fixed-schedule baseline instead of the confidence-aware rule
  int fixed_k;         // fixed schedule: tokens to commit this step (0 at steps past the block length)
  // error word of the step's workspace (optional): its bits are reported in
  // *all_done above bit 0 and the word is cleared
  int* err;
  // optional word in coherent pinned host memory: receives seq << 8 | the
  // *all_done value with a system-scope release, so the host can wait for the
  // step by polling it instead of a stream synchronisation
  int* host_flag;
  int seq;
};
void launch_commit(const CommitArgs& a, hipStream_t s);

}  // namespace dllm
