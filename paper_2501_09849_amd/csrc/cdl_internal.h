// Internal declarations shared by the translation units of libcdl (not installed).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "cdl.h"
#include "cdl_conv_patch.h"

namespace cdl {

// Most blocks a quantizer kernel that loops over its tensor is launched with.  256 CUs x 8 resident blocks of 256 threads.
constexpr int kMaxQuantBlocks = 2048;
constexpr int kQuantThreads = 256;

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// Record a failed HIP call; returns CDL_ERR_HIP.
int hip_failed(hipError_t e);

// Returns CDL_ERR_HIP (and records the code) when the most recent launch failed.
int check_launch();

// Brackets the kernels launched during its lifetime with two HIP events when profiling is on.
class ProfileScope {
public:
    ProfileScope(const char *name, hipStream_t stream);
    ~ProfileScope();
    ProfileScope(const ProfileScope &) = delete;
    ProfileScope &operator=(const ProfileScope &) = delete;
private:
    int slot_;
    hipStream_t stream_;
};

// Launch KERNEL on STREAM, timed under NAME when profiling is on.
#define CDL_LAUNCH(NAME, STREAM, KERNEL, GRID, BLOCK, LDS, ...)                       \
    do {                                                                              \
        ::cdl::ProfileScope cdl_ps_(NAME, STREAM);                                    \
        hipLaunchKernelGGL(KERNEL, GRID, BLOCK, LDS, STREAM, __VA_ARGS__);            \
    } while (0)

// ---- streaming loads and stores ------------------------------------------------------------
// Large tensors that a pass reads or writes exactly once go through non-temporal accesses: they are not
// kept in the caches, and a pass over data that is not cached anyway runs faster that way (a reduction over
// 805 MB: 183 us with ordinary loads, 122 us with these; quantizer forward and backward on 50 M entries:
// -10 %).  A tensor that fits the 256 MB last-level cache and is visited again soon is better off with
// ordinary accesses (25.6 M entries back to back: +7 % with these), hence the flag.
#if defined(__HIPCC__)
typedef float cdl_v4f __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float4 load_stream4(const float *p, bool stream = true)
{
    if (!stream) return *reinterpret_cast<const float4 *>(p);
    const cdl_v4f v = __builtin_nontemporal_load(reinterpret_cast<const cdl_v4f *>(p));
    return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store_stream4(float *p, float a, float b, float c, float d, bool stream = true)
{
    if (!stream) { *reinterpret_cast<float4 *>(p) = make_float4(a, b, c, d); return; }
    const cdl_v4f v = {a, b, c, d};
    __builtin_nontemporal_store(v, reinterpret_cast<cdl_v4f *>(p));
}
// entries from which a tensor counts as large (32 MiB of fp32)
constexpr long long kStreamFrom = 1ll << 23;
__device__ __forceinline__ void store_stream_u32(void *p, unsigned int v)
{
    __builtin_nontemporal_store(v, reinterpret_cast<unsigned int *>(p));
}
#endif
// Whether a product stores its output [n / cols][cols] past the caches: beyond the 256 MB of the last one (smaller, the pass that follows
// finds it there: a step on 100000 x 64 x 288 229 us against 233), and rows on whole cache lines (60000 x 1500, forward: 127 us
// with ordinary stores, 147 with these).
inline bool stream_output(int64_t n, int64_t cols, const void *out)
{
    return n > (64ll << 20) && cols % 32 == 0 && (reinterpret_cast<uintptr_t>(out) & 127) == 0;
}

// ---- quantizer (cdl_quantizer.hip) -------------------------------------------------------
size_t quantize_workspace_bytes(int64_t n, int32_t n_levels);

int launch_quantize_fwd(const float *theta, int64_t n, const cdl_qparams &p,
                        int8_t *idx, float *soft, float *marg, float *entropy_bits,
                        void *ws, hipStream_t stream);

// scalars: the part of a call's workspace that holds the blocks' sums of the two scalar gradients (quantize_scalar_bytes).
// g and dtheta may be the same tensor.
// Behind them, the table of the soft regime (cdl_soft.hip): made where the call has a workspace and kSoftFrom entries or more.
constexpr int64_t kSoftFrom = 1 << 16;
constexpr int kSoftMaxBins = 512;
constexpr int kSoftCoefs = 10;
constexpr size_t kSoftBinBytes = kSoftCoefs * sizeof(double), kSoftTableBytes = kSoftMaxBins * kSoftBinBytes;
size_t quantize_sum_bytes(int64_t n);        // 16 or 32 bytes per block
size_t quantize_scalar_bytes(int64_t n);     // the sums, then the table
void *quantize_scalar_area(void *ws, int64_t n, int32_t n_levels);
int launch_quantize_bwd(const float *theta, const float *g, int64_t n, const cdl_qparams &p,
                        float *dtheta, float *d_delta, float *d_alpha,
                        void *scalars, hipStream_t stream);

int launch_quantize_draw(const float *theta, const float *u, int64_t n, const cdl_qparams &p, int8_t *idx, hipStream_t stream);

int launch_entropy_bwd(const float *theta, const float *marg, const float *g_in, int64_t n, const cdl_qparams &p,
                       float scale, float *dtheta, float *d_delta, float *d_alpha, void *ws, hipStream_t stream);

// Scratch that lives inside the library (one file-scope device array per GPU) for the entry point that takes
// no workspace: whether it holds what a forward call needs, and its device address on the current device (looked up on first use).
constexpr size_t kStaticScratchBytes = 8u << 20;
bool quantizer_static_fits(int64_t n, int32_t n_levels);
int quantizer_static_scratch(void **ptr);

// 0, or 128 for level sets that reach beyond 127: what the kernels subtract from a level index before storing it.
int index_offset(const cdl_qparams &p);

// Half-width of the band of levels around the nearest one that the kernels visit for a given
// kappa = alpha*delta^2 (levels further out carry less than fp32 resolution of the result).
int quantizer_window(double kappa, int n_levels);

// ---- index GEMMs (cdl_qgemm.hip) ---------------------------------------------------------
size_t qgemm_fwd_workspace_bytes(int32_t M, int32_t N, int32_t K, bool with_offsets);
size_t qgemm_bwd_workspace_bytes(int32_t M, int32_t N, int32_t K);

// a_offset / b_offset: what was subtracted from the level indices of that operand before they were stored (0 or 128)
int launch_qgemm_fwd(const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K,
                     float delta_a, float delta_b, int32_t a_offset, int32_t b_offset, int32_t *acc, float *y,
                     void *ws, hipStream_t stream);

// The same product for problems with few output tiles (cdl_qgemm_small.hip): any K >= 16, no workspace.
bool qgemm_small_serves(int32_t M, int32_t N, int32_t K, int32_t a_offset, int32_t b_offset);
int launch_qgemm_small(const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K, float scale, int32_t a_offset,
                       int32_t b_offset, int32_t *acc, float *y, hipStream_t stream);

// The same, and the forward product of a convolution, with few output columns (cdl_fwd_thin.hip).
struct ConvWindows;
bool qgemm_thin_serves(int32_t M, int32_t N, int32_t K, int32_t a_offset, int32_t b_offset);
int launch_qgemm_thin(const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K, float scale, int32_t a_offset, int32_t *acc, float *y,
                      hipStream_t stream);
bool qconv_thin_serves(int64_t M, int32_t N, int32_t K, int32_t x_offset);
int launch_qconv_thin(const int8_t *x_idx, const int8_t *w_idx, const ConvWindows &w, int32_t N, float scale, int32_t x_offset, int32_t *acc, float *y,
                      hipStream_t stream);

// cw != null: a_idx is not an [M][K] matrix but the activations [B][H][W][C] of a convolutional layer, whose matrix of
// input windows (M = B*P*Q rows, K = R*S*C columns) is the operand; only d_b_hat (the weight gradient) is served.
struct ConvWindows {
    int B, H, W, C, R, S, stride, pad, P, Q;
};

// Both products of a small layer directly (cdl_bwd_direct.hip).  only_b: for a layer whose dL/dQ(a) is formed
// elsewhere (the plan is the same whichever of the others are asked for).  words: the diagnostic words may have to tell limb counts; col_abs_b: what they need of a dL/dQ(a) formed elsewhere, or null.
// asked: products (1 or 2) that are to be exact where sums in double serve; 0: by time alone.
struct BwdPlan;
constexpr size_t kBwdDirectRecordBytes = 8192 * 2 * sizeof(unsigned long long);
bool bwd_direct_serves(int32_t M, int32_t N, int32_t K, bool only_b, double *partial, int max_splits, bool words, int asked);
int launch_bwd_direct(const float *g, const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K, float delta_a, float delta_b,
                      int32_t a_offset, int32_t b_offset, float *d_a_hat, float *d_b_hat, BwdPlan *plan, void *records, double *partial, int max_splits,
                      bool only_b, bool words, const unsigned int *col_abs_b, hipStream_t stream);
// Whether the diagnostic words of a product formed directly tell the limb counts and bounds that limbs would have had (else: no limbs).
bool bwd_direct_diag(int32_t M, int32_t N, int32_t K);

// The same for the gradients of a convolution, by classes of input pixels (cdl_conv_patch.h).
bool conv_dw_direct_serves(int64_t M, int32_t N, int32_t K);
int launch_conv_dw_direct(const float *g, const int8_t *x_idx, const ConvWindows &w, int32_t N, float delta_x, int32_t x_offset, float *d_w_hat,
                          double *partial, int max_splits, hipStream_t stream);
bool conv_dx_direct_serves(int64_t pixels, int32_t N, int32_t C, int32_t R, int32_t S, int32_t stride);
int launch_conv_dx_direct(const float *g, const int8_t *w_idx, const ConvDxGrid *grids, int n_grids, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N,
                          int32_t R, int32_t S, int32_t P, int32_t Q, int32_t stride, float delta_w, float *d_x_hat, hipStream_t stream);

// cdl_limb_rows.hip: dL/dQ(a) over short contractions; frag: b_idx in the fragments of the matrix instructions, tile_bytes for 32 columns
bool limb_rows_serves(int64_t M, int32_t N, int32_t K);
int launch_limb_rows(const float *g, const int8_t *frag, int64_t tile_bytes, int32_t M, int32_t N, int32_t K, const BwdPlan *plan, const double *row_corr, float *out,
                     hipStream_t stream);

// The same for few channels on both sides (cdl_conv_thin.hip); grids: of stride 1, one.
bool conv_dx_thin_serves(const ConvDxGrid *grids, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N, int32_t R, int32_t S, int32_t P, int32_t Q, int32_t stride);
int launch_conv_dx_thin(const float *g, const int8_t *w_idx, const ConvDxGrid &grid, int32_t B, int32_t C, int32_t N, int32_t P, int32_t Q, float delta_w,
                        float *d_x_hat, hipStream_t stream);

// The same on limbs, from patches of g in LDS (cdl_conv_patch.hip).  wr: the weights per class as [ld / 32][C / 32][2][32][16] (halves of 32
// contraction entries, channels, entries), a tap's channels padded with zeros to Np, a multiple of 32; pixel_max: the largest |g| of
// every pixel, as the bits of a float; block_max [n_max <= kPatchMaxima], col_abs [n_abs]: their maxima are the largest |g| of all and the
// largest sum of |w| of a column of any class.
bool conv_dx_patch_serves(const ConvDxGrid *grids, int n_grids, int32_t B, int32_t C, int32_t N, int32_t P, int32_t Q);
struct PatchMaxima { const unsigned int *pixel_max, *block_max, *col_abs; int n_max, n_abs; };
constexpr int kPatchMaxima = 2048;
int launch_conv_dx_patch(const float *g, const int8_t *wr, const PatchMaxima &maxima, int64_t ld, const ConvDxGrid *grids, int n_grids, int32_t B, int32_t H,
                         int32_t W, int32_t C, int32_t N, int32_t Np, int32_t P, int32_t Q, int32_t stride, float delta_w, float *d_x_hat, hipStream_t stream);

// The same on limbs, from digits made beforehand (cdl_conv_dx.hip).  wr: the weights per class as [ld / 64][C][64]; Np: N padded to whole chunks of 16 channels;
// planes: room for the digits of g, kMaxLimbs * M_out * Np bytes; zeros: a page of zeros.
int launch_conv_dx_planes(const float *g, const int8_t *wr, int64_t ld, const ConvDxGrid *grids, int n_grids, int32_t B, int32_t H, int32_t W,
                          int32_t C, int32_t N, int32_t Np, int32_t P, int32_t Q, int32_t stride, const BwdPlan *plan, int8_t *planes,
                          const int8_t *zeros, float *d_x_hat, hipStream_t stream);

int launch_qgemm_bwd(const float *g, const int8_t *a_idx, const int8_t *b_idx,
                     int32_t M, int32_t N, int32_t K, float delta_a, float delta_b, int32_t a_offset, int32_t b_offset,
                     float *d_a_hat, float *d_b_hat, void *ws, hipStream_t stream, const ConvWindows *cw = nullptr);

// The backward products followed by the quantizers' backward passes: dL/dQ(a) goes to d_theta_a (and dL/dQ(b) to d_theta_b
// where d_b_hat is not asked for) and is turned into the gradient in place.
int launch_qgemm_bwd_quantize_bwd(const float *g, const int8_t *a_idx, const int8_t *b_idx, int32_t M, int32_t N, int32_t K,
                                  int32_t a_offset, int32_t b_offset, float delta_b, const float *theta_a, const cdl_qparams &p_a,
                                  float *d_theta_a, float *d_delta_a, float *d_alpha_a, float *d_b_hat, const float *theta_b,
                                  const cdl_qparams *p_b, float *d_theta_b, float *d_delta_b, float *d_alpha_b, void *ws, hipStream_t stream);

// Forward product with the quantizer of the activations in its prologue (K % 128 == 0, indices stored without an offset).
int launch_qgemm_quantize_fwd(const float *x, const cdl_qparams &p, const int8_t *b_idx, int32_t M, int32_t N, int32_t K,
                              float delta_b, float *y, hipStream_t stream);

// Forward product of a convolutional layer over level indices, without an im2col matrix (C % 16 == 0).
size_t qconv_fwd_workspace_bytes(int32_t N, int32_t x_offset);
int qconv_max_chunks();   // most 16-byte chunks of the contraction R*S*C the kernels index
int launch_qconv_fwd(const int8_t *x_idx, const int8_t *w_idx, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N,
                     int32_t R, int32_t S, int32_t stride, int32_t pad, float delta_x, float delta_w, int32_t x_offset,
                     int32_t *acc, float *y, void *ws, hipStream_t stream);

// Activation gradient of a convolutional layer (N % 128 == 0, stride 1 or 2): d_x_hat [B][H][W][C].
size_t qconv_bwd_activations_workspace_bytes(int32_t B, int32_t H, int32_t W, int32_t C, int32_t N, int32_t R, int32_t S, int32_t stride, int32_t pad);
int launch_qconv_bwd_activations(const float *g, const int8_t *w_idx, int32_t B, int32_t H, int32_t W, int32_t C, int32_t N,
                                 int32_t R, int32_t S, int32_t stride, int32_t pad, float delta_w, float *d_x_hat, void *ws,
                                 hipStream_t stream);

// ---- Huffman-coded size (cdl_huffman.hip) --------------------------------------------------
size_t huffman_workspace_bytes(int64_t n);

int launch_huffman_bits(const int8_t *idx, int64_t n, int lo, int n_levels, unsigned long long *counts,
                        unsigned long long *total_bits, float *bits_per_entry, void *ws, hipStream_t stream);

int launch_mfma_probe(int iters, int random_operands, int blocks, int *sink, hipStream_t stream);

}  // namespace cdl
