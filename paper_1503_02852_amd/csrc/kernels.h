// Launch wrappers of the HIP kernels (implemented in the .hip files).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "program.h"

namespace rnng {

// ---------------------------------------------------------------------------------------
// Grouped fp32 MFMA GEMM:  C[M][N] (+)= sum over pairs  A_p(M x K_p) * B_p(K_p x N)
// ---------------------------------------------------------------------------------------
constexpr int GEMM_MAX_PAIRS = 40;         // of a launch, all problems together
constexpr int GEMM_MAX_PROBLEMS = 24;
constexpr int GEMM_WIDE_ROW = 1 << 22;     // rows of so many floats and more: 128 of them are beyond a 32-bit byte offset

struct GemmPair {
    const float* A;   // K-contiguous modes: element (m, k) at A[(m + a_row_off) * lda + k], zero if the
                      // shifted row falls outside [0, a_rows);  M-contiguous mode: element (m, k) at A[k * lda + m]
    const float* B;   // K-contiguous mode: element (k, n) at B[n * ldb + k];  N-contiguous: B[k * ldb + n]
    int K, lda, ldb, a_row_off, a_rows;      // (a row ends after K, M or N floats: lda, ldb are exactly that)
};
struct GemmProblem {
    float* C; int ldc, M, N, first_pair, n_pairs;
    int window_M;           // M if all frames of the window were in this call (M where that is so, and where M is no frames)
    int accumulate;         // 1: C += result instead of C = result
    const float* bias;      // stored is f(result + bias[column]) (NULL: none), f by act (ACT_*); only where the result is stored by
    int act;                // one workgroup (split == 1, no accumulate)
    int min_split;          // tiles of 64 and 128 split the contraction into no fewer parts than this, if several workgroups may add to
                            // a result (their sums round no less than these; tiles of 32 add sums of 64 columns by themselves)
    // by plan_gemm_group:
    int split;              // > 1: that many workgroups share the contraction of a tile and add to C, which must be zero
    int kind;               // 0, 1, 2: tiles of 32, 64, 128; 3: of 32, with rows of GEMM_WIDE_ROW floats or more
    int chunks, narrow;
};
struct GemmGroup {
    GemmProblem p[GEMM_MAX_PROBLEMS];
    GemmPair pair[GEMM_MAX_PAIRS];
    int first_block[GEMM_MAX_PROBLEMS];      // from here on set by launch_gemm_group
    int n_blocks, group_m;
    int n_problems, n_pairs;
};
enum GemmMode {
    GEMM_NT = 0,   // A K-contiguous, B K-contiguous      (forward:  Y_dst = Y_src W^T)
    GEMM_NN = 1,   // A K-contiguous, B N-contiguous      (backward: dY_src = dS_dst W)
    GEMM_TN = 2    // A M-contiguous, B N-contiguous      (gradient: G = dS_dst^T Y_src)
};
// Chooses tiles and splits by estimated time; one_writer: no splits.
void plan_gemm_group(GemmMode mode, GemmGroup& g, bool one_writer);
hipError_t launch_gemm_group(GemmMode mode, const GemmGroup& g, hipStream_t stream);

// ---------------------------------------------------------------------------------------
// Element-wise node programs, step matrix-vector products, softmax, reductions
// ---------------------------------------------------------------------------------------
// Runs a node program for frames [t0, t1) and all streams.  quads: all of its vectors are max_dim wide, a multiple of 4.
hipError_t launch_node_program(const PlanView& pv, int prog_off, int max_dim, bool quads, const float* weights,
                               int T, int N, int t0, int t1, hipStream_t stream);
// Matrix-vector task list for frame t (per-step launch).
hipError_t launch_step_matvec(const PlanView& pv, int mv_off, int n_tasks, int max_out, const float* weights,
                              int T, int N, int t, hipStream_t stream);
// In-place row softmax over `rows` rows of width dim.
hipError_t launch_softmax_rows(float* y, int64_t rows, int dim, hipStream_t stream);
// ds = y - onehot(target) (0 where target < 0); *loss += sum of -ln y[target].
// A target not below dim leaves its frame out and sets *flag to 3.
hipError_t launch_softmax_ce_delta(const float* y, const int32_t* targets, float* ds, double* loss, unsigned* flag,
                                   int64_t rows, int dim, hipStream_t stream);
// Squared-error output layer: ds = (y - d) f'(s) element by element (0 where d is NaN), f' from y
// for act = linear / sigmoid / tanh / rectifier; *loss += 1/2 sum (d - y)^2.
hipError_t launch_squared_error_delta(const float* y, const float* d, float* ds, double* loss, int64_t n, int act,
                                      hipStream_t stream);
// Column-sum tasks (diagonal-weight and bias gradients), atomically added into grads.
// The sums run over frames [t0, T); factors may reach back to frames before t0.
hipError_t launch_colsum(const PlanView& pv, int tasks_off, int n_tasks, int max_dim, const float* weights, float* grads,
                         int T, int N, int t0, bool one_writer, hipStream_t stream);
// A fresh window: zeroes its control words and the history frames in front of it, `frames` frames of
// frame_floats[b] floats of every buffer b (0: the buffer keeps none).
hipError_t launch_zero_history(float* const* buf_ptr, const int64_t* frame_floats, int n_bufs, int frames, unsigned* ctrl, int ctrl_words, hipStream_t stream);
// Moves `stored` frames of up to SHIFT_MAX_TENSORS tensors `frames` frames ahead, in place (the last `frames` keep what they held).
constexpr int SHIFT_MAX_TENSORS = 96;
struct ShiftTensors { void* p[SHIFT_MAX_TENSORS]; int64_t frame_words[SHIFT_MAX_TENSORS]; int count; };      // 32-bit words per frame
hipError_t launch_shift_frames(const ShiftTensors& s, int frames, int stored, hipStream_t stream);
hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t stream);
// rnn_forward_static's array for windows that need twins of ragged tiles beside RNN_STATIC_WORKSPACE_BYTES (32 MiB): at most
// four times as many floats as their tensors (width 1), and the space between tensors.
constexpr int64_t STATIC_LARGE_BYTES = 161 << 20;
hipError_t static_large_workspace(void** p);
hipError_t launch_copy(float* dst, const float* src, int64_t n, hipStream_t stream);
// dst[c][r] = src[r][c] for a row-major rows x cols matrix.
hipError_t launch_transpose(float* dst, const float* src, int rows, int cols, hipStream_t stream);
// n 32-bit words from HOST memory to DEVICE memory, carried as kernel arguments (the words are read
// when the call is made; no staging buffer, no allocation).
hipError_t launch_upload_words(uint32_t* d_dst, const uint32_t* h_src, int64_t n, hipStream_t stream);
// Writes the hardware XCD id of workgroup b (256 threads each) to out[b], b < n_blocks.
hipError_t launch_xcc_probe(unsigned* out, int n_blocks, hipStream_t stream);
// Folds the words that step launches have left the ids of their XCDs in (step_layout.h) into the flag ctrl[0].
hipError_t launch_xcd_words_fold(unsigned* ctrl, hipStream_t stream);
// One-hot sources given as class indices [total_rows]: C[f][j] (+)= W[j][idx[f - shift_rows]] for rows
// [row0, row0 + rows), and the matching weight gradient G[j][idx[f - shift_rows]] += ds[f][j].
hipError_t launch_onehot_gather(float* C, const float* W, const int* idx, int n_dst, int n_src, int64_t row0, int64_t rows,
                                int64_t shift_rows, int64_t total_rows, bool accumulate, hipStream_t stream);
// One-hot weight gradient, G stored whole (no zeros needed in it, nothing is added to what it held).
// Used where the matrix has at least 4,096 columns and at least as many as the window has rows.  Zero fill and scatter
// against this, us of the gradient call, 512 x 4,096: 64 / 256 / 1,024 / 4,096 rows 27 / 39 / 58 / 132 against 28 / 35 / 38 / 46;
// 64 x 38,000: 26 / 34 / 38 / 47 against 28 / 35 / 36 / 39; 2,048 x 38,000: 83 / 108 / 180 / 481 against 84 / 98 / 109 / 159.  The line is
// on the safe side: the scatter's atomics lose beyond it too (512 x 512, 4,096 rows: 135 against 45; 512 x 4,096, 65,536 rows:
// 1,755 against 353).
bool onehot_grad_in_rows(int n_dst, int n_src, int64_t rows);
hipError_t launch_onehot_grad_rows(float* G, const float* ds, const int* idx, int n_dst, int n_src, int64_t shift_rows, int64_t total_rows,
                                   hipStream_t stream);
// The same added to what G holds.  ordered: the rows are added one after another in increasing order (one
// writer per element: the sums are the same bits from run to run), else with float atomics from many workgroups.
hipError_t launch_onehot_scatter(float* G, const float* ds, const int* idx, int n_dst, int n_src, int64_t shift_rows, int64_t total_rows,
                                 bool ordered, hipStream_t stream);

// ---------------------------------------------------------------------------------------
// Persistent recurrent-step kernel (all T steps of one recurrent node and direction)
// ---------------------------------------------------------------------------------------
struct StepLaunchPlan {
    bool ok; int G, NB, xcd_stride; size_t lds_bytes;
    int threads = 256;      // per workgroup (run-time specialised variants only)
};
// Chooses the number of workgroups for a component's step descriptor; ok = false if the
// component does not fit the kernel's limits (then the caller steps with per-frame launches).
int step_nb_for(int N);   // streams per pass of the step kernel for N streams (0: not supported)
bool plan_step_launch(const int32_t* words, int desc_off, int N, int force_G, StepLaunchPlan& out);
hipError_t launch_recurrent_steps(const PlanView& pv, const StepLaunchPlan& lp, int desc_off, const float* weights,
                                  unsigned* ctrl, int T, int N, bool backward, int spin_limit, int t_begin, int t_end,
                                  hipStream_t stream);
// Fills n floats with the "not yet written" bit pattern the step kernel's consumers wait on.
hipError_t launch_fill_sentinel(float* p, int64_t n, hipStream_t stream);
// The same for up to FILL_MAX_RANGES ranges with one launch (a step launch's exchanged tensors).
constexpr int FILL_MAX_RANGES = 16;
// A range of frames of a tile-blocked twin whose width is no multiple of 4 names its tensor's stream
// count and width (twin_n, twin_dim; 0: an ordinary range): the padding becomes zero, so that its
// pollers neither wait for it nor add anything.
struct FillRanges { float* p[FILL_MAX_RANGES]; long long n[FILL_MAX_RANGES]; int twin_n[FILL_MAX_RANGES], twin_dim[FILL_MAX_RANGES], count; };
hipError_t launch_fill_sentinel_ranges(const FillRanges& r, hipStream_t stream);
// The same and launch_zero_history's work (n_bufs 0: the words alone) in one launch; fields, n_fields: more words to clear.
hipError_t launch_fill_sentinel_and_clear(const FillRanges& r, float* const* buf_ptr, const int64_t* frame_floats, int n_bufs, int frames, unsigned* words, int n_words,
                                          unsigned* fields, int n_fields, hipStream_t stream);

}  // namespace rnng
