// Element-wise kernels: node programs over many frames (additive / multiplicative layers,
// activation functions and their derivatives: paper Section 2.1 and the delta / epsilon
// equations of Section 2.2), row softmax with the cross-entropy output delta (Section 2.2),
// column sums for diagonal-weight and bias gradients, and fills.
#include "interp.h"
#include "kernels.h"

namespace rnng {
namespace {

// One thread per (frame, stream, unit); the accumulator entries of the program (if any) are
// read from their one-frame buffers.
__global__ __launch_bounds__(256)
void node_program_kernel(PlanView pv, int prog_off, int max_dim,
                                                           const float* __restrict__ weights,
                                                           int T, int N, int t0, long long total) {
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const long long row = idx / max_dim;
    const UnitMap um{0, 1, (int)(idx - row * max_dim)};
    const int t = t0 + (int)(row / N), n = (int)(row % N);
    const ProgramView pg(pv.words + prog_off);
    float s[MAX_SLOTS];
    auto acc = [&](int buf, int dim, int nn, int i, int) { return pv.buf_ptr[buf][(size_t)nn * dim + i]; };
    load_gathers(s, pg, pv, um, T, N, t, n, acc, true);
    load_invariants(s, pg, weights, um);
    run_ops(s, pg);
    run_stores(s, pg, pv, um, N, t, n, [](float* p, float v) { *p = v; });
}

// The same for short programs all of whose vectors have one width, a multiple of 4: four units per thread, so that a program word is
// read and decoded once for four of them (it was bound by that: products and sums of 8,192 x 1,024 elements 42.5 -> 22.6 us).
typedef float program_float4 __attribute__((ext_vector_type(4), aligned(4)));
__global__ __launch_bounds__(256) void node_program4_kernel(PlanView pv, int prog_off, int dim, const float* __restrict__ weights,
                                                            int T, int N, int t0, long long total) {
    const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
    if (idx >= total) return;
    const int quads = dim / 4;
    const long long row = idx / quads;
    const int i = 4 * (int)(idx - row * quads), t = t0 + (int)(row / N), n = (int)(row % N);
    const ProgramView pg(pv.words + prog_off);
    float s0[QUAD_SLOTS], s1[QUAD_SLOTS], s2[QUAD_SLOTS], s3[QUAD_SLOTS];
    auto put = [&](int k, program_float4 v) { s0[k] = v.x; s1[k] = v.y; s2[k] = v.z; s3[k] = v.w; };
    for (int g = 0; g < pg.n_gather; ++g) {
        cwords_t e = pg.ga + g * GA_WORDS;
        const int frame = t + uni(e[GA_FRAME_OFF]);
        program_float4 v = {0.0f, 0.0f, 0.0f, 0.0f};
        if (frame >= 0 && frame < T) v = *reinterpret_cast<const program_float4*>(((cbufs_t)pv.buf_ptr)[uni(e[GA_BUF])] + ((size_t)frame * N + n) * dim + i);
        put(g, v);
    }
    for (int v = 0; v < pg.n_inv; ++v) put(pg.n_gather + v, *reinterpret_cast<const program_float4*>(weights + uni(pg.iv[v * IV_WORDS + IV_W_OFF]) + i));
    for (int p = 0; p < pg.n_ops; ++p) {
        const int packed = uni(pg.mo[p * MO_WORDS + MO_PACKED]), c = uni(pg.mo[p * MO_WORDS + MO_C]);
        const int opc = packed & 0xFF, d = (packed >> 8) & 0xFF, a = (packed >> 16) & 0xFF, b = (packed >> 24) & 0xFF;
        auto all = [&](auto f) {
            s0[d] = f(s0[a], s0[b], s0[c]); s1[d] = f(s1[a], s1[b], s1[c]);
            s2[d] = f(s2[a], s2[b], s2[c]); s3[d] = f(s3[a], s3[b], s3[c]);
        };
        switch (opc) {
            case MOP_MOV: all([](float x, float, float) { return x; }); break;
            case MOP_ADD: all([](float x, float y, float) { return x + y; }); break;
            case MOP_MUL: all([](float x, float y, float) { return x * y; }); break;
            case MOP_FMA: all([](float x, float y, float z) { return fmaf(x, y, z); }); break;
            case MOP_SIG: all([](float x, float, float) { return sigmoid_f(x); }); break;
            case MOP_TANH: all([](float x, float, float) { return tanh_f(x); }); break;
            case MOP_DSIG: all([](float x, float y, float) { return x * y * (1.0f - y); }); break;
            case MOP_DTANH: all([](float x, float y, float) { return x * (1.0f - y * y); }); break;
            case MOP_RELU: all([](float x, float, float) { return fmaxf(x, 0.0f); }); break;
            case MOP_DRELU: all([](float x, float y, float) { return y > 0.0f ? x : 0.0f; }); break;
            case MOP_MAX: all([](float x, float y, float) { return fmaxf(x, y); }); break;
            case MOP_GE: all([](float x, float y, float) { return x >= y ? 1.0f : 0.0f; }); break;
            case MOP_GT: all([](float x, float y, float) { return x > y ? 1.0f : 0.0f; }); break;
            default: all([](float, float, float) { return 0.0f; }); break;
        }
    }
    for (int q = 0; q < pg.n_stores; ++q) {
        cwords_t e = pg.st + q * ST_WORDS;
        const int k = uni(e[ST_SLOT]);
        *reinterpret_cast<program_float4*>(((cbufs_t)pv.buf_ptr)[uni(e[ST_BUF])] + ((size_t)t * N + n) * dim + i) = program_float4{s0[k], s1[k], s2[k], s3[k]};
    }
}

// One wavefront per output unit u of a task; all streams n in a loop.
__global__ __launch_bounds__(256) void step_matvec_kernel(PlanView pv, int mv_off, const float* __restrict__ weights,
                                                          int T, int N, int t) {
    const int32_t* w = pv.words + mv_off + 1;
    for (int task = 0; task < (int)blockIdx.y; ++task) w += MV_HEADER_WORDS + w[MV_NEDGES] * MVE_WORDS;
    const int n_out = w[MV_NOUT], n_edges = w[MV_NEDGES];
    const int lane = threadIdx.x & 63;
    const int u = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (u >= n_out) return;
    float* acc = pv.buf_ptr[w[MV_ACC_BUF]];
    for (int n = 0; n < N; ++n) {
        float s = 0.0f;
        for (int e = 0; e < n_edges; ++e) {
            const int32_t* ed = w + MV_HEADER_WORDS + e * MVE_WORDS;
            const int frame = t + ed[MVE_FRAME_OFF];
            if (frame < 0 || frame >= T) continue;
            const int K = ed[MVE_KLEN];
            const float* W = weights + ed[MVE_W_OFF];
            const float* x = pv.buf_ptr[ed[MVE_SRC_BUF]] + ((size_t)frame * N + n) * K;
            if (ed[MVE_TRANSPOSED]) { for (int k = lane; k < K; k += 64) s += W[(size_t)k * n_out + u] * x[k]; }
            else { for (int k = lane; k < K; k += 64) s += W[(size_t)u * K + k] * x[k]; }
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
        if (lane == 0) acc[(size_t)n * n_out + u] = s;
    }
}

__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, 64));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// One wavefront per row, in place; the row (at most 64 R columns) stays in registers between its one read and
// its one write.
template <int R>
__global__ __launch_bounds__(256) void softmax_rows_kernel(float* __restrict__ y, long long rows, int dim) {
    const long long row = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rows) return;
    const int lane = threadIdx.x & 63;
    float* p = y + row * dim;
    float v[R];
    float m = -INFINITY;
#pragma unroll
    for (int j = 0; j < R; ++j) v[j] = lane + 64 * j < dim ? p[lane + 64 * j] : -INFINITY;
#pragma unroll
    for (int j = 0; j < R; ++j) m = fmaxf(m, v[j]);
    m = wave_max(m);
    float s = 0.0f;
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (lane + 64 * j < dim) s += v[j] = __expf(v[j] - m);
    s = wave_sum(s);
    const float inv = 1.0f / s;
#pragma unroll
    for (int j = 0; j < R; ++j)
        if (lane + 64 * j < dim) p[lane + 64 * j] = v[j] * inv;
}

// Wide rows: bound by memory.  One workgroup per row; its first 4096 CHUNKS columns stay in registers, sixteen bytes
// per load (which need 4-byte alignment only, so any width will do), columns beyond them are read three times.
// One wavefront per row leaves 2048 rows two wavefronts per SIMD with one 4-byte load in flight each, three times over:
// 2048 rows of 20,000, softmax and output delta (below) together 0.30 ms less per window than that (3.03 -> 2.72 ms for a
// 38,000-512-20,000 LSTM on class indices).  Up to 2048 columns a row fits the registers of one wavefront, which
// then has no barriers: one layer's forward pass, a workgroup / a wavefront per row, 64 rows of 2048 27 / 28 us, 2,048 rows
// of 1,100 / 2,048 55 / 46 and 71 / 64, 8,192 rows 124 / 93 and 169 / 145 (three reads by a wavefront: 104 and 168).
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));
constexpr int SMX_THREADS = 1024, SMX_CHUNK = 4 * SMX_THREADS;
template <int CHUNKS>
__global__ __launch_bounds__(SMX_THREADS) void softmax_wide_rows_kernel(float* __restrict__ y, long long rows, int dim) {
    constexpr int WIDE = SMX_CHUNK * CHUNKS;
    __shared__ float part[2][SMX_THREADS / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    for (long long row = blockIdx.x; row < rows; row += gridDim.x) {
        float* p = y + row * dim;
        float v[CHUNKS][4];
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const int i = c * SMX_CHUNK + 4 * tid;
            if (i + 3 < dim) {
                const floatx4u x = *reinterpret_cast<const floatx4u*>(p + i);
#pragma unroll
                for (int e = 0; e < 4; ++e) v[c][e] = x[e];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[c][e] = i + e < dim ? p[i + e] : -INFINITY;
            }
        }
        float m = -INFINITY;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) m = fmaxf(m, v[c][e]);
        for (int i = WIDE + tid; i < dim; i += SMX_THREADS) m = fmaxf(m, p[i]);
        m = wave_max(m);
        if (lane == 0) part[0][wave] = m;
        __syncthreads();
        m = wave_max(part[0][lane & (SMX_THREADS / 64 - 1)]);
        float s = 0.0f;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c * SMX_CHUNK + 4 * tid + e < dim) s += v[c][e] = __expf(v[c][e] - m);
        for (int i = WIDE + tid; i < dim; i += SMX_THREADS) s += __expf(p[i] - m);
        s = wave_sum(s);
        if (lane == 0) part[1][wave] = s;
        __syncthreads();
        s = wave_sum(lane < SMX_THREADS / 64 ? part[1][lane] : 0.0f);
        const float inv = 1.0f / s;
#pragma unroll
        for (int c = 0; c < CHUNKS; ++c) {
            const int i = c * SMX_CHUNK + 4 * tid;
            if (i + 3 < dim) {
                floatx4u x;
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = v[c][e] * inv;
                *reinterpret_cast<floatx4u*>(p + i) = x;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < dim) p[i + e] = v[c][e] * inv;
            }
        }
        for (int i = WIDE + tid; i < dim; i += SMX_THREADS) p[i] = __expf(p[i] - m) * inv;
    }
}

// One wavefront per row.  The workgroups' losses meet in one address, about 13 ns each: a workgroup takes several rows where
// there are few values, so that the additions don't outlast the rows (the launch's rule below).
__global__ __launch_bounds__(256) void softmax_ce_delta_kernel(const float* __restrict__ y, const int32_t* __restrict__ targets,
                                                               float* __restrict__ ds, double* loss, unsigned* flag, long long rows, int dim) {
    __shared__ double wl[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double l = 0.0;
    for (long long row = (long long)blockIdx.x * 4 + wave; row < rows; row += 4LL * gridDim.x) {
        int tg = targets[row];
        if (tg >= dim) { if (lane == 0) atomicMax(flag, 3u); tg = -1; }      // not a class of this layer: the frame is left out
        const float* p = y + row * dim;
        float* d = ds + row * dim;
        for (int i = lane; i < dim; i += 64) d[i] = tg >= 0 ? p[i] - (i == tg ? 1.0f : 0.0f) : 0.0f;
        if (tg >= 0 && lane == 0) l += (double)-__logf(p[tg]);
    }
    if (lane == 0) wl[wave] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double s = wl[0] + wl[1] + wl[2] + wl[3];
        if (s != 0.0) atomicAdd(loss, s);
    }
}

// The same for wide rows: one workgroup per segment of a row, sixteen values per thread, all loads in flight.
constexpr int CE_SEGMENT = 4096;
__global__ __launch_bounds__(256) void softmax_ce_delta_wide_kernel(const float* __restrict__ y, const int32_t* __restrict__ targets,
                                                                    float* __restrict__ ds, double* loss, unsigned* flag,
                                                                    long long rows, int dim) {
    const int first = (int)blockIdx.y * CE_SEGMENT + 4 * (int)threadIdx.x;
    for (long long row = blockIdx.x; row < rows; row += gridDim.x) {
        int tg = targets[row];
        if (tg >= dim) { if (threadIdx.x == 0) atomicMax(flag, 3u); tg = -1; }
        const float* p = y + row * dim;
        float* d = ds + row * dim;
        floatx4u x[CE_SEGMENT / 1024];
#pragma unroll
        for (int c = 0; c < CE_SEGMENT / 1024; ++c) {
            const int i = first + 1024 * c;
            if (i + 3 < dim) {
                x[c] = *reinterpret_cast<const floatx4u*>(p + i);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) x[c][e] = i + e < dim ? p[i + e] : 0.0f;
            }
        }
#pragma unroll
        for (int c = 0; c < CE_SEGMENT / 1024; ++c) {
            const int i = first + 1024 * c;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (tg >= 0 && i + e == tg) {
                    const double l = (double)-__logf(x[c][e]);
                    if (l != 0.0) atomicAdd(loss, l);
                }
                x[c][e] = tg >= 0 ? x[c][e] - (i + e == tg ? 1.0f : 0.0f) : 0.0f;
            }
            if (i + 3 < dim) {
                *reinterpret_cast<floatx4u*>(d + i) = x[c];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (i + e < dim) d[i + e] = x[c][e];
            }
        }
    }
}

// Squared error E = 1/2 sum_j (d_j - y_j)^2 on an output layer y = f(s) (Section 2.2: the output delta
// follows the error criterion and the layer's activation): dE/ds = (y - d) f'(s).
__global__ __launch_bounds__(256) void squared_error_delta_kernel(const float* __restrict__ y, const float* __restrict__ d,
                                                                  float* __restrict__ ds, double* loss, long long n, int act) {
    __shared__ double wl[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double l = 0.0;
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += 256LL * gridDim.x) {
        const float yi = y[i], di = d[i];
        const float err = di != di ? 0.0f : yi - di;      // a NaN target element carries no error
        const float fp = act == 1 ? yi * (1.0f - yi) : act == 2 ? 1.0f - yi * yi : act == 4 ? (yi > 0.0f ? 1.0f : 0.0f) : 1.0f;
        ds[i] = err * fp;
        l += (double)(0.5f * err * err);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) l += __shfl_xor(l, off, 64);
    if (lane == 0) wl[wave] = l;
    __syncthreads();
    if (threadIdx.x == 0) {
        const double s = wl[0] + wl[1] + wl[2] + wl[3];
        if (s != 0.0) atomicAdd(loss, s);
    }
}

// The sum over rows of the product of NF factors without comparisons, for one unit.  Bound by memory: the factors' addresses are
// worked out once and eight rows' loads are in flight.  One row at a time, each behind the reads of its descriptor, before: three layers of
// 1,024 units at 64 x 128 frames 407 -> 150 us, 2 x 512 at 32 x 256 119 -> 44, 2 x 256 at 1,024 frames 19 -> 7.
template <int NF>
__device__ __forceinline__ float colsum_products(const PlanView& pv, const int32_t* w, const float* __restrict__ weights, int i, int dim, long long N,
                                                 long long rows, long long r, long long step) {
    const float* q[NF];
    long long shift[NF];
    float wf[NF];
    bool weighted[NF];
#pragma unroll
    for (int j = 0; j < NF; ++j) {
        const int32_t* f = w + CS_HEADER_WORDS + j * CF_WORDS;
        shift[j] = f[CF_FRAME_OFF] * N;
        q[j] = pv.buf_ptr[f[CF_BUF]] + i;
        weighted[j] = f[CF_W_OFF] >= 0;
        wf[j] = weighted[j] ? weights[f[CF_W_OFF] + i] : 1.0f;
    }
    constexpr int U = 8;
    float s = 0.0f;
    for (; r < rows; r += U * step) {
        float v[NF][U];
        bool ok[NF][U];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                const long long at = r + u * step + shift[j];
                ok[j][u] = at >= 0 && at < rows && r + u * step < rows;
                v[j][u] = q[j][(ok[j][u] ? at : 0) * dim];
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float prod = 1.0f;
#pragma unroll
            for (int j = 0; j < NF; ++j) {
                const float x = ok[j][u] ? v[j][u] : 0.0f;
                prod *= weighted[j] ? x * wf[j] : x;
            }
            s += r + u * step < rows ? prod : 0.0f;
        }
    }
    return s;
}

// grid: (ceil(dim / 64), n_tasks, row splits); block (64, 4).
__global__ __launch_bounds__(256) void colsum_kernel(PlanView pv, int tasks_off, const float* __restrict__ weights,
                                                     float* __restrict__ grads, int T, int N, int t0) {
    __shared__ float part[4][64];
    const int32_t* w = pv.words + tasks_off;
    for (int task = 0; task < (int)blockIdx.y; ++task) w += CS_HEADER_WORDS + w[CS_NFACTORS] * CF_WORDS;
    const int dim = w[CS_DIM], nf = w[CS_NFACTORS];
    if ((int)blockIdx.x * 64 >= dim) return;
    const int i = blockIdx.x * 64 + threadIdx.x;
    const long long rows = (long long)T * N, first = (long long)t0 * N + (long long)blockIdx.z * 4 + threadIdx.y, step = 4LL * gridDim.z;
    bool plain = nf <= 2;
    for (int j = 0; j < nf && plain; ++j) plain = w[CS_HEADER_WORDS + j * CF_WORDS + CF_CMP] == 0;
    float s = 0.0f;
    if (i < dim && plain && nf == 1) s = colsum_products<1>(pv, w, weights, i, dim, N, rows, first, step);
    else if (i < dim && plain && nf == 2) s = colsum_products<2>(pv, w, weights, i, dim, N, rows, first, step);
    else if (i < dim) {
        for (long long r = first; r < rows; r += step) {
            const int t = (int)(r / N), n = (int)(r % N);
            float prod = 1.0f;
            auto value = [&](int j) {
                const int32_t* f = w + CS_HEADER_WORDS + j * CF_WORDS;
                const int frame = t + f[CF_FRAME_OFF];
                float v = 0.0f;
                if (frame >= 0 && frame < T) v = pv.buf_ptr[f[CF_BUF]][((size_t)frame * N + n) * dim + i];
                if (f[CF_W_OFF] >= 0) v *= weights[f[CF_W_OFF] + i];
                return v;
            };
            for (int j = 0; j < nf; ++j) {
                const int cmp = w[CS_HEADER_WORDS + j * CF_WORDS + CF_CMP];
                if (cmp != 0 && j + 1 < nf) {      // [this >= next] or [this > next]: a maximum node's routing
                    const float a = value(j), b = value(j + 1);
                    prod *= (cmp == 1 ? a >= b : a > b) ? 1.0f : 0.0f;
                    ++j;
                } else {
                    prod *= value(j);
                }
            }
            s += prod;
        }
    }
    part[threadIdx.y][threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.y == 0 && i < dim) {
        const float tot = part[0][threadIdx.x] + part[1][threadIdx.x] + part[2][threadIdx.x] + part[3][threadIdx.x];
        unsafeAtomicAdd(&grads[w[CS_OUT_OFF] + i], tot);
    }
}

__global__ __launch_bounds__(256) void fill_kernel(float* __restrict__ p, long long n, float v) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += 256LL * gridDim.x) p[i] = v;
}

}  // namespace

hipError_t launch_node_program(const PlanView& pv, int prog_off, int max_dim, bool quads, const float* weights,
                               int T, int N, int t0, int t1, hipStream_t stream) {
    const long long total = (long long)(t1 - t0) * N * max_dim;
    if (total <= 0) return hipSuccess;
    if (quads) {
        hipLaunchKernelGGL(node_program4_kernel, dim3((unsigned)((total / 4 + 255) / 256)), dim3(256), 0, stream, pv, prog_off, max_dim, weights, T, N, t0, total / 4);
        return hipGetLastError();
    }
    const unsigned blocks = (unsigned)((total + 255) / 256);
    hipLaunchKernelGGL(node_program_kernel, dim3(blocks), dim3(256), 0, stream, pv, prog_off, max_dim, weights, T, N, t0, total);
    return hipGetLastError();
}

hipError_t launch_step_matvec(const PlanView& pv, int mv_off, int n_tasks, int max_out, const float* weights,
                              int T, int N, int t, hipStream_t stream) {
    if (n_tasks <= 0 || max_out <= 0) return hipSuccess;
    hipLaunchKernelGGL(step_matvec_kernel, dim3((max_out + 3) / 4, n_tasks), dim3(256), 0, stream, pv, mv_off, weights, T, N, t);
    return hipGetLastError();
}

hipError_t launch_softmax_rows(float* y, int64_t rows, int dim, hipStream_t stream) {
    if (rows <= 0) return hipSuccess;
    const dim3 grid((unsigned)((rows + 3) / 4)), block(256);
    if (dim <= 64) hipLaunchKernelGGL((softmax_rows_kernel<1>), grid, block, 0, stream, y, (long long)rows, dim);
    else if (dim <= 256) hipLaunchKernelGGL((softmax_rows_kernel<4>), grid, block, 0, stream, y, (long long)rows, dim);
    else if (dim <= 1024) hipLaunchKernelGGL((softmax_rows_kernel<16>), grid, block, 0, stream, y, (long long)rows, dim);
    else if (dim <= 2048) hipLaunchKernelGGL((softmax_rows_kernel<32>), grid, block, 0, stream, y, (long long)rows, dim);
    else {
        // a workgroup's registers hold the row, but no instance more of them than it needs: forward pass of one
        // layer with one / two / five / ten chunks, 2,048 rows of 4,100 columns 92 / 92 / 107 / 128 us, 8,192 155 / 149 /
        // 163 / 177, 20,000 346 / 333 / 314 / 325, 40,960 782 / 768 / 770 / 666, 65,536 1,292 / 1,275 / 1,366 / 1,240
        const dim3 wide((unsigned)std::min<int64_t>(rows, 1 << 20)), threads(SMX_THREADS);
        if (dim <= SMX_CHUNK) hipLaunchKernelGGL((softmax_wide_rows_kernel<1>), wide, threads, 0, stream, y, (long long)rows, dim);
        else if (dim <= 2 * SMX_CHUNK) hipLaunchKernelGGL((softmax_wide_rows_kernel<2>), wide, threads, 0, stream, y, (long long)rows, dim);
        else if (dim <= 5 * SMX_CHUNK) hipLaunchKernelGGL((softmax_wide_rows_kernel<5>), wide, threads, 0, stream, y, (long long)rows, dim);
        else hipLaunchKernelGGL((softmax_wide_rows_kernel<10>), wide, threads, 0, stream, y, (long long)rows, dim);
    }
    return hipGetLastError();
}

hipError_t launch_softmax_ce_delta(const float* y, const int32_t* targets, float* ds, double* loss, unsigned* flag,
                                   int64_t rows, int dim, hipStream_t stream) {
    if (rows <= 0) return hipSuccess;
    // By segments where a wavefront per row is too few of them or walks its row for too long; else a workgroup
    // has too little to do for its start.  Wavefronts against segments, µs of the backward pass of one layer:
    // 256 rows of 1,100 / 4,096 columns 12.6 / 18.6 against 11.8 / 12.2; 512 rows of 1,100 / 2,048 / 4,096 12.3 /
    // 14.8 / 21.2 against 15.0 / 14.4 / 15.2; 1,024 rows of 2,048 / 4,096 16.6 / 23.9 against 21.7 / 22.3; 2,048 rows
    // of 1,100 / 4,096 / 5,000 / 20,000 17.6 / 32.7 / 39.3 / 163 against 34.1 / 37.9 / 38.0 / 69; 8,192 rows of 1,100 /
    // 6,000 / 8,192 42 / 113 / 145 against 109 / 117 / 123.
    if (dim > 1024 && dim > std::min<int64_t>(4 * rows, 4096 + std::min<int64_t>(rows, 8192) / 4)) {
        hipLaunchKernelGGL(softmax_ce_delta_wide_kernel, dim3((unsigned)std::min<int64_t>(rows, 1 << 20), (dim + CE_SEGMENT - 1) / CE_SEGMENT),
                           dim3(256), 0, stream, y, targets, ds, loss, flag, (long long)rows, dim);
        return hipGetLastError();
    }
    // Additions to the loss against rows that a wavefront walks one after the other, each of which costs about as much as 128
    // values beside its own.  512 / 2,048 workgroups, us of the backward pass of one layer: 8,192 rows of 30 / 256 / 600 / 1,000
    // columns 17 / 34, 19 / 35, 28 / 39, 37 / 42; 32,768 of 30 / 128 / 256 / 400 / 1,000 24 / 36, 28 / 38, 43 / 43, 58 / 49, 108 / 68;
    // 65,536 of 128 51 / 45; 131,072 of 30 67 / 46; 400,000 of 30 183 / 78.  Beyond 1,024 columns there is no such side (2,048 rows of 1,500 /
    // 2,000 20.5 / 21.4 and 24.4 / 23.2, 4,096 32.9 / 31.1 and 37.2 / 32.3).
    const int64_t blocks = std::min<int64_t>((rows + 3) / 4, dim <= 1024 && rows * (dim + 128) <= 12 << 20 ? 512 : 2048);
    hipLaunchKernelGGL(softmax_ce_delta_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, y, targets, ds, loss, flag, (long long)rows, dim);
    return hipGetLastError();
}

hipError_t launch_squared_error_delta(const float* y, const float* d, float* ds, double* loss, int64_t n, int act,
                                      hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    // (their losses meet in one address, 13 ns each.  512 / 2,048 workgroups, us of the backward pass of one layer: 2^18 values 15 / 21, 2^20 17 / 34,
    // 2^22 26 / 39, 2^23 37 / 45, 2^24 60 / 56, 2^26 322 / 158)
    if (blocks > 512) blocks = n > (1 << 23) ? std::min<long long>(blocks, 2048) : 512;
    hipLaunchKernelGGL(squared_error_delta_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, y, d, ds, loss, (long long)n, act);
    return hipGetLastError();
}

hipError_t launch_colsum(const PlanView& pv, int tasks_off, int n_tasks, int max_dim, const float* weights, float* grads,
                         int T, int N, int t0, bool one_writer, hipStream_t stream) {
    if (n_tasks <= 0 || max_dim <= 0) return hipSuccess;
    const long long rows = (long long)(T - t0) * N;
    int splits = (int)((rows + 63) / 64);
    if (splits > 128) splits = 128;
    if (splits < 1 || one_writer) splits = 1;      // one workgroup per (task, 64 units): a fixed order of additions
    hipLaunchKernelGGL(colsum_kernel, dim3((max_dim + 63) / 64, n_tasks, splits), dim3(64, 4), 0, stream, pv, tasks_off,
                       weights, grads, T, N, t0);
    return hipGetLastError();
}

namespace {
__global__ __launch_bounds__(256) void copy_kernel(float* __restrict__ dst, const float* __restrict__ src, long long n) {
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < n; i += 256LL * gridDim.x) dst[i] = src[i];
}
constexpr int UPLOAD_CHUNK_WORDS = 960;      // 3840 bytes of kernel arguments
struct UploadChunk { uint32_t w[UPLOAD_CHUNK_WORDS]; };
__global__ __launch_bounds__(256) void upload_words_kernel(uint32_t* __restrict__ dst, UploadChunk c, int n) {
    for (int i = threadIdx.x; i < n; i += 256) dst[i] = c.w[i];
}
}  // namespace

namespace {
__global__ __launch_bounds__(256) void transpose_kernel(float* __restrict__ dst, const float* __restrict__ src, int rows, int cols) {
    __shared__ float tile[32][33];
    const int c0 = blockIdx.x * 32, r0 = blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int i = ty; i < 32; i += 8)
        if (r0 + i < rows && c0 + tx < cols) tile[i][tx] = src[(size_t)(r0 + i) * cols + c0 + tx];
    __syncthreads();
    for (int i = ty; i < 32; i += 8)
        if (c0 + i < cols && r0 + tx < rows) dst[(size_t)(c0 + i) * rows + r0 + tx] = tile[tx][i];
}
}  // namespace

hipError_t launch_transpose(float* dst, const float* src, int rows, int cols, hipStream_t stream) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    hipLaunchKernelGGL(transpose_kernel, dim3((cols + 31) / 32, (rows + 31) / 32), dim3(256), 0, stream, dst, src, rows, cols);
    return hipGetLastError();
}

hipError_t launch_copy(float* dst, const float* src, int64_t n, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, dst, src, (long long)n);
    return hipGetLastError();
}

hipError_t launch_upload_words(uint32_t* d_dst, const uint32_t* h_src, int64_t n, hipStream_t stream) {
    for (int64_t off = 0; off < n; off += UPLOAD_CHUNK_WORDS) {
        UploadChunk c;
        const int m = (int)std::min<int64_t>(UPLOAD_CHUNK_WORDS, n - off);
        for (int i = 0; i < m; ++i) c.w[i] = h_src[off + i];
        hipLaunchKernelGGL(upload_words_kernel, dim3(1), dim3(256), 0, stream, d_dst + off, c, m);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

namespace {
// blockIdx.x: the buffer; behind the last one the control words.
__global__ __launch_bounds__(256) void zero_history_kernel(float* const* __restrict__ buf_ptr, const int64_t* __restrict__ frame_floats, int n_bufs, int frames,
                                                           unsigned* __restrict__ ctrl, int ctrl_words) {
    const int b = blockIdx.x;
    if (b == n_bufs) {
        if (blockIdx.y == 0) for (int i = threadIdx.x; i < ctrl_words; i += 256) ctrl[i] = 0u;
        return;
    }
    const long long n = (long long)frames * frame_floats[b];
    if (n <= 0) return;
    float* p = buf_ptr[b];
    for (long long i = blockIdx.y * 256 + threadIdx.x; i < n; i += 256LL * gridDim.y) p[i] = 0.0f;
}

// y(t) <- y(t + frames) for all stored frames of up to SHIFT_MAX_TENSORS tensors.  A thread walks a chain of its own, the elements
// that lie whole shifts apart (of one or four floats), so that source and destination may overlap; eight of
// a chain's elements are in flight, in registers (with HIP's own uint4 they lay in scratch between load and store: 2 x 512
// LSTM on 32 streams, 16 of 256 frames 137 -> 97 us).  One copy per tensor and piece before: 2 x 512 LSTM, 256 of 512 frames 121 -> 8 us, one of 2 frames 59 -> 3 us.
typedef unsigned int shift_uint4 __attribute__((ext_vector_type(4)));
template <class V>
__device__ __forceinline__ void shift_tensor(V* y, long long frame, int frames, int stored) {
    const long long step = frame * frames, last = frame * (stored - frames);
    for (long long i = (long long)blockIdx.x * 256 + threadIdx.x; i < step && i < last; i += 256LL * gridDim.x) {
        long long at = i;
        for (; at + 7 * step < last; at += 8 * step) {
            V v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = y[at + (j + 1) * step];
#pragma unroll
            for (int j = 0; j < 8; ++j) y[at + j * step] = v[j];
        }
        for (; at < last; at += step) y[at] = y[at + step];
    }
}
__global__ __launch_bounds__(256) void shift_frames_kernel(const ShiftTensors s, int frames, int stored) {
    const int b = blockIdx.y;
    void* p = s.p[b];
    if (s.frame_words[b] % 4 == 0 && ((uintptr_t)p & 15) == 0) shift_tensor(static_cast<shift_uint4*>(p), s.frame_words[b] / 4, frames, stored);
    else shift_tensor(static_cast<uint32_t*>(p), s.frame_words[b], frames, stored);
}
}  // namespace

hipError_t launch_zero_history(float* const* buf_ptr, const int64_t* frame_floats, int n_bufs, int frames, unsigned* ctrl, int ctrl_words, hipStream_t stream) {
    hipLaunchKernelGGL(zero_history_kernel, dim3((unsigned)n_bufs + 1, frames > 0 ? 4 : 1), dim3(256), 0, stream, buf_ptr, frame_floats, n_bufs, frames, ctrl, ctrl_words);
    return hipGetLastError();
}

hipError_t launch_shift_frames(const ShiftTensors& s, int frames, int stored, hipStream_t stream) {
    if (s.count <= 0) return hipSuccess;
    int64_t most = 0;
    for (int i = 0; i < s.count; ++i) most = std::max(most, s.frame_words[i] * std::min(frames, stored - frames));
    const dim3 grid((unsigned)std::max<int64_t>(1, std::min<int64_t>((most / 4 + 255) / 256, 1024)), (unsigned)s.count);
    hipLaunchKernelGGL(shift_frames_kernel, grid, dim3(256), 0, stream, s, frames, stored);
    return hipGetLastError();
}

hipError_t launch_fill(float* p, int64_t n, float v, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    long long blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, p, (long long)n, v);
    return hipGetLastError();
}


namespace {
// One-hot source (Section 4's word-input layer): C[f][j] (+)= W[j][idx[f - shift]] for rows f of
// frames [row0, row0 + rows); an index of -1 (or a frame before the window) contributes nothing.
__global__ __launch_bounds__(256) void onehot_gather_kernel(float* __restrict__ C, const float* __restrict__ W, const int* __restrict__ idx,
                                                            int n_dst, int n_src, long long row0, long long rows, long long shift_rows,
                                                            long long total_rows, int accumulate) {
    for (long long r = blockIdx.x; r < rows; r += gridDim.x) {
        const long long f = row0 + r, fs = f - shift_rows;
        const int c = (fs >= 0 && fs < total_rows) ? idx[fs] : -1;
        for (int j = threadIdx.x; j < n_dst; j += 256) {
            const float v = (c >= 0 && c < n_src) ? W[(size_t)j * n_src + c] : 0.0f;
            float* dst = C + f * n_dst + j;
            *dst = accumulate ? *dst + v : v;
        }
    }
}
// G[j][c] = sum of ds[f][j] over the rows f >= shift with idx[f - shift] = c, for a whole row segment j, [c0, c0 + OHR_SEGMENT):
// bound by the write of G.  The segment is summed up in LDS (80 KiB, two workgroups per compute unit) and stored once, so
// G needs no zeros in it and takes no atomics in memory, each of which moves a line.  Row j goes to XCD j / (n_dst / 8), so that
// the workgroups that read neighbouring columns of ds share its lines in one L2.
// 4 gates of 512 x 38,000, 2048 frames: 0.17 ms less per window than zero fill and scatter (2.72 -> 2.56 ms).
constexpr int OHR_THREADS = 1024, OHR_SEGMENT = 20480;
__global__ __launch_bounds__(OHR_THREADS) void onehot_grad_rows_kernel(float* __restrict__ G, const float* __restrict__ ds, const int* __restrict__ idx,
                                                                       int n_dst, int n_src, long long shift_rows, long long total_rows) {
    __shared__ __align__(16) float row[OHR_SEGMENT];
    const int tid = threadIdx.x, x = blockIdx.x & 7, q = n_dst / 8, r = n_dst - 8 * q;
    const int j = x * q + (x < r ? x : r) + (int)(blockIdx.x >> 3);
    const int c0 = (int)blockIdx.y * OHR_SEGMENT, n = min(OHR_SEGMENT, n_src - c0);
    for (int i = tid; i < OHR_SEGMENT / 4; i += OHR_THREADS) reinterpret_cast<float4*>(row)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    __syncthreads();
    for (long long f = shift_rows + tid; f < total_rows; f += OHR_THREADS) {
        const int c = idx[f - shift_rows] - c0;
        if (c >= 0 && c < n) unsafeAtomicAdd(&row[c], ds[f * n_dst + j]);
    }
    __syncthreads();
    float* dst = G + (size_t)j * n_src + c0;
    for (int i = 4 * tid; i < n; i += 4 * OHR_THREADS) {
        if (i + 3 < n) {
            *reinterpret_cast<floatx4u*>(dst + i) = floatx4u{row[i], row[i + 1], row[i + 2], row[i + 3]};
        } else {
            for (int e = i; e < n; ++e) dst[e] = row[e];
        }
    }
}
// G[j][idx[f - shift]] += ds[f][j] over all rows f >= shift.
__global__ __launch_bounds__(256) void onehot_scatter_kernel(float* __restrict__ G, const float* __restrict__ ds, const int* __restrict__ idx,
                                                             int n_dst, int n_src, long long shift_rows, long long total_rows) {
    for (long long f = shift_rows + blockIdx.x; f < total_rows; f += gridDim.x) {
        const int c = idx[f - shift_rows];
        if (c < 0 || c >= n_src) continue;
        for (int j = threadIdx.x; j < n_dst; j += 256) unsafeAtomicAdd(&G[(size_t)j * n_src + c], ds[f * n_dst + j]);
    }
}
}  // namespace

hipError_t launch_onehot_gather(float* C, const float* W, const int* idx, int n_dst, int n_src, int64_t row0, int64_t rows,
                                int64_t shift_rows, int64_t total_rows, bool accumulate, hipStream_t stream) {
    if (rows <= 0) return hipSuccess;
    const int grid = (int)std::min<int64_t>(rows, 8192);
    hipLaunchKernelGGL(onehot_gather_kernel, dim3(grid), dim3(256), 0, stream, C, W, idx, n_dst, n_src, (long long)row0, (long long)rows,
                       (long long)shift_rows, (long long)total_rows, accumulate ? 1 : 0);
    return hipGetLastError();
}

bool onehot_grad_in_rows(int n_dst, int n_src, int64_t rows) {
    return n_src >= 4096 && rows <= n_src && n_dst <= (1 << 20);
}

hipError_t launch_onehot_grad_rows(float* G, const float* ds, const int* idx, int n_dst, int n_src, int64_t shift_rows, int64_t total_rows,
                                   hipStream_t stream) {
    hipLaunchKernelGGL(onehot_grad_rows_kernel, dim3(n_dst, (n_src + OHR_SEGMENT - 1) / OHR_SEGMENT), dim3(OHR_THREADS), 0, stream, G, ds, idx,
                       n_dst, n_src, (long long)shift_rows, (long long)total_rows);
    return hipGetLastError();
}

namespace {
// The same sum with one writer per element: thread j walks the rows in order.
__global__ __launch_bounds__(256) void onehot_scatter_ordered_kernel(float* __restrict__ G, const float* __restrict__ ds, const int* __restrict__ idx,
                                                                     int n_dst, int n_src, long long shift_rows, long long total_rows) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= n_dst) return;
    for (long long f = shift_rows; f < total_rows; ++f) {
        const int c = idx[f - shift_rows];
        if (c >= 0 && c < n_src) G[(size_t)j * n_src + c] += ds[f * n_dst + j];
    }
}
}  // namespace

hipError_t launch_onehot_scatter(float* G, const float* ds, const int* idx, int n_dst, int n_src, int64_t shift_rows, int64_t total_rows,
                                 bool ordered, hipStream_t stream) {
    if (total_rows - shift_rows <= 0) return hipSuccess;
    if (ordered) {
        hipLaunchKernelGGL(onehot_scatter_ordered_kernel, dim3((n_dst + 255) / 256), dim3(256), 0, stream, G, ds, idx, n_dst, n_src,
                           (long long)shift_rows, (long long)total_rows);
        return hipGetLastError();
    }
    const int grid = (int)std::min<int64_t>(total_rows - shift_rows, 8192);
    hipLaunchKernelGGL(onehot_scatter_kernel, dim3(grid), dim3(256), 0, stream, G, ds, idx, n_dst, n_src, (long long)shift_rows, (long long)total_rows);
    return hipGetLastError();
}

}  // namespace rnng
