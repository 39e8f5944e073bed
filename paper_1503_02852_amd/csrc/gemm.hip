// Grouped GEMM with fp32 operands and results on the CDNA matrix cores, for the batched part of the
// intra-stream schedule (paper Section 3.1: everything outside the recurrent nodes is computed for
// all frames of the window at once) and for the weight gradients (Section 2.2, last equation: a sum
// over all frames of outer products, i.e. one GEMM whose contraction runs over frames).
//
// Products in three bf16 parts.  v_mfma_f32_32x32x2_f32 does 64 multiply-adds per clock and SIMD,
// v_mfma_f32_32x32x16_bf16 512, with the same fp32 accumulators.  An fp32 number is the exact sum
// of three bf16 numbers (8 + 8 + 8 significant bits; a0 = bf16(a), a1 = bf16(a - a0), a2 = a - a0 - a1),
// so a product a b is the sum of nine exact products of parts; the three smallest (a1 b2, a2 b1,
// a2 b2, below 2^-26 |a b|, an eighth of the rounding of one fp32 addition) are left out and six
// matrix instructions do the work of eight fp32 ones in 6/64 of their time.  Sums stay fp32.
// A part of a number that is not finite, or rounds to infinity, is NaN, and so is its whole row or
// column of the tile: a workgroup that finds a result that is not finite computes its tile again
// with fp32 instructions (tile_fp32), which gives the infinities and NaN of the operands.
#include <cstdlib>

#include "kernels.h"

namespace rnng {
namespace {

constexpr int BM = 128, BN = 128, NTHREADS = 256;
constexpr int XK = 32;                   // k per chunk of the bf16 loop
constexpr int XOCTET = 130;              // 16-byte units from one octet of a plane to the next: 128 rows, and 2 so that
                                         // eight threads that store four octets of two rows use different banks
constexpr int XPLANE = XK / 8 * XOCTET;  // units per part

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

// =============================================================================================
// fp32 instructions: tiles with results that are not finite
// =============================================================================================
// K chunk 16; operand tiles go through LDS in k-major order ([k][m], row stride 132 floats) so that
// the operand fetch of a wavefront is a conflict-free ds_read_b32 for both operand orientations.
constexpr int BK = 16;
constexpr int STRIDE = 132;   // floats per k-row in LDS

// ---- K-contiguous source: element (r, k) at base[(r + row_off) * ld + k] --------------------
__device__ __forceinline__ void load_kc(float (&r)[8], const float* __restrict__ base, int ld, int row0, int row_limit,
                                        int row_off, int src_rows, int k0, int k_limit, bool vec_ok, int tid) {
    const int k = k0 + 4 * (tid & 3);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int row = row0 + (tid >> 2) + 64 * j;
        const int srow = row + row_off;
        const bool ok = row < row_limit && srow >= 0 && srow < src_rows;
        const float* p = base + (size_t)(ok ? srow : 0) * ld + k;
        if (ok && vec_ok && k + 3 < k_limit) {
            floatx4 v = *reinterpret_cast<const floatx4*>(p);
            r[4 * j + 0] = v.x; r[4 * j + 1] = v.y; r[4 * j + 2] = v.z; r[4 * j + 3] = v.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) r[4 * j + e] = (ok && k + e < k_limit) ? p[e] : 0.0f;
        }
    }
}
// A thread holds four consecutive k of one row; k rows lie 132 floats apart, so the four threads
// that share a row index group would hit two banks twice if all stored their element e at once.
// Instruction i stores element (e0 + i) % 4 with e0 = 0, 2, 2, 0 for tid % 4 = 0 .. 3: the 32 lanes
// of a half-wavefront then fall into four disjoint windows of eight banks.
__device__ __forceinline__ void store_kc(float* __restrict__ lds, const float (&r)[8], int tid) {
    const int a = tid & 3, e0 = (a == 1 || a == 2) ? 2 : 0;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int e = (e0 + i) & 3;
            const float v = e == 0 ? r[4 * j] : e == 1 ? r[4 * j + 1] : e == 2 ? r[4 * j + 2] : r[4 * j + 3];
            lds[(4 * a + e) * STRIDE + (tid >> 2) + 64 * j] = v;
        }
}

// ---- M/N-contiguous source: element (k, c) at base[k * ld + c] ------------------------------
__device__ __forceinline__ void load_mc(float (&r)[8], const float* __restrict__ base, int ld, int c0, int c_limit,
                                        int k0, int k_limit, bool vec_ok, int tid) {
    const int c = c0 + 4 * (tid & 31);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int k = k0 + (tid >> 5) + 8 * j;
        const bool ok = k < k_limit;
        const float* p = base + (size_t)(ok ? k : 0) * ld + c;
        if (ok && vec_ok && c + 3 < c_limit) {
            floatx4 v = *reinterpret_cast<const floatx4*>(p);
            r[4 * j + 0] = v.x; r[4 * j + 1] = v.y; r[4 * j + 2] = v.z; r[4 * j + 3] = v.w;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) r[4 * j + e] = (ok && c + e < c_limit) ? p[e] : 0.0f;
        }
    }
}
__device__ __forceinline__ void store_mc(float* __restrict__ lds, const float (&r)[8], int tid) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        floatx4 v = {r[4 * j + 0], r[4 * j + 1], r[4 * j + 2], r[4 * j + 3]};
        *reinterpret_cast<floatx4*>(&lds[((tid >> 5) + 8 * j) * STRIDE + 4 * (tid & 31)]) = v;
    }
}

template <bool A_KC, bool B_KC>
__device__ __forceinline__ void tile_fp32(const GemmProblem& P, int split, int split_k, int m0, int n0, float* __restrict__ sA,
                                       floatx16 (&acc)[2][2]) {
    float* const sB = sA + BK * STRIDE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.0f;
    for (int p = 0; p < P.n_pairs; ++p) {
        const GemmPair pr = P.pairs[p];
        const int nk = (pr.K + XK - 1) / XK;      // the share of the contraction is the one of the bf16 loop
        const int k_begin = (int)((long long)nk * split / split_k) * XK;
        const int k_end = min(pr.K, (int)((long long)nk * (split + 1) / split_k) * XK);
        const bool a_vec = (pr.lda & 3) == 0 && aligned16(pr.A);
        const bool b_vec = (pr.ldb & 3) == 0 && aligned16(pr.B);
        float ra[8], rb[8];
        for (int k0 = k_begin; k0 < k_end; k0 += BK) {
            if (A_KC) load_kc(ra, pr.A, pr.lda, m0, P.M, pr.a_row_off, pr.a_rows, k0, k_end, a_vec, tid);
            else load_mc(ra, pr.A, pr.lda, m0, P.M, k0, k_end, a_vec, tid);
            if (B_KC) load_kc(rb, pr.B, pr.ldb, n0, P.N, 0, P.N, k0, k_end, b_vec, tid);
            else load_mc(rb, pr.B, pr.ldb, n0, P.N, k0, k_end, b_vec, tid);
            __syncthreads();
            if (A_KC) store_kc(sA, ra, tid); else store_mc(sA, ra, tid);
            if (B_KC) store_kc(sB, rb, tid); else store_mc(sB, rb, tid);
            __syncthreads();
#pragma unroll
            for (int kk = 0; kk < BK / 2; ++kk) {
                const int krow = (2 * kk + (lane >> 5)) * STRIDE + (lane & 31);
                const float a0 = sA[krow + wm * 64], a1 = sA[krow + wm * 64 + 32];
                const float b0 = sB[krow + wn * 64], b1 = sB[krow + wn * 64 + 32];
                acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b0, acc[0][0], 0, 0, 0);
                acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, b1, acc[0][1], 0, 0, 0);
                acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b0, acc[1][0], 0, 0, 0);
                acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, b1, acc[1][1], 0, 0, 0);
            }
        }
    }
}

// =============================================================================================
// bf16 parts
// =============================================================================================
// Block tile 128 x 128, 4 wavefronts in a 2 x 2 arrangement, each with a 64 x 64 sub-tile as 2 x 2
// accumulators of 32 x 32.  Chunk of 32 k: a thread loads 16 values of each operand ahead of time
// (under the previous chunk's products), splits them and stores them to LDS as octets of eight k
// of one row, one plane per part, [plane][octet][row]: a wavefront's 128-bit operand reads are
// consecutive.  Octet q of a chunk holds k = 4 q .. 4 q + 3 and 16 + 4 q .. 16 + 4 q + 3 (the order of a
// contraction is free), so that four threads that share a row load 64 consecutive bytes.
__device__ __forceinline__ int octet_k(int q, int e) { return 4 * q + (e & 3) + 4 * (e & 4); }

// K-contiguous source: element (r, k) at base[(r + row_off) * ld + k].  Thread: octet tid % 4 of rows tid / 4 and
// tid / 4 + 64.  M/N-contiguous source: element (k, c) at base[k * ld + c].  Thread: octet tid / 64 of columns tid % 64
// and tid % 64 + 64 (a wavefront's load is 256 consecutive bytes, whatever the alignment).  Rows or columns
// beyond the matrix take the last one's values: their results are not stored.
// A chunk that lies whole in the contraction, of rows that lie whole in the source, is loaded
// without branches from one scalar address (`chunk`: the tile's first row and the chunk's first k, or
// the chunk's first k and the tile's first column) with 32-bit lane offsets kept for the whole tile.
typedef floatx4 floatx4u __attribute__((aligned(4)));      // (128-bit global loads need 4-byte alignment only)
struct LaneOffsets { unsigned at[2]; };                     // bytes
template <bool KC>
__device__ __forceinline__ LaneOffsets lane_offsets(int ld, int first, int limit, int tid) {
    LaneOffsets o;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int r = min(first + (KC ? tid >> 2 : tid & 63) + 64 * j, limit - 1) - first;
        o.at[j] = 4u * (KC ? (unsigned)r * (unsigned)ld + 4u * (tid & 3) : (unsigned)r);
    }
    return o;
}
template <bool KC>
__device__ __forceinline__ void xload_whole(float (&r)[16], const float* __restrict__ chunk, int ld, const LaneOffsets& o, int tid) {
    if (KC) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const floatx4 v = *reinterpret_cast<const floatx4u*>(reinterpret_cast<const char*>(chunk + 16 * h) + o.at[j]);
#pragma unroll
                for (int e = 0; e < 4; ++e) r[8 * j + 4 * h + e] = v[e];
            }
    } else {
        const int q = __builtin_amdgcn_readfirstlane(tid >> 6);
        const float* p = chunk + (size_t)(4 * q) * ld;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
#pragma unroll
            for (int j = 0; j < 2; ++j) r[8 * j + e] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p) + o.at[j]);
            p += e == 3 ? (size_t)13 * ld : (size_t)ld;
        }
    }
}
__device__ __forceinline__ void xload_kc(float (&r)[16], const float* __restrict__ base, int ld, int row0, int row_limit,
                                         int row_off, int src_rows, int k0, int k_limit, int tid) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int srow = min(row0 + (tid >> 2) + 64 * j, row_limit - 1) + row_off;
        const bool ok = srow >= 0 && srow < src_rows;
        const float* p = base + (size_t)(ok ? srow : 0) * ld;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + octet_k(tid & 3, e);
            r[8 * j + e] = (ok && k < k_limit) ? p[k] : 0.0f;
        }
    }
}
__device__ __forceinline__ void xload_mc(float (&r)[16], const float* __restrict__ base, int ld, int c0, int c_limit,
                                         int k0, int k_limit, int tid) {
    const int q = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const int c = min(c0 + (tid & 63) + 64 * j, c_limit - 1);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int k = k0 + octet_k(q, e);      // (uniform)
            r[8 * j + e] = k < k_limit ? base[(size_t)k * ld + c] : 0.0f;
        }
    }
}
// Splits eight values and stores the octet's three parts.
__device__ __forceinline__ void store_octet(uintx4* __restrict__ lds, const float* __restrict__ v, int q, int row) {
    uintx4 part[3];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        floatx2 x = {v[2 * i], v[2 * i + 1]};
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            const bf16x2 b = __builtin_convertvector(x, bf16x2);
            const unsigned u = __builtin_bit_cast(unsigned, b);
            part[p][i] = u;
            x.x -= __uint_as_float(u << 16);
            x.y -= __uint_as_float(u & 0xffff0000u);
        }
    }
#pragma unroll
    for (int p = 0; p < 3; ++p) lds[p * XPLANE + q * XOCTET + row] = part[p];
}
template <bool KC>
__device__ __forceinline__ void xstore(uintx4* __restrict__ lds, const float (&r)[16], int tid) {
#pragma unroll
    for (int j = 0; j < 2; ++j) store_octet(lds, r + 8 * j, KC ? tid & 3 : tid >> 6, (KC ? tid >> 2 : tid & 63) + 64 * j);
}

template <bool A_KC, bool B_KC>
__global__ __launch_bounds__(NTHREADS, 2) void gemm_kernel(const GemmGroup g) {
    __shared__ uintx4 lds[2 * 3 * XPLANE];
    uintx4* const sA = lds;
    uintx4* const sB = lds + 3 * XPLANE;

    const int pi = blockIdx.z / g.split_k;
    const int split = blockIdx.z - pi * g.split_k;
    const GemmProblem& P = g.p[pi];
    const int tiles_m = (P.M + BM - 1) / BM, tiles_n = (P.N + BN - 1) / BN;
    const int n_tiles = tiles_m * tiles_n;
    if ((int)blockIdx.x >= n_tiles) return;
    // Which tile a workgroup takes.  Workgroups go to the eight XCDs in turn and each XCD has an
    // L2 of its own, so workgroup b takes tile start(b % 8) + b / 8: every XCD works on one
    // consecutive range of tiles.  Inside the range the tiles run down groups of g.group_m row
    // blocks before they move to the next column block, so that the workgroups that are resident
    // together on an XCD share both A panels and B panels in its L2.
    int tile = blockIdx.x;
    const int GM = g.group_m;
    if (GM > 0) {
        const int q = n_tiles / 8, r = n_tiles - 8 * q, x = tile & 7;
        tile = x * q + (x < r ? x : r) + (tile >> 3);
    }
    int tm, tn;
    if (GM > 1) {
        const int per_group = GM * tiles_n, group = tile / per_group, first_m = group * GM;
        const int gsz = tiles_m - first_m < GM ? tiles_m - first_m : GM;
        const int in_group = tile - group * per_group;
        tn = in_group / gsz; tm = first_m + in_group - tn * gsz;
    } else {
        tm = tile / tiles_n; tn = tile - tm * tiles_n;
    }
    const int m0 = tm * BM, n0 = tn * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // acc: products of leading parts; low: the others, 2^-8 of acc, so that their sums round far below
    // acc's.  2-norm errors against float64, fp32 instructions / one accumulator / two: K = 38,000
    // 1.23e-6 / 1.27e-6 / 4.2e-7, K = 512 4.0e-7 / 3.4e-7 / 1.2e-7.
    floatx16 acc[2][2], low[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = low[a][b][e] = 0.0f;

    for (int p = 0; p < P.n_pairs; ++p) {
        const GemmPair pr = P.pairs[p];
        const int nk = (pr.K + XK - 1) / XK;
        const int c_begin = (int)((long long)nk * split / g.split_k);
        const int c_end = (int)((long long)nk * (split + 1) / g.split_k);
        if (c_begin >= c_end) continue;
        float ra[16], rb[16];
        const int a_first = m0 + pr.a_row_off, a_last = min(m0 + BM, P.M) - 1 + pr.a_row_off;
        const bool rows_whole = (!A_KC || (a_first >= 0 && a_last < pr.a_rows && pr.lda < (1 << 22))) && (!B_KC || pr.ldb < (1 << 22));
        const LaneOffsets ao = lane_offsets<A_KC>(pr.lda, m0, P.M, tid), bo = lane_offsets<B_KC>(pr.ldb, n0, P.N, tid);
        auto fetch = [&](int c) {
            const int k0 = c * XK;
            if (rows_whole && k0 + XK <= pr.K) {
                xload_whole<A_KC>(ra, A_KC ? pr.A + (ptrdiff_t)a_first * pr.lda + k0 : pr.A + (size_t)k0 * pr.lda + m0, pr.lda, ao, tid);
                xload_whole<B_KC>(rb, B_KC ? pr.B + (size_t)n0 * pr.ldb + k0 : pr.B + (size_t)k0 * pr.ldb + n0, pr.ldb, bo, tid);
            } else {
                if (A_KC) xload_kc(ra, pr.A, pr.lda, m0, P.M, pr.a_row_off, pr.a_rows, k0, pr.K, tid);
                else xload_mc(ra, pr.A, pr.lda, m0, P.M, k0, pr.K, tid);
                if (B_KC) xload_kc(rb, pr.B, pr.ldb, n0, P.N, 0, P.N, k0, pr.K, tid);
                else xload_mc(rb, pr.B, pr.ldb, n0, P.N, k0, pr.K, tid);
            }
        };
        fetch(c_begin);
        for (int c = c_begin; c < c_end; ++c) {
            __syncthreads();
            xstore<A_KC>(sA, ra, tid);
            xstore<B_KC>(sB, rb, tid);
            __syncthreads();
            if (c + 1 < c_end) fetch(c + 1);
#pragma unroll
            for (int kk = 0; kk < XK / 16; ++kk) {
                bf16x8 a[2][3], b[2][3];
                const int at = (2 * kk + (lane >> 5)) * XOCTET + (lane & 31);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int q = 0; q < 3; ++q) {
                        a[i][q] = __builtin_bit_cast(bf16x8, sA[q * XPLANE + at + wm * 64 + 32 * i]);
                        b[i][q] = __builtin_bit_cast(bf16x8, sB[q * XPLANE + at + wn * 64 + 32 * i]);
                    }
                // small products first
                constexpr int PA[6] = {2, 0, 1, 1, 0, 0}, PB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
                for (int q = 0; q < 6; ++q)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) {
                            floatx16& to = q == 5 ? acc[i][j] : low[i][j];
                            to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i][PA[q]], b[j][PB[q]], to, 0, 0, 0);
                        }
            }
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) acc[a][b] += low[a][b];

    // x - x is 0 for a finite x, else NaN
    float check = 0.0f;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) check += acc[a][b][e] - acc[a][b][e];
    if (__syncthreads_or(check != 0.0f)) tile_fp32<A_KC, B_KC>(P, split, g.split_k, m0, n0, reinterpret_cast<float*>(lds), acc);

    // 32x32 accumulator layout: register e of lane l holds row 8*(e/4) + 4*(l/32) + e%4, column l%32.
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int col = n0 + wn * 64 + b * 32 + (lane & 31);
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int row = m0 + wm * 64 + a * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
                if (row < P.M && col < P.N) {
                    float* dst = P.C + (size_t)row * P.ldc + col;
                    if (g.split_k > 1) unsafeAtomicAdd(dst, acc[a][b][e]);
                    else if (g.accumulate) *dst += acc[a][b][e];
                    else *dst = acc[a][b][e];
                }
            }
        }
}

}  // namespace

hipError_t launch_gemm_group(GemmMode mode, const GemmGroup& g, hipStream_t stream) {
    if (g.n_problems <= 0) return hipSuccess;
    int max_tiles = 0;
    for (int i = 0; i < g.n_problems; ++i) {
        const int t = ((g.p[i].M + BM - 1) / BM) * ((g.p[i].N + BN - 1) / BN);
        max_tiles = t > max_tiles ? t : max_tiles;
    }
    if (max_tiles == 0) return hipSuccess;
    dim3 grid(max_tiles, 1, g.n_problems * g.split_k), block(NTHREADS);
    static const int group_m = [] { const char* env = std::getenv("RNNG_GEMM_GROUP_M"); return env ? std::atoi(env) : 8; }();
    GemmGroup gg = g;
    gg.group_m = group_m < 0 ? 0 : group_m;
    switch (mode) {
        case GEMM_NT: hipLaunchKernelGGL((gemm_kernel<true, true>), grid, block, 0, stream, gg); break;
        case GEMM_NN: hipLaunchKernelGGL((gemm_kernel<true, false>), grid, block, 0, stream, gg); break;
        case GEMM_TN: hipLaunchKernelGGL((gemm_kernel<false, false>), grid, block, 0, stream, gg); break;
    }
    return hipGetLastError();
}

}  // namespace rnng
