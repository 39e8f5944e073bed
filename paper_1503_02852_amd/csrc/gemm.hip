// Grouped fp32 GEMM on the CDNA matrix cores (v_mfma_f32_32x32x2_f32) for the batched part of
// the intra-stream schedule (paper Section 3.1: everything outside the recurrent nodes is
// computed for all frames of the window at once) and for the weight gradients (Section 2.2,
// last equation: a sum over all frames of outer products, i.e. one GEMM whose contraction
// runs over frames).
//
// gemm_kernel: tiles of 128 x 128 or 64 x 64, 256 threads = 4 wavefronts in a 2 x 2 arrangement, the
// contraction in chunks of 16.  Bound by the matrix instructions, which a SIMD takes at one per 64
// clocks as long as nothing else asks for the vector pipe when the next one is due: one vector
// instruction per matrix instruction, as address arithmetic and bounds tests came to, cost 15 % of
// the rate.  So the time loop has none besides the copies to LDS:
//   - global loads go through buffer descriptors, moved ahead in scalar registers; the bounds check
//     takes the place of every test of a row or column (a row or a column outside the matrix reads zeros or
//     a neighbour's values, and these reach only results that are not stored);
//   - both operands lie in LDS as [k][row], XOR-swizzled, so that every operand fetch is
//     ds_read2st64_b32 from one base register with constant offsets, free of bank conflicts;
//   - two LDS buffers, one barrier per chunk, operands fetched one group of multiplications ahead.
// 8,192^3 library product 153 TFLOP/s; four products 8192 x 1024 x 1024 (NT) 112 -> 137 TFLOP/s, eight of
// 4096 x 4096, K = 2048 (TN) 131 -> 144, 8192 x 1024 from four gates (NN) 117 -> 137, 2048 x 20,000 x 512 105 -> 130.
//
// gemm_small_kernel: tiles of 32 x 32 for the products that have few tiles of the larger kind, where what
// counts is how long one workgroup takes to walk its contraction.  Eight wavefronts take the chunks
// in turn, each straight from memory into the operand registers (no LDS, four chunks in flight, so that the
// latency is paid once per 512 columns), and add their parts up in LDS.  1 x 30 x 512: 61 -> 5.5 us, 1024 x 61 x 256
// 36 -> 5.2, 61 x 256, K = 1024 (TN) 20 -> 4.0.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "graph.h"
#include "interp.h"
#include "kernels.h"

namespace rnng {
namespace {

constexpr int BK = 16, NTHREADS = 256;
constexpr int RSRC_FLAGS = 0x00020000;
constexpr int OUTSIDE = (int)0x80000000u;      // a byte offset beyond every descriptor

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int uintx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int rsrc_bytes(long long floats) {
    return floats <= 0 ? 0 : floats < (1 << 29) - 1 ? (int)(4 * floats) : 0x7ffffffc;
}
__device__ __forceinline__ int chunks_of(int K) { return K / BK + (K % BK != 0); }
// the part of n chunks that belongs to part `split` of `parts`
__device__ __forceinline__ void chunk_range(int n, int split, int parts, int& begin, int& end) {
    const int q = n / parts, r = n - q * parts;
    begin = split * q + min(split, r);
    end = begin + q + (split < r ? 1 : 0);
}
// The problem that workgroup b belongs to.
__device__ __forceinline__ int problem_of(const GemmGroup& g, int b) {
    const int lane = threadIdx.x & 63;
    const bool mine = lane < g.n_problems && b >= g.first_block[lane < g.n_problems ? lane : 0];
    return __builtin_amdgcn_readfirstlane(__popcll(__ballot(mine)) - 1);
}

// One operand of a tile: R = 64 T rows (of A) or columns (of B), chunk by chunk.
//   KC:  K-contiguous, element (row, k) at base[(row + row_off) * ld + k]; rows outside [0, src_rows) are zero
//   !KC: element (k, c) at base[k * ld + c]
// A thread loads T times four consecutive floats of a chunk: of one row (KC) or of one k.
template <bool KC, int T> struct Operand {
    static constexpr int R = 64 * T, LDS = BK * R, C4 = R / 4;
    const float* p; long long left;      // from the chunk's first element; floats until the matrix ends
    int step, voff[T];
    __device__ __forceinline__ void begin(const float* base, int ld, int r0, int row_off, int src_rows, int K, int k0, int tid) {
        if (KC) {
            const int first = min(max(r0 + row_off, 0), src_rows - 1);
            p = base + (long long)first * ld + k0; left = (long long)(src_rows - first) * ld - k0; step = BK;
#pragma unroll
            for (int j = 0; j < T; ++j) {
                const int row = r0 + (tid >> 2) + 64 * j + row_off;
                voff[j] = row >= 0 && row < src_rows ? ((row - first) * ld + 4 * (tid & 3)) * 4 : OUTSIDE;
            }
        } else {
            p = base + (long long)k0 * ld + r0; left = (long long)(K - k0) * ld - r0; step = BK * ld;
#pragma unroll
            for (int j = 0; j < T; ++j) voff[j] = ((tid / C4 + NTHREADS / C4 * j) * ld + 4 * (tid % C4)) * 4;
        }
    }
    __device__ __forceinline__ void load(uintx4 (&r)[T]) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p), 0, rsrc_bytes(left), RSRC_FLAGS);
#pragma unroll
        for (int j = 0; j < T; ++j) r[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff[j], 0, 0);
        p += step; left -= step;
    }
    // Element (k, c) of a chunk lies at k R + (c ^ swizzle(k)).  The two halves of a wavefront fetch k and k + 1:
    // 32 floats apart they fall on different banks; a KC thread stores four k of one row, and the
    // quads' columns are moved by 16 so that the four threads of a row don't meet in a bank.
    static constexpr int swizzle(int k) { return (KC ? 16 * ((k >> 2) & 3) : 0) ^ (32 * (k & 1)); }
    __device__ __forceinline__ static void store(float* lds, const uintx4 (&r)[T], int tid, int k_left) {
        if (KC) {
            const int kq = tid & 3;
            float* even = lds + 4 * kq * R + ((tid >> 2) ^ (16 * kq));
            float* odd = lds + 4 * kq * R + R + ((tid >> 2) ^ (16 * kq) ^ 32);
#pragma unroll
            for (int j = 0; j < T; ++j) {
                uintx4 v = r[j];
                if (k_left < BK) {      // the row's end: what follows is another row
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = 4 * kq + e < k_left ? v[e] : 0u;
                }
                even[64 * j] = __uint_as_float(v[0]); odd[64 * j] = __uint_as_float(v[1]);
                even[64 * j + 2 * R] = __uint_as_float(v[2]); odd[64 * j + 2 * R] = __uint_as_float(v[3]);
            }
        } else {
#pragma unroll
            for (int j = 0; j < T; ++j) {
                const int k = tid / C4 + NTHREADS / C4 * j;
                *reinterpret_cast<uintx4*>(lds + k * R + ((4 * (tid % C4)) ^ swizzle(k))) = r[j];
            }
        }
    }
    // The operands of quad q (k = 4q .. 4q + 3): f[i][t] of multiply step i (k = 4q + 2i and the next one), row block t.
    __device__ __forceinline__ static const float* at(const float* lds, int row, int h, int q) { return lds + h * R + (row ^ (32 * h) ^ (KC ? 16 * q : 0)); }
    __device__ __forceinline__ static void fetch(float (&f)[2][T], const float* at, int q) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int t = 0; t < T; ++t) f[i][t] = at[(4 * q + 2 * i) * R + 64 * t];
    }
};

// What a node's program does to its products (interp.h), in the order it does it.
__device__ __forceinline__ float finish(float v, bool has_bias, float bias, int act) {
    if (has_bias) v += bias;
    return act == ACT_SIGMOID ? sigmoid_f(v) : act == ACT_TANH ? tanh_f(v) : act == ACT_RELU ? fmaxf(v, 0.0f) : v;
}

template <bool A_KC, bool B_KC, int T>
__global__ __launch_bounds__(NTHREADS, T == 2 ? 4 : 6) void gemm_kernel(const GemmGroup g) {
    using OA = Operand<A_KC, T>;
    using OB = Operand<B_KC, T>;
    constexpr int TILE = 64 * T, HALF = OA::LDS + OB::LDS;
    __shared__ __attribute__((aligned(16))) float lds[2 * HALF];

    // Which tile a workgroup takes.  Workgroups go to the eight XCDs in turn and each XCD has an
    // L2 of its own, so workgroup b takes tile start(b % 8) + b / 8: every XCD works on one
    // consecutive range of tiles.  Inside the range the tiles run down groups of g.group_m row
    // blocks before they move to the next column block, so that the workgroups that are resident
    // together on an XCD share both A panels and B panels in its L2.
    // (Ranges of a problem's own tiles, whose first workgroup is a multiple of 8: with ranges of a launch's tiles some XCDs got
    // the short contractions and others the long ones.)
    const int pi = problem_of(g, blockIdx.x);
    const GemmProblem& P = g.p[pi];
    const int tiles_m = (P.M + TILE - 1) / TILE, tiles_n = (P.N + TILE - 1) / TILE, n_tiles = tiles_m * tiles_n;
    int tile = blockIdx.x - g.first_block[pi], split = 0;
    if (tile >= n_tiles * P.split) return;
    if (g.group_m > 0) {
        const int n = n_tiles * P.split, q = n / 8, r = n - 8 * q, x = tile & 7;
        tile = x * q + min(x, r) + (tile >> 3);
    }
    if (P.split > 1) { split = tile / n_tiles; tile -= split * n_tiles; }
    int tm, tn;
    if (g.group_m > 1) {
        const int per_group = g.group_m * tiles_n, group = tile / per_group, first_m = group * g.group_m;
        const int gsz = min(tiles_m - first_m, g.group_m), in_group = tile - group * per_group;
        tn = in_group / gsz; tm = first_m + in_group - tn * gsz;
    } else {
        tm = tile / tiles_n; tn = tile - tm * tiles_n;
    }
    const int m0 = tm * TILE, n0 = tn * TILE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, h = lane >> 5;
    // a wavefront's row blocks lie 64 rows apart (the offset unit of ds_read2st64)
    const int arow = 32 * (wave >> 1) + (lane & 31), brow = 32 * (wave & 1) + (lane & 31);
    const float* pa[4]; const float* pb[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) { pa[q] = OA::at(lds, arow, h, q); pb[q] = OB::at(lds + OA::LDS, brow, h, q); }

    floatx16 acc[T][T];
#pragma unroll
    for (int x = 0; x < T; ++x)
#pragma unroll
        for (int y = 0; y < T; ++y)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[x][y][e] = 0.0f;

    auto sync = [&]() {      // orders LDS only: global loads stay in flight
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    for (int p = P.first_pair; p < P.first_pair + P.n_pairs; ++p) {
        const GemmPair& pr = g.pair[p];
        int c = 0, c_end = chunks_of(pr.K);
        if (P.split > 1) chunk_range(c_end, split, P.split, c, c_end);
        if (c >= c_end) continue;
        OA oa; OB ob;
        oa.begin(pr.A, pr.lda, m0, pr.a_row_off, pr.a_rows, pr.K, c * BK, tid);
        ob.begin(pr.B, pr.ldb, n0, 0, P.N, pr.K, c * BK, tid);
        int k_left = pr.K - c * BK;
        uintx4 ra[T], rb[T];
        float fa[2][2][T], fb[2][2][T];
        sync();      // the chunk behind the previous pair's last one has been fetched by everyone
        oa.load(ra); ob.load(rb);
        OA::store(lds, ra, tid, k_left); OB::store(lds + OA::LDS, rb, tid, k_left);
        oa.load(ra); ob.load(rb);
        sync();
        OA::fetch(fa[0], pa[0], 0); OB::fetch(fb[0], pb[0], 0);
        // Multiplies the chunk in one LDS buffer while the next one goes from registers to the other buffer and the one
        // after that is loaded.  Behind the last chunk the same happens with what lies there (inside the
        // descriptors' bounds) and is not used: no branch in the loop.
        auto chunk = [&](auto half) {
            constexpr int cur = decltype(half)::value * HALF, nxt = HALF - cur;
            k_left -= BK;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (q < 3) {
                    OA::fetch(fa[(q + 1) & 1], pa[q + 1] + cur, q + 1); OB::fetch(fb[(q + 1) & 1], pb[q + 1] + cur, q + 1);
                } else {
                    sync();
                    OA::fetch(fa[0], pa[0] + nxt, 0); OB::fetch(fb[0], pb[0] + nxt, 0);
                }
                if (q == 1) {
                    OA::store(lds + nxt, ra, tid, k_left); OB::store(lds + nxt + OA::LDS, rb, tid, k_left);
                    oa.load(ra); ob.load(rb);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int x = 0; x < T; ++x)
#pragma unroll
                        for (int y = 0; y < T; ++y) acc[x][y] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[q & 1][i][x], fb[q & 1][i][y], acc[x][y], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        while (true) {
            chunk(std::integral_constant<int, 0>{});
            if (++c == c_end) break;
            chunk(std::integral_constant<int, 1>{});
            if (++c == c_end) break;
        }
    }

    // 32x32 accumulator layout: register e of lane l holds row 8*(e/4) + 4*(l/32) + e%4, column l%32.
    const int row0 = m0 + 32 * (wave >> 1) + 4 * h;
    if (P.split > 1 || P.accumulate) {
#pragma unroll
        for (int x = 0; x < T; ++x)
#pragma unroll
            for (int y = 0; y < T; ++y)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int row = row0 + 64 * x + 8 * (e >> 2) + (e & 3), col = n0 + brow + 64 * y;
                    if (row < P.M && col < P.N) unsafeAtomicAdd(P.C + (size_t)row * P.ldc + col, acc[x][y][e]);
                }
        return;
    }
    const __amdgpu_buffer_rsrc_t rc = __builtin_amdgcn_make_buffer_rsrc(P.C + (long long)m0 * P.ldc + n0, 0, rsrc_bytes((long long)(P.M - m0) * P.ldc - n0), RSRC_FLAGS);
    const int row_bytes = 4 * P.ldc;
    // What finish() does, f chosen outside the unrolled elements and their values stored sixteen at a time: chosen per element, all of
    // them at once, it took 48 registers more than there are.
    auto store = [&](auto f) {
#pragma unroll
        for (int y = 0; y < T; ++y) {
            const int col = n0 + brow + 64 * y;
            const int at = col < P.N ? (row0 - m0) * row_bytes + 4 * (brow + 64 * y) : OUTSIDE;
            const float bias = P.bias != nullptr && col < P.N ? P.bias[col] : -0.0f;      // (v + -0 is v, -0 too)
#pragma unroll
            for (int x = 0; x < T; ++x) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(f(acc[x][y][e] + bias)), rc, at + (64 * x + 8 * (e >> 2) + (e & 3)) * row_bytes, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    };
    if (P.act == ACT_SIGMOID) store([](float v) { return sigmoid_f(v); });
    else if (P.act == ACT_TANH) store([](float v) { return tanh_f(v); });
    else if (P.act == ACT_RELU) store([](float v) { return fmaxf(v, 0.0f); });
    else store([](float v) { return v; });
}

constexpr int SMALL_WAVES = 8, SMALL_DEPTH = 4, SMALL_TILE = 32;
constexpr int SMALL_GRID_X = 1 << 16;      // workgroups beyond that go to the grid's y

// An operand of 32 rows or columns: a lane holds eight k of one of them, k = 8 (lane / 32) + 0 .. 7 of a chunk (the order in
// which a sum's products meet is free).  WIDE: rows too long for 32-bit offsets, element by element.
template <bool KC, bool WIDE> struct DirectOperand {
    static constexpr int NV = WIDE ? 0 : KC ? 1 : 8;
    int voff[NV > 0 ? NV : 1], ld, K, k0;
    const float* p; long long left; bool ok;
    __device__ __forceinline__ void begin(const float* base, int ld_, int r0, int limit, int row_off, int src_rows, int K_, int lane) {
        ld = ld_; K = K_; k0 = 8 * (lane >> 5);
        if (WIDE) {
            const int r = r0 + (lane & 31);
            ok = r < limit && (!KC || (r + row_off >= 0 && r + row_off < src_rows));
            p = base + (KC ? (long long)(ok ? r + row_off : 0) * ld : (ok ? r : 0));
        } else if (KC) {
            const int first = min(max(r0 + row_off, 0), src_rows - 1), row = r0 + (lane & 31) + row_off;
            p = base + (long long)first * ld; left = (long long)(src_rows - first) * ld;
            voff[0] = row >= 0 && row < src_rows ? ((row - first) * ld + k0) * 4 : OUTSIDE;
        } else {
            p = base + r0; left = (long long)K * ld - r0;
#pragma unroll
            for (int k = 0; k < NV; ++k) voff[k] = ((k0 + k) * ld + (lane & 31)) * 4;
        }
    }
    __device__ __forceinline__ void load(uintx4 (&r)[2], int c) const {
        if (WIDE) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const long long kk = (long long)c * BK + k0 + k;
                r[k >> 2][k & 3] = ok && kk < K ? __float_as_uint(p[KC ? kk : kk * ld]) : 0u;
            }
            return;
        }
        const long long at = (long long)c * BK * (KC ? 1 : ld);
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(p) + at, 0, rsrc_bytes(left - at), RSRC_FLAGS);
        if (KC) {
#pragma unroll
            for (int j = 0; j < 2; ++j) r[j] = __builtin_amdgcn_raw_buffer_load_b128(rs, voff[0] + 16 * j, 0, 0);
            const int k_left = K - c * BK - k0;
            if (K - c * BK < BK) {
#pragma unroll
                for (int e = 0; e < 8; ++e) r[e >> 2][e & 3] = e < k_left ? r[e >> 2][e & 3] : 0u;
            }
        } else {
#pragma unroll
            for (int k = 0; k < NV; ++k) r[k >> 2][k & 3] = __builtin_amdgcn_raw_buffer_load_b32(rs, voff[k], 0, 0);
        }
    }
};

template <bool A_KC, bool B_KC, bool WIDE>
__global__ __launch_bounds__(64 * SMALL_WAVES, 4) void gemm_small_kernel(const GemmGroup g) {
    __shared__ float part[SMALL_WAVES][16 * 64];
    const int b = blockIdx.y * SMALL_GRID_X + blockIdx.x;
    if (b >= g.n_blocks) return;
    const int pi = problem_of(g, b);
    const GemmProblem& P = g.p[pi];
    const int tiles_m = (P.M + SMALL_TILE - 1) / SMALL_TILE, tiles_n = (P.N + SMALL_TILE - 1) / SMALL_TILE, n_tiles = tiles_m * tiles_n;
    int tile = b - g.first_block[pi], split = 0;
    if (P.split > 1) { split = tile / n_tiles; tile -= split * n_tiles; }
    const int tn = tile / tiles_m, m0 = (tile - tn * tiles_m) * SMALL_TILE, n0 = tn * SMALL_TILE;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    floatx16 sum;
#pragma unroll
    for (int e = 0; e < 16; ++e) sum[e] = 0.0f;
    for (int p = P.first_pair; p < P.first_pair + P.n_pairs; ++p) {
        const GemmPair& pr = g.pair[p];
        int c_begin = 0, c_end = chunks_of(pr.K);
        if (P.split > 1) chunk_range(c_end, split, P.split, c_begin, c_end);
        DirectOperand<A_KC, WIDE> oa; DirectOperand<B_KC, WIDE> ob;
        oa.begin(pr.A, pr.lda, m0, P.M, pr.a_row_off, pr.a_rows, pr.K, lane);
        ob.begin(pr.B, pr.ldb, n0, P.N, 0, P.N, pr.K, lane);
        for (int c0 = c_begin + wave; c0 < c_end; c0 += SMALL_WAVES * SMALL_DEPTH) {
            uintx4 ra[SMALL_DEPTH][2], rb[SMALL_DEPTH][2];
#pragma unroll
            for (int d = 0; d < SMALL_DEPTH; ++d)
                if (c0 + SMALL_WAVES * d < c_end) { oa.load(ra[d], c0 + SMALL_WAVES * d); ob.load(rb[d], c0 + SMALL_WAVES * d); }
            floatx16 acc;      // of 64 columns: a sum of such sums rounds less than one long chain
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll
            for (int d = 0; d < SMALL_DEPTH; ++d)
                if (c0 + SMALL_WAVES * d < c_end) {
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        acc = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(ra[d][e >> 2][e & 3]), __uint_as_float(rb[d][e >> 2][e & 3]), acc, 0, 0, 0);
                }
            sum += acc;
        }
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) part[wave][e * 64 + lane] = sum[e];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 16 / SMALL_WAVES; ++j) {
        const int e = wave + SMALL_WAVES * j;
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < SMALL_WAVES; ++w) s += part[w][e * 64 + lane];
        const int row = m0 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3), col = n0 + (lane & 31);
        if (row < P.M && col < P.N) {
            float* dst = P.C + (size_t)row * P.ldc + col;
            if (P.split > 1 || P.accumulate) unsafeAtomicAdd(dst, s);
            else *dst = finish(s, P.bias != nullptr, P.bias != nullptr ? P.bias[col] : 0.0f, P.act);
        }
    }
}

constexpr int TILE_OF[4] = {SMALL_TILE, 64, 128, SMALL_TILE};      // by GemmProblem::kind

int64_t tiles_of(const GemmProblem& p, int kind) {
    const int64_t b = TILE_OF[kind];
    return ((p.M + b - 1) / b) * ((p.N + b - 1) / b);
}
// (tiles of 32 have short sums by themselves)
int split_of(const GemmProblem& p, int kind, int factor, bool one_writer) {
    if (one_writer) return 1;
    const int s = std::min(factor, std::max(1, p.chunks / 8));
    return kind == 0 || kind == 3 ? s : std::max(p.min_split, s);
}
// Estimated time (us) of the problems with mask bit 0 / 1 (narrow ones / the others) in one launch.  A workgroup takes its compute
// unit for a start (and, of a split contraction, as long again for its atomics) and a time per chunk, and its own chain is no shorter
// than `alone` us per chunk.  Measured / estimated, us:
//   tiles of 128: NT 4 x 8192 x 1024 x 1024 494 / 496, 2048 x 20,000 x 512 316 / 331, 2048 x 1024 x 1024 77 / 81; TN 12 x 512 x 512, K = 8192 in 8 parts
//     385 / 396, 12 x 250 x 250, K = 3000 in 8 / 24 parts 67 / 62, 89 / 79
//   tiles of 64: 566 / 643, 364 / 514, 47 / 43; 409 / 425, 53 / 59, 88 / 92
//   tiles of 32: 1021 / 1088, 709 / 732, 74 / 71; in one part 489 / 535, 56 / 53
// (Tiles of 64 for 2048 x 20,000 x 512 are 41 % off; the kind with the least estimate is the fastest one but for 12 x 250 x 250, where 32 takes 3 us
// more than 64.)
double estimate(GemmMode mode, const GemmGroup& g, int mask, int kind, int factor, bool one_writer) {
    static const double start[3] = {0.8, 0.8, 4.0}, alone[3] = {0.04, 0.41, 1.15};
    const double each[3] = {mode == GEMM_TN ? 0.085 : 0.12, 0.30, 0.90};
    double work = 0.0, chain = 0.0, blocks = 0.0;
    for (int i = 0; i < g.n_problems; ++i) {
        const GemmProblem& p = g.p[i];
        if (p.kind == 3 || !((mask >> (p.narrow ? 0 : 1)) & 1)) continue;
        const int s = split_of(p, kind, factor, one_writer);
        const double n = (double)tiles_of(p, kind) * s, c = (double)((p.chunks + s - 1) / s);
        blocks += n;
        work += n * (start[kind] * (s > 1 ? 2.0 : 1.0) + each[kind] * c);
        chain = std::max(chain, start[kind] + alone[kind] * c);
    }
    if (blocks == 0.0) return 0.0;
    const double rounds = blocks / 256.0;
    return 3.0 + std::max(chain, work / 256.0 * ((double)(int64_t)(rounds + 0.999) / rounds));
}

}  // namespace

void plan_gemm_group(GemmMode mode, GemmGroup& g, bool one_writer) {
    bool pieces = false;
    for (int i = 0; i < g.n_problems; ++i) {
        GemmProblem& p = g.p[i];
        p.chunks = 0;
        int ld = p.ldc;
        for (int q = p.first_pair; q < p.first_pair + p.n_pairs; ++q) {
            const int c = g.pair[q].K / BK + (g.pair[q].K % BK != 0);
            p.chunks = (int)std::min<int64_t>((int64_t)p.chunks + c, 1 << 30);
            ld = std::max(ld, std::max(g.pair[q].lda, g.pair[q].ldb));
        }
        // Not quite one tile of the largest kind across.  Counted as narrow up to 63 / 95 / 128 / 191 rows or columns, us of the gradient products: 100
        // outputs of 1,024 units, 4,096 frames 133 / 132 / 132 / 131, 128 outputs, 8,192 frames 212 / 212 / 196 / 196, but three gated layers
        // of 1,024 on 128 inputs, 8,192 frames 3,315 / 3,315 / 3,380, and 160 outputs 111 / 111 / 111 / 126.
        p.narrow = std::min(p.window_M, p.N) < 96;
        p.kind = ld >= GEMM_WIDE_ROW ? 3 : 0;
        pieces = pieces || p.M != p.window_M;
    }
    // Weight gradients are added to zeros that the caller has stored; other products are split only where they have to be, since the
    // order in which the parts are added changes from run to run.  (Three products of 512 x 512, 8,192 frames in up to 1 / 4 / 8 / 64 / 256 parts 143 /
    // 133 / 130 / 130 / 130 us; with fewer frames or units alike from 1 on: what they cannot do without, min_split, makes enough workgroups.)
    int most = mode == GEMM_TN ? 64 : 1;
    for (int i = 0; i < g.n_problems; ++i) most = std::max(most, g.p[i].min_split);
    // every problem in tiles of one size, or the narrow ones in smaller tiles and a launch of their own; kinds lo[m] .. hi[m] for
    // the narrow ones (m = 0) and the others
    int lo[2] = {0, 0}, hi[2] = {2, 2}, kind[2] = {0, 0}, factor[2] = {1, 1};
    auto choose = [&]() {
        auto cheapest = [&](int mask, int k, int& f) {
            double t = 1e30;
            for (int s = 1; s <= (one_writer ? 1 : most); s *= 2) {
                const double e = estimate(mode, g, mask, k, s, one_writer);
                if (e < t) { t = e; f = s; }
            }
            return t;
        };
        double best = 1e30, part[2][3];
        int part_factor[2][3];
        for (int k = 0; k < 3; ++k) {
            int f = 1;
            const double t = cheapest(3, k, f);
            if (t < best && k >= lo[0] && k >= lo[1] && k <= hi[0] && k <= hi[1]) { best = t; kind[0] = kind[1] = k; factor[0] = factor[1] = f; }
            for (int m = 0; m < 2; ++m) part[m][k] = cheapest(1 << m, k, part_factor[m][k]);
        }
        for (int a = lo[0]; a <= hi[0]; ++a)
            for (int b = std::max(a + 1, lo[1]); b <= hi[1]; ++b)
                if (part[0][a] > 0.0 && part[1][b] > 0.0 && part[0][a] + part[1][b] < best) {
                    best = part[0][a] + part[1][b];
                    kind[0] = a; kind[1] = b; factor[0] = part_factor[0][a]; factor[1] = part_factor[1][b];
                }
    };
    if (pieces) {
        // Tiles of 32 add in another order than those of 64 and 128 (which add alike): the whole window's rows say which of
        // the two a problem takes, so that a frame's result does not depend on how many frames share a call.
        int rows[GEMM_MAX_PROBLEMS];
        for (int i = 0; i < g.n_problems; ++i) { rows[i] = g.p[i].M; g.p[i].M = g.p[i].window_M; }
        choose();
        for (int i = 0; i < g.n_problems; ++i) g.p[i].M = rows[i];
        for (int m = 0; m < 2; ++m) { lo[m] = kind[m] == 0 ? 0 : 1; hi[m] = kind[m] == 0 ? 0 : 2; }
    }
    choose();
    for (int i = 0; i < g.n_problems; ++i) {
        GemmProblem& p = g.p[i];
        const int m = p.narrow ? 0 : 1;
        if (p.kind != 3) p.kind = kind[m];
        p.split = split_of(p, p.kind, factor[m], one_writer);
    }
}

hipError_t launch_gemm_group(GemmMode mode, const GemmGroup& g, hipStream_t stream) {
    static const int group_m = [] { const char* env = std::getenv("RNNG_GEMM_GROUP_M"); return env ? std::atoi(env) : 8; }();
    for (int kind = 3; kind >= 0; --kind) {
        GemmGroup l;
        l.n_problems = 0;
        int order[GEMM_MAX_PROBLEMS];      // the longest contractions start first
        for (int i = 0; i < g.n_problems; ++i) {
            if (g.p[i].kind != kind || g.p[i].M <= 0 || g.p[i].N <= 0) continue;
            int at = l.n_problems++;
            for (; at > 0 && g.p[order[at - 1]].chunks / g.p[order[at - 1]].split < g.p[i].chunks / g.p[i].split; --at) order[at] = order[at - 1];
            order[at] = i;
        }
        int64_t blocks = 0;
        int pairs = 0;
        for (int j = 0; j < l.n_problems; ++j) {
            GemmProblem& p = l.p[j] = g.p[order[j]];
            l.first_block[j] = (int)std::min<int64_t>(blocks, INT32_MAX);
            for (int q = 0; q < p.n_pairs; ++q) l.pair[pairs + q] = g.pair[p.first_pair + q];
            p.first_pair = pairs; pairs += p.n_pairs;
            blocks += tiles_of(p, kind) * p.split;
            if (kind == 1 || kind == 2) blocks = (blocks + 7) / 8 * 8;
        }
        if (blocks == 0) continue;
        if (blocks >= (int64_t(1) << 31)) return hipErrorInvalidConfiguration;
        l.n_blocks = (int)blocks; l.group_m = group_m < 0 ? 0 : group_m;
        const dim3 grid((unsigned)blocks), block(NTHREADS);
        const dim3 sgrid((unsigned)std::min<int64_t>(blocks, SMALL_GRID_X), (unsigned)((blocks + SMALL_GRID_X - 1) / SMALL_GRID_X)), sblock(64 * SMALL_WAVES);
#define RNNG_GEMM_LAUNCH(A_KC, B_KC)                                                                                        \
        if (kind == 2) hipLaunchKernelGGL((gemm_kernel<A_KC, B_KC, 2>), grid, block, 0, stream, l);                         \
        else if (kind == 1) hipLaunchKernelGGL((gemm_kernel<A_KC, B_KC, 1>), grid, block, 0, stream, l);                    \
        else if (kind == 0) hipLaunchKernelGGL((gemm_small_kernel<A_KC, B_KC, false>), sgrid, sblock, 0, stream, l);          \
        else hipLaunchKernelGGL((gemm_small_kernel<A_KC, B_KC, true>), sgrid, sblock, 0, stream, l);
        switch (mode) {
            case GEMM_NT: RNNG_GEMM_LAUNCH(true, true) break;
            case GEMM_NN: RNNG_GEMM_LAUNCH(true, false) break;
            case GEMM_TN: RNNG_GEMM_LAUNCH(false, false) break;
        }
#undef RNNG_GEMM_LAUNCH
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace rnng
