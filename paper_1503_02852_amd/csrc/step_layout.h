// LDS layout of the persistent recurrent-step kernel, computed identically on the host (to
// size the launch and to decide whether a component fits) and on the device.
//
// A component's step descriptor is [n_phases, (mv_off, prog_off) x n_phases] in the plan words.
// G workgroups each own a contiguous chunk of every layer's units.  Per phase, the
// matrix-vector work of a workgroup is a set of output slots, slot = task * cmax + local unit,
// each served by L consecutive lanes that split the contraction; a lane's weights are stored
// lane-major ([edge][j][thread][4 floats]) so every ds_read_b128 of a wavefront is contiguous.
#pragma once
#if !defined(__HIPCC_RTC__)
#include <cstdint>
#endif

#include "program.h"

#if defined(__HIPCC__) || defined(__HIPCC_RTC__)
#define RNNG_HD __host__ __device__
#else
#define RNNG_HD
#endif

namespace rnng {

constexpr int STEP_THREADS = 256;
constexpr unsigned STEP_LDS_LIMIT = 148 * 1024;   // dynamic LDS per workgroup (the static tables take 11.3 KiB of the 160 KiB)
constexpr unsigned MSTEP_LDS_LIMIT = 152 * 1024;  // the same for the matrix-core variant with weights in LDS (tables of 6.4 KiB)
constexpr int STEP_MAX_PHASES = 4;
constexpr int STEP_MAX_TASKS = 8;      // per phase
constexpr int STEP_MAX_EDGES = 8;      // per task
constexpr int STEP_MAX_SOURCES = 8;    // distinct (buffer, frame offset) vectors read per step
constexpr int STEP_PF_MAX_STEPS = 16;  // steps per block of early-loaded static gather values
constexpr int STEP_PF_PAIRS_PER_THREAD = 2;
constexpr int STEP_MAX_GATHERS = 24;   // per program (loads are issued from an unrolled loop)

// A tile-blocked twin (see plan.h) holds its units in quads: twin_pad(dim) per stream.  A frame of N streams
// is one block of 16 streams after the other, the last one with the rows that are left, so padding a
// row costs at most three units and padding the streams nothing.
RNNG_HD inline int twin_pad(int v) { return (v + 3) & ~3; }
// Floats from a frame's start to (stream n, unit i).
RNNG_HD inline int twin_offset(int N, int dim, int n, int i) {
    const int first = n & ~15, rows = N - first < 16 ? N - first : 16;
    return first * twin_pad(dim) + (i >> 2) * 4 * rows + (n - first) * 4 + (i & 3);
}

RNNG_HD inline int step_pow2_floor(int v) { int p = 1; while (p * 2 <= v) p *= 2; return p; }

struct StepEdge { int w_off, k_len, transposed, src; };    // src = index into StepLayout::src
struct StepTask { int n_out, chunk, n_edges; StepEdge e[STEP_MAX_EDGES]; };
struct StepPhase {
    int mv_off, prog_off;
    int n_tasks, cmax, n_slots, L;       // L lanes per slot (power of two), n_slots * L <= 256
    int n_e_max;                         // max edges per task
    int J[STEP_MAX_EDGES];               // float4 iterations per lane for edge index e (max over tasks)
    int w_base[STEP_MAX_EDGES];          // float offset of the weight region of edge index e
    int acc_base;                        // float offset of the accumulators [slot][NB]
    int item_chunk;                      // element-wise items: local unit = tid % item_chunk, stream = tid / item_chunk
    int n_static, pf_steps, pf_base;     // ring of early-loaded STATIC gather values: [2][pf_steps][n_static * items]
    StepTask task[STEP_MAX_TASKS];
};
struct StepSource { int buf, frame_off, k_len, k_pad, x_base, first_phase; };
struct StepLayout {
    int ok;                 // 0: does not fit the kernel's limits (reason in `why`)
    int why;
    int n_phases, n_sources, total_floats;
    StepPhase ph[STEP_MAX_PHASES];
    StepSource src[STEP_MAX_SOURCES];
};

// A single-phase component's layout as the plan tables carry it: StepLayout up to its first phase, then the sources.
constexpr int STEP_LAYOUT_HEAD = 5 + (int)(sizeof(StepPhase) / 4), STEP_LAYOUT_WORDS = STEP_LAYOUT_HEAD + (int)(sizeof(StepSource) * STEP_MAX_SOURCES / 4);

constexpr int STEP_MAX_GROUPS = 4;

// Control words behind ctrl that hold the XCDs of one launch each (behind those of the step trace).
constexpr int XCD_WORDS_FIRST = 192, XCD_WORDS = 60;
// Matrix-core launches whose stream groups each sit on one XCD: control words in which the groups' workgroups find out whether they do, in front
// of those.  A field of 32 / xcd_fields(G) bits a group of G <= 32 workgroups: which XCDs (8 bits), how many workgroups have said so.
constexpr int XCD_FIELD_WORDS_FIRST = 144, XCD_FIELD_WORDS = 48, MSTEP_LOCAL_MAX_UNITS = 120;
RNNG_HD constexpr int xcd_fields(int G) { return G <= 3 ? 3 : 2; }
RNNG_HD constexpr int xcd_field_words(int G, int units) { return (units + xcd_fields(G) - 1) / xcd_fields(G); }
static_assert(XCD_FIELD_WORDS_FIRST + XCD_FIELD_WORDS <= XCD_WORDS_FIRST, "control words");
static_assert(xcd_field_words(3, MSTEP_LOCAL_MAX_UNITS) <= XCD_FIELD_WORDS && xcd_field_words(4, 8 * (32 / 4)) <= XCD_FIELD_WORDS, "a launch's fields");
RNNG_HD inline bool xcd_word_split(unsigned w) {      // has a group been on more than one XCD?
    bool split = false;
    for (int g = 0; g < STEP_MAX_GROUPS; ++g) { const unsigned b = (w >> (8 * g)) & 0xFF; split = split || (b & (b - 1)) != 0; }
    return split;
}

struct StepArgs {
    float* const* buf_ptr;                   // buffer table (read-only for the kernel's lifetime)
    const int32_t* words;                    // plan words (likewise)
    const float* weights;
    unsigned* ctrl;                          // [0]: set to 1 when a wait ran into the spin limit
    int desc_off, T, N, backward, G, xcd_stride, spin_limit;
    const int32_t* lay;                      // the component's layout (STEP_LAYOUT_WORDS words), or NULL: the kernel works it out
    int table_bytes;                         // of the plan tables from buf_ptr on
    // Chain launches (several recurrent components side by side): group g runs descriptor
    // grp_desc_off[g] on grp_G[g] workgroups; block b belongs to group b % 8, part b / 8, which
    // puts each group on one XCD.  n_groups == 0: a single component (desc_off, G, xcd_stride).
    int n_groups, grp_desc_off[STEP_MAX_GROUPS], grp_G[STEP_MAX_GROUPS];
    const int32_t* grp_lay[STEP_MAX_GROUPS];
    // Chains of the matrix-core build: group g takes the blocks [grp_first[g], grp_first[g] +
    // grp_G[g] * grp_J[g]) (all groups use all XCDs).
    int grp_J[STEP_MAX_GROUPS], grp_first[STEP_MAX_GROUPS];
    // Frames [t_begin, t_end) are computed (forward: ascending, backward: descending); frames of
    // the window outside this range hold the results of earlier calls (T is the whole window).
    int t_begin, t_end;
    // Matrix-core build: the streams are split into J groups of N / J; workgroup w owns unit chunk
    // w % G of stream group w / G (G * J workgroups in all).  1 elsewhere.
    int J;
    // Matrix-core build with its stream groups on one XCD each: the first of the launch's field words (zero before it), or -1: everything is
    // written through.
    // Wave-autonomous builds: word (behind ctrl) in which this launch's workgroups leave the XCDs they run
    // on, bit 8 g + id for group g, or -1.  With a word, tensors exchanged inside a group are written
    // with plain stores (the XCD's L2 holds them, and the group's polling loads are served there), and
    // the host reports a group on more than one XCD.  With -1 every exchanged tensor is written through.
    int xcd_word;
    // Matrix-core build with the two-dimensional split: the partial sums that the workgroups hand
    // to each other, [frame][workgroup][column slice][row][stream] (sentinel-filled by the host).
    float* partial;
    // Wave-autonomous build compiled for one store window (MV::SW): the window that holds every
    // tensor the kernel stores (the workspace; at most 2 GiB).
    float* store_base;
    unsigned store_bytes;
    // Streaming build: a copy of the parameter buffer in which the matrices that the kernel reads
    // transposed are stored transposed (same offsets), and the size of both buffers in bytes.
    const float* weights_t;
    unsigned weight_bytes;
    // Matrix-core build with tile-blocked exchange: buffer twin_base + b is the blocked twin of
    // the exchanged tensor b (see the kernel).
    int twin_base;
};

RNNG_HD inline int step_count(const StepArgs& a) { return a.t_end - a.t_begin; }
RNNG_HD inline int step_frame(const StepArgs& a, int st) { return a.backward ? a.t_end - 1 - st : a.t_begin + st; }


// words: plan words; desc_off: step descriptor; G workgroups; NB streams per pass; N streams.
RNNG_HD inline void compute_step_layout(const int32_t* words, int desc_off, int G, int NB, int N, StepLayout& out) {
    out.ok = 0; out.why = 0; out.n_sources = 0; out.total_floats = 0;
    const int32_t* d = words + desc_off;
    out.n_phases = d[0];
    if (out.n_phases > STEP_MAX_PHASES) { out.why = 1; return; }
    int cur = 0;
    for (int p = 0; p < out.n_phases; ++p) {
        StepPhase& ph = out.ph[p];
        ph.mv_off = d[1 + 2 * p]; ph.prog_off = d[2 + 2 * p];
        ph.n_tasks = 0; ph.cmax = 0; ph.n_slots = 0; ph.L = 1; ph.n_e_max = 0; ph.acc_base = 0;
        for (int e = 0; e < STEP_MAX_EDGES; ++e) { ph.J[e] = 0; ph.w_base[e] = 0; }
        const int32_t* pg = words + ph.prog_off;
        if (pg[PG_NGATHER] > STEP_MAX_GATHERS) { out.why = 2; return; }
        ph.item_chunk = (pg[PG_MAXDIM] + G - 1) / G;
        if (ph.item_chunk * N > STEP_THREADS) { out.why = 3; return; }
        ph.n_static = 0; ph.pf_steps = 0; ph.pf_base = 0;
        for (int g = 0; g < pg[PG_NGATHER]; ++g)
            if (pg[PG_HEADER_WORDS + g * GA_WORDS + GA_KIND] == GA_KIND_STATIC) ++ph.n_static;
        {
            const int pairs = ph.n_static * ph.item_chunk * N;
            if (pairs > 0 && pairs <= STEP_PF_PAIRS_PER_THREAD * STEP_THREADS) {
                int st = step_pow2_floor(4096 / pairs);
                ph.pf_steps = st < 2 ? 2 : st > STEP_PF_MAX_STEPS ? STEP_PF_MAX_STEPS : st;
                ph.pf_base = cur; cur += 2 * ph.pf_steps * pairs;
                cur = (cur + 3) / 4 * 4;
            }
        }
        if (ph.mv_off < 0) continue;
        const int32_t* w = words + ph.mv_off;
        ph.n_tasks = w[0];
        if (ph.n_tasks > STEP_MAX_TASKS) { out.why = 4; return; }
        ++w;
        for (int t = 0; t < ph.n_tasks; ++t) {
            StepTask& tk = ph.task[t];
            tk.n_out = w[MV_NOUT]; tk.n_edges = w[MV_NEDGES]; tk.chunk = (tk.n_out + G - 1) / G;
            if (tk.n_edges > STEP_MAX_EDGES) { out.why = 5; return; }
            if (tk.chunk > ph.cmax) ph.cmax = tk.chunk;
            if (tk.n_edges > ph.n_e_max) ph.n_e_max = tk.n_edges;
            for (int e = 0; e < tk.n_edges; ++e) {
                const int32_t* ed = w + MV_HEADER_WORDS + e * MVE_WORDS;
                tk.e[e].w_off = ed[MVE_W_OFF]; tk.e[e].k_len = ed[MVE_KLEN]; tk.e[e].transposed = ed[MVE_TRANSPOSED];
                int s = 0;
                for (; s < out.n_sources; ++s)
                    if (out.src[s].buf == ed[MVE_SRC_BUF] && out.src[s].frame_off == ed[MVE_FRAME_OFF]) break;
                if (s == out.n_sources) {
                    if (s == STEP_MAX_SOURCES) { out.why = 6; return; }
                    out.src[s].buf = ed[MVE_SRC_BUF]; out.src[s].frame_off = ed[MVE_FRAME_OFF];
                    out.src[s].k_len = ed[MVE_KLEN]; out.src[s].k_pad = (ed[MVE_KLEN] + 255) / 256 * 256;
                    out.src[s].first_phase = p; out.src[s].x_base = 0;
                    ++out.n_sources;
                }
                tk.e[e].src = s;
            }
            w += MV_HEADER_WORDS + tk.n_edges * MVE_WORDS;
        }
        ph.n_slots = ph.n_tasks * ph.cmax;
        if (ph.n_slots > STEP_THREADS) { out.why = 7; return; }
        ph.L = step_pow2_floor(STEP_THREADS / ph.n_slots);
        if (ph.L > 64) ph.L = 64;
        for (int t = 0; t < ph.n_tasks; ++t)
            for (int e = 0; e < ph.task[t].n_edges; ++e) {
                const int j = (ph.task[t].e[e].k_len + 4 * ph.L - 1) / (4 * ph.L);
                if (j > ph.J[e]) ph.J[e] = j;
            }
        for (int e = 0; e < ph.n_e_max; ++e) { ph.w_base[e] = cur; cur += ph.J[e] * STEP_THREADS * 4; }
        ph.acc_base = cur; cur += ph.n_slots * NB;
        cur = (cur + 3) / 4 * 4;
    }
    for (int s = 0; s < out.n_sources; ++s) { out.src[s].x_base = cur; cur += NB * out.src[s].k_pad; }
    out.total_floats = cur;
    out.ok = 1;
}

}  // namespace rnng
