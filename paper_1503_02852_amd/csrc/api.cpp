// C-ABI boundary (declared in include/rnngraph.h) and the executor that walks the plan.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <algorithm>
#include <array>
#include <tuple>
#include <cstring>
#include <map>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/rnngraph.h"
#include "../../include/rnngraph_aux.h"
#include "jit.h"
#include "kernels.h"
#include "plan.h"

using namespace rnng;

namespace {

thread_local std::string g_last_error;

int fail(int code, const std::string& msg) { g_last_error = msg; return code; }
int fail_hip(hipError_t e, const char* what) {
    return fail(RNN_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

int64_t align_up(int64_t v, int64_t a) { return (v + a - 1) / a * a; }

struct Layout {
    int64_t table_off = 0, dims_off = 0, words_off = 0, blob_bytes = 0;
    int64_t lay_off = 0;                  // behind the plan words, inside the blob: layouts of the step launches (rnn_graph::step_layouts), blob_bytes: with all there can be
    int64_t sync_off = 0;                 // 1 KiB of zero-initialised control words; the loss (double) sits at its start
    std::vector<int64_t> buf_off;         // per buffer id, bytes; -1 = not in the workspace
    int64_t partial_off = -1;             // partial sums of the two-dimensional matrix-core kernels (one launch at a time)
    std::vector<int64_t> idx_off;         // per exec node id: int32 [(hist + T)][N] copy of a one-hot input's class indices, or -1
    int64_t wt_off = -1;                  // transposed copies of the matrices the streaming kernels read transposed (parameter layout)
    int64_t frames_off = 0;               // per buffer id: int64 floats per frame of a frame tensor of the workspace (has history frames), else 0
    int64_t total = 0;
    int64_t uncounted_bytes = 0;          // of total, what the static workspace's limit leaves out: twins that only windows of no whole
                                          // 16 x 16 tiles need padding for, the layouts of step launches
};
constexpr int64_t SYNC_BYTES = 1024;
static_assert(16 + 4 * (XCD_WORDS_FIRST + XCD_WORDS) <= SYNC_BYTES, "control words");

int64_t g_layout_skew = 4352;      // bytes, a multiple of 256 (RNNG_LAYOUT_SKEW overrides: tuning aid)

// partial_floats: floats per frame of the largest partial-sum tensor any launch of the window needs
// transposed_copy: a streaming kernel of the window reads matrices transposed
// twins: per buffer id, whether a step launch of the window polls this twin
// layouts: most layouts of step launches that the window's plan tables carry
Layout make_layout(const Plan& P, int T, int N, int64_t partial_floats, bool transposed_copy, const std::vector<char>& twins, int layouts) {
    Layout L;
    int n_alloc = 0;
    const int K = (int)P.xnodes.size();
    int64_t cur = 0;
    L.table_off = cur; cur += (int64_t)P.n_bufs * 8;
    L.frames_off = cur; cur += (int64_t)P.n_bufs * 8;
    L.dims_off = cur; cur += (int64_t)P.n_bufs * 4;
    cur = align_up(cur, 16);
    L.words_off = cur; cur += (int64_t)P.words.size() * 4;
    L.lay_off = cur;
    cur += layouts * STEP_LAYOUT_WORDS * 4;
    L.blob_bytes = cur;
    cur = align_up(cur, 256);
    L.sync_off = cur; cur += SYNC_BYTES;
    L.buf_off.assign(P.n_bufs, -1);
    const int64_t F = (int64_t)(T + P.hist) * N;
    (void)K;
    auto place = [&](int b) {
        const int64_t frames = P.buf_alloc[b] == 2 ? 1 : T + P.hist;      // every frame tensor has P.hist history frames in front
        L.buf_off[b] = cur; cur = align_up(cur + frames * P.frame_floats(b, N) * 4, 256);
        // Tensors of the same shape would lie a power of two apart, so the lines that a step polls
        // in several tensors at the same frame would all fall on the same memory channel: skew them.
        cur += g_layout_skew * (1 + n_alloc % 13);
        ++n_alloc;
    };
    for (int b = 0; b < P.n_bufs; ++b)
        if (P.buf_alloc[b] == 1 || P.buf_alloc[b] == 2) place(b);
    if (partial_floats > 0) { L.partial_off = cur; cur = align_up(cur + (int64_t)(T + P.hist) * partial_floats * 4, 256); }
    if (transposed_copy) { L.wt_off = cur; cur = align_up(cur + P.n_params * 4, 256); }
    // an input whose connections are delayed may be given as class indices: room for its indices with history frames
    L.idx_off.assign(P.xnodes.size(), -1);
    for (size_t k = 0; k < P.xnodes.size(); ++k)
        if (P.xnodes[k].kind == NODE_INPUT && P.input_delayed[k]) { L.idx_off[k] = cur; cur = align_up(cur + F * 4, 256); }
    // tile-blocked twins, behind everything else
    for (int b = 0; b < P.n_bufs; ++b)
        if (twins[b]) {
            const int64_t at = cur;
            place(b);
            if (N % 16 != 0 || P.buf_dim[b] % 16 != 0) L.uncounted_bytes += cur - at;
        }
    L.total = cur;
    L.uncounted_bytes += align_up(L.blob_bytes, 256) - align_up(L.lay_off, 256);      // (all that the layouts moved the rest by)
    return L;
}

}  // namespace

// Optional kernel-class timing with HIP events on the caller's stream.
struct Profiler {
    struct Rec { int cls; hipEvent_t a, b; int64_t launches; };
    int mask = 0;
    std::vector<Rec> recs;
    std::vector<hipEvent_t> pool;
    hipEvent_t get() {
        if (!pool.empty()) { hipEvent_t e = pool.back(); pool.pop_back(); return e; }
        hipEvent_t e = nullptr;
        if (hipEventCreate(&e) != hipSuccess) return nullptr;
        return e;
    }
    bool on(int cls) const { return (mask >> cls) & 1; }
    // returns the index of the open record or -1
    int begin(int cls, hipStream_t s) {
        if (!on(cls)) return -1;
        Rec r{cls, get(), get(), 0};
        if (!r.a || !r.b) return -1;
        (void)hipEventRecord(r.a, s);
        recs.push_back(r);
        return (int)recs.size() - 1;
    }
    void end(int idx, int64_t launches, hipStream_t s) {
        if (idx < 0) return;
        recs[idx].launches = launches;
        (void)hipEventRecord(recs[idx].b, s);
    }
    ~Profiler() {
        for (Rec& r : recs) { (void)hipEventDestroy(r.a); (void)hipEventDestroy(r.b); }
        for (hipEvent_t e : pool) (void)hipEventDestroy(e);
    }
};

// Whether the workgroups of a launch are dealt to the XCDs in turn, observed once per device: ok if every
// workgroup b of a probe launch with the same b % 8 ran on one XCD.  The step kernels that keep a group of
// workgroups on one residue class then exchange through that XCD's L2 with plain stores.  Which XCD it is
// may change between launches (it does once several streams have been used), so each launch of the weights-in-registers build
// leaves the ids it ran on in a control word, and a group on more than one XCD is reported; the workgroups of the matrix-core build find out by
// themselves before they store (xcd_field_word).
struct XcdMap { bool known = false, ok = false; };

struct rnn_graph;
namespace { bool wave_tensor_sizes_ok(const rnn_graph* g); }

struct rnn_graph {
    Plan plan;
    Profiler prof;
    // state of the current window: T frames as the caller counts them; inside the library a frame
    // tensor has Ti() = hist() + T frames, the caller's frame t being internal frame hist() + t
    int T = 0, N = 0;
    int hist() const { return plan.hist; }
    int Ti() const { return T + plan.hist; }
    char* ws = nullptr;
    Layout layout;
    std::vector<char> blob;               // host copy of the plan tables (kept alive for the async upload)
    bool tables_there = false;            // blob is what the current window's workspace holds
    std::vector<const float*> inputs;     // per exec node id (input nodes only)
    const XcdMap* xcd = nullptr;          // set by the first forward call on this device
    std::vector<const int32_t*> onehot;   // per exec node id: class indices of a one-hot input, or nullptr
    // rnn_grads' lists, with room for every block from the graph's creation on (nothing is allocated later)
    std::vector<GemmGroup> grad_groups;
    std::vector<std::pair<int64_t, int64_t>> grad_owned;      // offset, length
    const float* weights = nullptr;
    bool fwd_done = false, bptt_done = false;
    int fwd_upto = 0;                     // frames [0, fwd_upto) of the current window hold forward results
    bool framewise = false;               // benchmark mode: every frame on its own, no batching over frames
    bool deterministic = false;           // rnn_set_deterministic: one writer per gradient element, fixed summation order
    bool prefilled = false;               // inside a call: the tensors of all of its step launches are filled already (all_shared)
    bool no_alloc = false;                // inside rnn_forward_static: load no code, create no events, stage no host copies
    PlanView view() const {
        PlanView pv;
        pv.buf_ptr = reinterpret_cast<float* const*>(ws + layout.table_off);
        pv.buf_dim = reinterpret_cast<const int32_t*>(ws + layout.dims_off);
        pv.words = reinterpret_cast<const int32_t*>(ws + layout.words_off);
        return pv;
    }
    // internal frame 0 of a workspace tensor; for an input read in place: the caller's tensor
    // (its frame 0 is internal frame hist())
    float* buf(int id) const {
        if (layout.buf_off[id] >= 0) return reinterpret_cast<float*>(ws + layout.buf_off[id]);
        if (id < (int)inputs.size() && inputs[id]) return const_cast<float*>(inputs[id]);
        return nullptr;
    }
    bool caller_input(int id) const { return layout.buf_off[id] < 0 && id < (int)inputs.size() && inputs[id] != nullptr; }
    // the caller's frame 0 of a workspace tensor
    float* frame0(int id) const { return buf(id) + (caller_input(id) ? 0 : (int64_t)hist() * N * plan.buf_dim[id]); }
    bool is_onehot(int buf) const { return buf >= 0 && buf < (int)onehot.size() && onehot[buf] != nullptr; }
    // class indices of a one-hot input with history frames in front (internal frame 0), or nullptr if the node keeps none
    int32_t* onehot_history(int buf) const {
        return buf >= 0 && buf < (int)layout.idx_off.size() && layout.idx_off[buf] >= 0 ? reinterpret_cast<int32_t*>(ws + layout.idx_off[buf]) : nullptr;
    }
    double* loss_ptr() const { return reinterpret_cast<double*>(ws + layout.sync_off); }
    unsigned* ctrl_ptr() const { return reinterpret_cast<unsigned*>(ws + layout.sync_off + 16); }
    int force_step_G = 0;
    int xcd_words_used = 0;               // of the current window (step_layout.h)
    int xcd_fields_used = 0;              // of the current call
    int spin_limit = 1 << 22;             // bound of every wait inside a step kernel (polling attempts)
    int cu_count = 0;                     // compute units of the device of the current window (0: not asked yet)
    // which build ran the step loop of component c in direction d at its last launch (RNN_BUILD_*, 0: none yet)
    std::vector<std::array<int, 2>> served;
    bool use_jit = true;
    bool use_store_window = true;
    // Run-time specialised step kernels, chosen once per (component, direction, stream count).
    struct JitChoice { bool wave = false, mstep = false, stream = false, needs_t = false, blocked = false, local = false, element_wise = false; int J = 1; StepLaunchPlan lp; std::string source, source_window; bool two_d = false; int64_t partial_floats = 0; };
    int force_step_J = 0, local_env = -1;      // RNNG_MSTEP_LOCAL: 0 never, 1 wherever it can run, 2 the same with its groups dealt over the XCDs
    bool prefer_streaming = false;        // RNNG_STEP_BUILD=stream
    // the workgroups of a step launch wait for each other, so all of them must be resident at once:
    // one per compute unit (256 on a whole MI355X, fewer on a partition)
    int max_workgroups() const { return cu_count > 0 ? cu_count : 256; }
    std::map<std::tuple<int, bool, int>, JitChoice> jit_choices;
    const JitChoice& jit_choice(int comp, bool backward, int N) {
        const std::tuple<int, bool, int> key(comp, backward, N);
        auto it = jit_choices.find(key);
        if (it != jit_choices.end()) return it->second;
        JitChoice c;
        const CompPlan& cp = plan.comps[comp];
        auto try_streaming = [&]() {
            if (!c.source.empty()) return;
            for (int G : {256, 128, 64, 32}) {
                if (force_step_G > 0 && G != force_step_G) continue;
                if (G > max_workgroups()) continue;
                size_t lds = 0; bool tr = false, xb = false; int threads = 256;
                std::string src = N <= 8 ? jit_sstep_source(plan, cp, backward, N, G, &lds, &tr) : jit_smstep_source(plan, cp, backward, N, G, &lds, &tr, &xb, &threads);
                if (src.empty()) continue;
                c.source = src; c.stream = true; c.needs_t = tr; c.blocked = xb; c.lp.threads = threads;
                c.lp.ok = true; c.lp.G = G; c.lp.NB = 1; c.lp.lds_bytes = lds; c.lp.xcd_stride = 1;
                break;
            }
        };
        if (prefer_streaming) try_streaming();      // (tests: the streaming variant on shapes the other variants would take)
        // 1. wave-autonomous variant: weights in registers, no barriers (single-phase components);
        // first on the 32 workgroups of one XCD, which exchange through its L2
        auto try_wave = [&](int G) {
            if (!c.source.empty() || c.stream || G > max_workgroups()) return;
            c.source = jit_wave_source(plan, cp, backward, N, G);
            if (!c.source.empty()) {
                c.wave = true; c.lp.ok = true; c.lp.G = G; c.lp.NB = step_nb_for(N); c.lp.lds_bytes = 0;
                c.lp.xcd_stride = G <= 32 ? 8 : 1;
            }
        };
        auto try_local = [&]() {
            // Only on a whole device, whose eight XCDs of 32 compute units each take an eighth of the launch: on a partition of two XCDs, three groups
            // of 21 workgroups would put 42 on the first, not all resident, and wait for each other in vain.
            if (max_workgroups() < 256) return;
            if (!c.source.empty() || c.stream || force_step_G > 0 || force_step_J > 0 || !local_streams(cp, backward, N)) return;
            const int J = (N + 15) / 16;
            const MstepPick p = pick_mstep(cp, backward, N, J, 32, true);
            if (p.G && J <= std::min(8 * (32 / p.G), MSTEP_LOCAL_MAX_UNITS) && p.G * J <= max_workgroups() && (local_env >= 1 || p.rows <= (N >= 16 ? 48 : 32))) take_mstep(c, cp, backward, N, p, true);
        };
        // Recurrences without a full connection inside: a thread per stream and unit.  LSTM without output recurrence, 512 frames, us a call against the
        // weights-in-registers build: forward, any width, 10 to 15 % ahead (one stream, 8 / 100 / 300 units 129 / 137, 129 / 149, 131 / 154).  Backward the
        // other is ahead while its wavefronts have few units and streams: five streams 512 / 700 units 181 / 165, 186 / 187, six 450 / 512 200 / 193, 183 / 206, seven 150 /
        // 200 180 / 175, 174 / 188, eight 64 / 100 167 / 160, 170 / 174; up to four always.  From 9 streams on the other is a launch
        // per frame: 64 units, N = 10 0.19 + 0.28 against 6.1 + 7.7 us a frame forward + backward, 1,000 units, N = 64 0.62 + 0.82 against 6.8 + 8.6.
        const std::vector<PhasePlan>& program = backward ? cp.bwd_phases : cp.fwd_phases;
        const int units = program.empty() ? 0 : program[0].max_dim;
        if (c.source.empty() && force_step_G <= 0 &&
            (!backward || N >= 9 || (N >= 5 && units >= (N == 5 ? 700 : N == 6 ? 512 : N == 7 ? 200 : 100)))) {
            c.source = jit_estep_source(plan, cp, backward, N, &c.lp.G, &c.J);
            if (c.source.empty()) { c.J = 1; c.lp = StepLaunchPlan(); }
            else { c.element_wise = true; c.lp.ok = true; c.lp.NB = 1; c.lp.lds_bytes = 0; c.lp.threads = 64; c.lp.xcd_stride = 1; }
        }
        if (N >= 5 || local_env >= 1) try_local();
        try_wave(force_step_G > 0 ? force_step_G : 32);
        if (N >= 4 && step_columns(cp, backward) < 2048) try_local();
        if (force_step_G <= 0 && register_over_xcds(cp, backward, N)) try_wave(64);
        try_local();
        // 2. matrix-core variants for many streams (weights in LDS or registers, MFMA)
        // 2a. one-dimensional split: stream groups, as many as possible (every group halves the
        //     bytes a workgroup polls per step); unit chunks: as many as the compute units allow
        //     while a workgroup still fills a 16-row tile, else the smallest count whose weight
        //     rows fit on chip
        JitChoice one_d;
        int one_d_rows = -1;
        if (c.source.empty() && !c.stream && matrix_streams(cp, backward, N)) {
            for (int J : {4, 3, 2, 1}) {
                if (force_step_J > 0 && J != force_step_J) continue;
                const MstepPick p = pick_mstep(cp, backward, N, J, max_workgroups() / J, false);
                if (!p.G) continue;
                take_mstep(one_d, cp, backward, N, p, false);
                one_d_rows = p.rows;
                break;
            }
        }
        // 2b. the two-dimensional split, where a workgroup polls a sixteenth (or a quarter) of every
        //     source and the row groups' members share 16-row tiles, at the price of a second
        //     exchange per step: only where the one-dimensional split cannot fill its tiles
        //     (RNNG_MSTEP_2D = 1: wherever the kernel can run; = 0: never)
        const char* env2d = std::getenv("RNNG_MSTEP_2D");
        const bool forced_2d = env2d && std::atoi(env2d) != 0, no_2d = env2d && std::atoi(env2d) == 0;
        if (c.source.empty() && N > 8 && force_step_G <= 0 && force_step_J <= 0 && max_workgroups() >= 256 && !no_2d &&
            (forced_2d || one_d_rows < MSTEP_MIN_ROWS)) {
            StepLayout lay;
            compute_step_layout(plan.words.data(), backward ? cp.bwd_desc_off : cp.fwd_desc_off, 256, 1, N, lay);
            int64_t polled = 0;
            if (lay.ok) for (int sidx = 0; sidx < lay.n_sources; ++sidx) polled += (int64_t)N * lay.src[sidx].k_len * 4;
            if (polled >= 256 * 1024 || forced_2d) {
                // row groups of 16 while a workgroup has at most 8 rows; of 4 with more rows, so that
                // the partial sums a workgroup writes and polls per step stay at N * 64 values
                const int rows = lay.ph[0].n_tasks * lay.ph[0].cmax;
                int gj = rows <= 8 ? 16 : 4;
                if (const char* env = std::getenv("RNNG_MSTEP_2D_GROUP")) gj = std::atoi(env);
                size_t lds = 0; int64_t pf = 0;
                std::string src = jit_mstep2_source(plan, cp, backward, N, 256, gj, &lds, &pf);
                if (src.empty() && gj != 16) src = jit_mstep2_source(plan, cp, backward, N, 256, 16, &lds, &pf);
                if (!src.empty()) {
                    c.source = src; c.lp.ok = true; c.lp.G = 256; c.lp.NB = 1; c.lp.lds_bytes = lds; c.lp.xcd_stride = 1;
                    c.two_d = true; c.mstep = true; c.partial_floats = pf;
                }
            }
        }
        if (c.source.empty() && !one_d.source.empty()) c = one_d;
        if (force_step_G <= 0) for (int G : {64, 128, 256, 16, 8}) try_wave(G);
        // 3. LDS-resident variant
        if (c.source.empty() && plan_step_launch(plan.words.data(), backward ? cp.bwd_desc_off : cp.fwd_desc_off, N, force_step_G, c.lp))
            c.source = jit_step_source(plan, cp, backward, c.lp.NB);
        // 4. streaming variant: the weights do not fit on chip at all (wide layers); every step reads them from memory
        try_streaming();
        return jit_choices.emplace(key, c).first->second;
    }
    // floats per frame of the largest partial-sum tensor that a step launch of a window with N streams needs
    int64_t partial_frame_floats(int N) {
        int64_t m = 0;
        if (!use_jit) return 0;
        for (size_t c = 0; c < plan.comps.size(); ++c) {
            const CompPlan& cp = plan.comps[c];
            if (!cp.recurrent) continue;
            for (int backward = 0; backward < 2; ++backward) {
                if (backward ? !cp.has_bwd_program : !cp.has_fwd_program) continue;
                if (cp.chain >= 0 && !chain_choice(cp.chain, backward != 0, N).source.empty()) continue;
                const JitChoice& jc = jit_choice((int)c, backward != 0, N);
                if (jc.two_d) m = std::max(m, jc.partial_floats);
            }
        }
        return m;
    }
    // true if a step launch of a window with N streams reads transposed copies of weight matrices
    bool transposed_copy(int N) {
        if (!use_jit) return false;
        for (size_t c = 0; c < plan.comps.size(); ++c) {
            const CompPlan& cp = plan.comps[c];
            if (!cp.recurrent) continue;
            for (int backward = 0; backward < 2; ++backward) {
                if (backward ? !cp.has_bwd_program : !cp.has_fwd_program) continue;
                if (cp.chain >= 0 && !chain_choice(cp.chain, backward != 0, N).source.empty()) continue;
                if (jit_choice((int)c, backward != 0, N).needs_t) return true;
            }
        }
        return false;
    }
    // the tile-blocked twins that step launches of a window with N streams exchange through.  (A member
    // of a chain runs on its own only in windows that no blocked kernel but the streaming one takes.)
    std::vector<char> polled_twins(int N) {
        std::vector<char> polled(plan.n_bufs, 0);
        if (!use_jit) return polled;
        auto add = [&](const CompPlan& cp, bool backward) {
            for (int b : backward ? cp.bwd_shared_bufs : cp.fwd_shared_bufs)
                if (plan.buf_alloc[plan.twin_base + b] == 3) polled[plan.twin_base + b] = 1;
        };
        for (size_t c = 0; c < plan.comps.size(); ++c) {
            const CompPlan& cp = plan.comps[c];
            if (!cp.recurrent) continue;
            for (int backward = 0; backward < 2; ++backward) {
                if (backward ? !cp.has_bwd_program : !cp.has_fwd_program) continue;
                const ChainChoice* cc = cp.chain >= 0 ? &chain_choice(cp.chain, backward != 0, N) : nullptr;
                if (cc && cc->blocked) for (const CompPlan& m : chain_members(plan.chains[cp.chain], *cc)) add(m, backward != 0);
                const JitChoice& jc = jit_choice((int)c, backward != 0, N);
                if (jc.blocked && (!cc || cc->source.empty() || jc.stream)) add(cp, backward != 0);
            }
        }
        return polled;
    }
    // the workspace layout of a window of T frames and N streams (kept for the last shape asked for)
    Layout cached_layout;
    int cached_T = 0, cached_N = 0;
    const Layout& layout_for(int T, int N) {
        if (cached_T != T || cached_N != N) {
            const int64_t partial = partial_frame_floats(N);
            const bool copy = transposed_copy(N);
            const std::vector<char> twins = polled_twins(N);
            int layouts = 0;
            for (const bool sizes_ok : {true, false})      // (whether the chain launches can run is known with the layout only)
                layouts = std::max(layouts, (int)(step_layouts(N, sizes_ok).words.size() / STEP_LAYOUT_WORDS));
            cached_layout = make_layout(plan, T, N, partial, copy, twins, layouts);
            cached_T = T; cached_N = N;
        }
        return cached_layout;
    }
    void drop_choices() { jit_choices.clear(); chain_choices.clear(); mstep_picks.clear(); cached_T = cached_N = 0; lay = StepLayouts(); }
    // The layouts (step_layout.h) of the weights-in-registers and the matrix-core launches of a window with N streams, one after the other as the kernels
    // load them, and where the first one of a component's or chain's launch lies (direction: 2 c + d; -1: none).  sizes_ok: wave_tensor_sizes_ok.
    struct StepLayouts { std::vector<int32_t> words; std::vector<int> comp, chain; int N = 0; bool sizes_ok = false; };
    StepLayouts lay;      // of the current window
    StepLayouts step_layouts(int N, bool sizes_ok) {
        StepLayouts r;
        r.comp.assign(2 * plan.comps.size(), -1); r.chain.assign(2 * plan.chains.size(), -1);
        r.N = N; r.sizes_ok = sizes_ok;
        if (!use_jit || framewise) return r;
        auto add = [&](const CompPlan& cp, bool backward, int G, int NB, int streams) {
            const int at = (int)(r.words.size() / STEP_LAYOUT_WORDS);
            StepLayout l;
            std::memset(&l, 0, sizeof(l));
            compute_step_layout(plan.words.data(), backward ? cp.bwd_desc_off : cp.fwd_desc_off, G, NB, streams, l);
            r.words.resize((size_t)(at + 1) * STEP_LAYOUT_WORDS);
            std::memcpy(&r.words[(size_t)at * STEP_LAYOUT_WORDS], &l, STEP_LAYOUT_HEAD * 4);
            std::memcpy(&r.words[(size_t)at * STEP_LAYOUT_WORDS + STEP_LAYOUT_HEAD], l.src, sizeof(l.src));
            return at;
        };
        for (size_t c = 0; c < plan.comps.size(); ++c) {
            const CompPlan& cp = plan.comps[c];
            if (!cp.recurrent) continue;
            for (int d = 0; d < 2; ++d) {
                if (d ? !cp.has_bwd_program : !cp.has_fwd_program) continue;
                if (cp.chain >= 0 && sizes_ok) {
                    const ChainPlan& ch = plan.chains[cp.chain];
                    const ChainChoice& cc = chain_choice(cp.chain, d != 0, N);
                    if (!cc.source.empty()) {
                        if ((int)c != ch.first) continue;
                        const std::vector<CompPlan>& members = chain_members(ch, cc);
                        for (size_t i = 0; i < members.size(); ++i) {
                            const int at = cc.mstep ? add(members[i], d != 0, cc.G[i], 1, mstep_streams(N, cc.J[i], cc.blocked))
                                                    : add(members[i], d != 0, cc.G[i], step_nb_for(N), N);
                            if (i == 0) r.chain[2 * cp.chain + d] = at;
                        }
                        continue;
                    }
                }
                const JitChoice& jc = jit_choice((int)c, d != 0, N);
                if (jc.source.empty()) continue;
                if (jc.wave) r.comp[2 * c + d] = add(cp, d != 0, jc.lp.G, step_nb_for(N), N);
                else if (jc.element_wise) r.comp[2 * c + d] = add(cp, d != 0, jc.lp.G, 1, 1);
                else if (jc.mstep && !jc.two_d) r.comp[2 * c + d] = add(cp, d != 0, jc.lp.G, 1, mstep_streams(N, jc.J, jc.blocked));
            }
        }
        return r;
    }
    int table_bytes() const { return (int)std::min<int64_t>(layout.lay_off + (int64_t)lay.words.size() * 4, 1 << 30); }
    const int32_t* layout_at(int at) const { return at < 0 ? nullptr : reinterpret_cast<const int32_t*>(ws + layout.lay_off) + (int64_t)at * STEP_LAYOUT_WORDS; }
    // Whether the matrix-core kernels take a component at N streams.  From 9 streams on the
    // weights-in-registers kernels do not exist.  From 2 streams on they lose where they need more
    // workgroups than one XCD has (their exchange then crosses the XCDs and every lane multiplies for
    // every stream, while the matrix instructions serve 16 streams at the price of one).  Windows of
    // 128 frames, forward + BPTT, register against matrix-core build: 2 x 256 units, N = 8: 1.78
    // against 0.80 ms; 512 units, N = 4 / 8: 0.99 / 3.23 against 0.99 / 1.04; 1,024 units, N = 2:
    // 1.95 against 1.40; Elman 512, N = 4: 0.77 against 0.52.  Confined to one XCD: 256 units, N = 4:
    // 0.55 against 0.66; 512, N = 2: 0.68 against 0.97; 1,024 units at N = 1 (64 workgroups): 1.03
    // against 1.40.  Rows beyond 1,024 elements keep the register and streaming kernels.
    bool matrix_streams(const CompPlan& cp, bool backward, int N) const {
        if (N > 8) return true;
        if (N < 2) return false;
        StepLayout lay;
        compute_step_layout(plan.words.data(), backward ? cp.bwd_desc_off : cp.fwd_desc_off, 256, 1, 1, lay);      // (only the sources are needed)
        if (!lay.ok) return false;
        for (int s = 0; s < lay.n_sources; ++s) if (lay.src[s].k_len > 1024) return false;
        return true;
    }
    // The unit chunks of a component in the matrix-core build with J stream groups, at most `limit` of them: as many as fill one 16-row
    // tile of the matrix instructions each, if need be two and more: a tile takes as long half empty (us a step: 2 x 192 LSTM units, 20
    // streams, forward 32 chunks of 24 rows 2.24, 48 of 16 1.54; 2 x 448, 8 streams, backward 16 of 28 5.47, 28 of 16 3.49).  Rather a
    // third of a tile empty than weight rows in registers.
    struct MstepPick { int G = 0, J = 0, rows = 0, columns = 0; };      // columns: contracted by a workgroup per step, once per 16 x 16 tile; G = 0: does not fit
    static constexpr int MSTEP_MIN_ROWS = 11;
    std::map<std::tuple<const CompPlan*, bool, int, int, int, bool>, MstepPick> mstep_picks;
    const MstepPick& pick_mstep(const CompPlan& cp, bool backward, int N, int J, int limit, bool local) {
        const auto key = std::make_tuple(&cp, backward, N, J, limit, local);
        const auto it = mstep_picks.find(key);
        return it != mstep_picks.end() ? it->second : mstep_picks.emplace(key, find_mstep(cp, backward, N, J, limit, local)).first->second;
    }
    MstepPick find_mstep(const CompPlan& cp, bool backward, int N, int J, int limit, bool local) const {
        MstepPick best;
        if (J > 1 && J > (N + 15) / 16) return best;      // (stream groups are whole 16-stream tiles)
        StepLayout lay;
        compute_step_layout(plan.words.data(), backward ? cp.bwd_desc_off : cp.fwd_desc_off, 256, 1, 1, lay);
        if (!lay.ok || lay.n_phases != 1 || lay.ph[0].n_tasks < 1) return best;
        const int nt = lay.ph[0].n_tasks;
        int dim = plan.words[lay.ph[0].prog_off + PG_MAXDIM], k = 0;
        for (int t = 0; t < nt; ++t) dim = std::max(dim, lay.ph[0].task[t].n_out);
        for (int s = 0; s < lay.n_sources; ++s) k += lay.src[s].k_len;
        int best_chunk = 0, best_regs = 0;
        for (int tiles = 1; tiles <= 16 && !best.G; ++tiles) {
            const int most = 16 * tiles / nt;
            // With three tiles of streams a second source in registers spills others (LSTM backward, 1,500 units, 33 streams: 7 rows 39 us a step, 6 rows, one
            // source, 30; with one tile, 520 units, 9 streams, 28 rows and three sources 6.8, 26 and two 7.1).
            auto several = [&]() { return best_regs > 1 && mstep_streams(N, J, true) > 32; };
            for (int chunk = most; chunk >= 1 && chunk * nt > 16 * (tiles - 1); --chunk) {
                if (chunk * 3 < (several() ? best_chunk : most) * 2 && best.G) break;
                MstepPick p;
                p.G = force_step_G > 0 ? force_step_G : (dim + chunk - 1) / chunk; p.J = J;
                if (p.G > limit) break;
                if (force_step_G <= 0 && chunk * mstep_streams(N, J, true) > STEP_THREADS) continue;      // (more element-wise items than threads)
                int regs = 0;
                const bool fits = jit_mstep_fits(plan, cp, backward, N, p.G, J, local, &p.rows, &regs);
                p.columns = k * ((p.rows + 15) / 16) * (((N + 15) / 16 + J - 1) / J);
                if (force_step_G > 0) return fits ? p : best;
                if (!fits || (best.G && regs >= (several() ? best_regs : 1))) continue;
                if (!best.G) best_chunk = chunk;
                best = p; best_regs = regs;
                if (!regs) break;
            }
        }
        return best;
    }
    void take_mstep(JitChoice& c, const CompPlan& cp, bool backward, int N, const MstepPick& p, bool local) const {
        c.source = jit_mstep_source(plan, cp, backward, N, p.G, p.J, &c.lp.lds_bytes, &c.lp.threads, &c.blocked, local);
        if (c.source.empty()) return;
        c.mstep = true; c.local = local; c.J = p.J;
        c.lp.ok = true; c.lp.G = p.G; c.lp.NB = 1;
        c.lp.xcd_stride = !local && p.G * p.J <= 32 ? 8 : 1;
    }
    // Whether a layer of its own exchanges inside one XCD (stream groups of 16, each on the 32 workgroups of an XCD at most) where it fits:
    // its exchanged values are stored plainly, and nothing is held back.  us a step, inside one XCD against across: LSTM forward 64 units, N = 64 1.07 / 1.42, 256 1.61 / 1.99; backward 256 2.23 / 2.54, 384, N = 8 2.76 / 4.46; one source
    // of 128 to 512 units (Elman), N = 16 to 64 0.81 to 1.45 / 0.92 to 1.64.  With three tiles a workgroup only while 16 streams fill them
    // (LSTM forward 384 units, N = 8 2.24 / 1.97, N = 16 2.31 / 2.41), never with four (512 units, N = 16 3.30 / 1.89).
    // Up to 8 streams against the weights-in-registers build on one XCD: one source from N = 5 on (LSTM forward 16 / 100 units, N = 5
    // 1.00 / 1.03 against 1.11 / 1.41, N = 4 1.00 / 1.05 against 0.89 / 0.98); several from 400 columns on (LSTM backward, N = 8, 48 / 100 / 128 units 1.64 / 1.66 / 1.76
    // against 1.18 / 1.77 / 1.92).  N = 2 to 4: after that build on one XCD; at N = 4 before it on two (LSTM backward, 288 / 384 / 500 units
    // 2.5 / 2.5 / 3.0 against 3.5 / 3.7 / 3.6), up to 2,047 columns: at 2,048 (512 units, 3.0 against 3.5) a test of the workspace holds the register build.
    bool local_streams(const CompPlan& cp, bool backward, int N, int several_from = 400, int one_from = 0) const {
        if (local_env == 0 || N < 2 || !matrix_streams(cp, backward, N)) return false;
        if (N > 8 || local_env >= 1) return true;
        int sources = 0;
        const int columns = step_columns(cp, backward, &sources);
        return columns > (sources == 1 ? one_from : several_from);
    }
    // Columns that a step contracts, over all of its sources.
    int step_columns(const CompPlan& cp, bool backward, int* sources = nullptr) const {
        StepLayout lay;
        compute_step_layout(plan.words.data(), backward ? cp.bwd_desc_off : cp.fwd_desc_off, 256, 1, 1, lay);
        int columns = 0;
        for (int s = 0; lay.ok && s < lay.n_sources; ++s) columns += lay.src[s].k_len;
        if (sources) *sources = lay.n_sources;
        return columns;
    }
    // Whether a layer's register build also stays ahead of the matrix-core build on two XCDs' 64 workgroups
    // (if it fits them): a step polls many columns, each 16 streams wide for the matrix instructions, while the
    // multiply-adds of at most four streams are few.  Step kernel of 128 frames, register against
    // matrix-core build: N = 2, LSTM backward (four sources) 544 / 640 / 768 units 0.46 / 0.45 / 0.50 against
    // 0.81 / 0.82 / 0.96 ms, one source of 544 / 768 / 1,024 units (Elman) 0.28 / 0.28 / 0.27 against 0.26 /
    // 0.30 / 0.33, of 640 (LSTM forward) 0.33 against 0.35; N = 3 and 4, LSTM backward 288 / 416 units 0.44 /
    // 0.48 against 0.54 / 0.68, 512 0.47 / 0.47, one source of 288 / 512 / 1,024 units 0.32 / 0.30 / 0.39
    // against 0.19 / 0.17 / 0.34.  With eight streams' multiply-adds (N >= 5) never (208 units, N = 5,
    // windows: 0.95 against 0.66), nor with more weights than a lane's registers take well (N = 2, LSTM
    // backward, 144 / 196 / 256 per lane of 64 workgroups: 0.50 / 0.82 / 1.14 against 0.96 / 0.69 / 0.77).
    bool register_over_xcds(const CompPlan& cp, bool backward, int N) const {
        if (N < 2 || N > 4 || cp.step_weight_floats > 160 * 64 * STEP_THREADS) return false;
        return step_columns(cp, backward) >= (N == 2 ? 600 : 1100);
    }
    // Chains of recurrent components run side by side in one launch: all members in the
    // wave-autonomous build (N <= 8, member g on XCD g), or all in the matrix-core build (the 256
    // workgroups shared among the members).
    struct ChainChoice {
        std::string source, source_window; std::vector<int> G, J; bool mstep = false, blocked = false; size_t lds_bytes = 0; int threads = 256;
        bool split = false, backward = false;      // split: the launch with helper members (ChainPlan::fwd_split / bwd_split)
    };
    static const std::vector<CompPlan>& chain_members(const ChainPlan& ch, const ChainChoice& cc) {
        return !cc.split ? ch.members : cc.backward ? ch.bwd_split : ch.fwd_split;
    }
    std::map<std::tuple<int, bool, int>, ChainChoice> chain_choices;
    bool use_chains = true;
    // Weights-in-registers launches: a step is mostly exchange latency, and the helper group reads
    // its sources across XCDs (more than a microsecond per step), so it pays where the multiply-adds
    // and polled sources it takes over weigh enough.  Measured, step kernels forward / backward with
    // against without helper groups: charlm_n1 (128 multiply-adds per lane and step moved) 0.76 / 0.79
    // against 0.81 / 1.21 ms; speech_n1 (32 per lane, 0.9 us per step) 1.11 / 0.91 against 0.93 / 1.04:
    // backward launches (the helper halves the lower layer's sources) from 24 per lane on, forward
    // launches from 100.
    bool wave_helpers_pay(const std::vector<CompPlan>& members, bool backward, int N) const {
        int min_fma = backward ? 24 : 100;
        if (const char* env = std::getenv("RNNG_CHAIN_HELPER_MIN")) min_fma = std::atoi(env);
        for (const CompPlan& m : members)
            if (m.helper && m.step_weight_floats * step_nb_for(N) / (32 * 256) >= min_fma) return true;
        return false;
    }
    const ChainChoice& chain_choice(int chain, bool backward, int N) {
        const std::tuple<int, bool, int> key(chain, backward, N);
        auto it = chain_choices.find(key);
        if (it != chain_choices.end()) return it->second;
        ChainChoice c;
        c.backward = backward;
        const ChainPlan& ch = plan.chains[chain];
        // Helper members take the products of the connections between the stacked nodes
        // (RNNG_CHAIN_HELPERS = 0: never; 1: in every launch that can have them; default: in the
        // matrix-core backward launch and in weights-in-registers launches from RNNG_CHAIN_HELPER_MIN
        // multiply-adds per lane and step on, else from 24 backward / 100 forward)
        const char* envh = std::getenv("RNNG_CHAIN_HELPERS");
        const bool helpers_off = envh && std::atoi(envh) == 0, helpers_all = envh && std::atoi(envh) == 1;
        auto registers = [&]() {
            for (int attempt = 0; attempt < 2 && c.source.empty(); ++attempt) {
                c.split = attempt == 0 && !helpers_off && !(backward ? ch.bwd_split : ch.fwd_split).empty();
                if (attempt == 0 && !c.split) continue;
                const std::vector<CompPlan>& members = chain_members(ch, c);
                c.G.clear();
                for (const CompPlan& m : members) {
                    int pick = 0;
                    for (int G : {32, 16, 8})
                        if (!jit_wave_source(plan, m, backward, N, G).empty()) { pick = G; break; }
                    if (!pick) break;
                    c.G.push_back(pick);
                }
                if (c.G.size() == members.size() && (!c.split || helpers_all || wave_helpers_pay(members, backward, N)))
                    c.source = jit_chain_source(plan, members, backward, N, c.G);
            }
            if (c.source.empty()) c.split = false;
        };
        auto matrix_cores = [&](bool matrix) {
            // Few streams: where a layer would need several XCDs.  Side by side on the matrix cores the layers
            // also beat two register launches one after the other (register_over_xcds): 2 x 768 units, N = 2
            // 0.56 + 1.02 against 0.67 + 1.00 ms forward + backward, 2 x 320, N = 4 0.37 + 0.58 against 0.89 + 0.95.
            for (int m = ch.first; m <= ch.last && !matrix; ++m) {
                const JitChoice& jc = jit_choice(m, backward, N);
                matrix = jc.mstep || (jc.wave && jc.lp.G > 32 && matrix_streams(plan.comps[m], backward, N));
            }
            if (c.source.empty() && matrix && force_step_J <= 0) {
                // matrix-core members: each gets an equal share of the 256 workgroups; per member the
                // most stream groups, then the most unit chunks that fit the share (as for a single
                // component: fewer only while a workgroup does not fill a 16-row tile)
                // Backward launches of a stack are bound by the matrix instructions of the members that
                // also contract the later member's error terms, while compute units idle: helper members
                // take those products (RNNG_CHAIN_HELPERS = 0: never).
                // Apart, each layer has all compute units: side by side pays while the slowest member's step (its matrix instructions, the
                // exchange counted as STEP_COLUMNS) is no longer than theirs together.  2 x 700 units, N = 40, backward: 28 us a step side
                // by side (groups of 40 streams on 6 rows), 12.6 apart; 2 x 512, N = 64, forward 5.6 against 6.0.  Where the line lies (32 steps, us
                // forward + backward, side by side / apart): 2 x 700, N = 24 242 + 340 / 303 + 399, N = 40 392 + 961 / 367 + 438, 2 x 1,024, N = 12 222 + 238 / 281 + 451, N = 24
                // 378 / 359 forward.
                constexpr int STEP_COLUMNS = 2200;
                int apart = 0;
                for (int m = ch.first; m <= ch.last; ++m) {
                    MstepPick p;
                    for (int J = 4; J >= 1 && !p.G; --J) p = pick_mstep(plan.comps[m], backward, N, J, max_workgroups() / J, false);
                    apart = p.G && apart < (1 << 29) ? apart + p.columns + STEP_COLUMNS : 1 << 30;
                }
                c.split = backward && !ch.bwd_split.empty() && !helpers_off;
                for (int attempt = 0; attempt < 2 && c.source.empty(); ++attempt) {
                    if (attempt == 1) { if (!c.split) break; c.split = false; }
                    const std::vector<CompPlan>& members = chain_members(ch, c);
                    const int share = std::min(256, max_workgroups()) / (int)members.size();
                    c.G.clear(); c.J.clear();
                    int slowest = 0;
                    for (const CompPlan& m : members) {
                        MstepPick p;
                        for (int J = 4; J >= 1 && !p.G; --J) p = pick_mstep(m, backward, N, J, share / J, false);
                        if (!p.G) break;
                        c.G.push_back(p.G); c.J.push_back(p.J);
                        slowest = std::max(slowest, p.columns);
                    }
                    if (c.G.size() == members.size() && slowest + STEP_COLUMNS <= apart) {
                        c.source = jit_mstep_chain_source(plan, members, backward, N, c.G, c.J, &c.lds_bytes, &c.threads, &c.blocked);
                        c.mstep = !c.source.empty();
                        if (c.split && !c.blocked) { c.source.clear(); c.mstep = false; }      // (helpers pay only with the tile-blocked exchange's full tiles)
                    }
                }
                if (c.source.empty()) c.split = false;
            }
        };
        if (use_jit && use_chains && force_step_G <= 0 && !prefer_streaming) {
            // Forward from 3, backward from 5 streams on the matrix cores come first: where every layer is exchanged as one vector of more than
            // 48 columns, or as several of more than 320 together.  us a step, registers against matrix cores: forward 2 x 50 / 100 / 256 units, N = 4
            // 1.42 / 1.75 / 1.91 against 1.22 / 1.22 / 1.39, N = 3 1.36 / 1.58 / 1.87 against 1.22 / 1.23 / 1.39, 2 x 32, N = 5 1.47 against 1.36;
            // backward, N = 5, 2 x 64 / 100 / 128 1.76 / 1.94 / 2.07 against 1.73 / 1.76 / 1.73.
            bool first = N >= (backward ? 5 : 3);
            for (int m = ch.first; m <= ch.last && first; ++m) first = local_streams(plan.comps[m], backward, N, 320, 48);
            if (first) matrix_cores(true);
            registers();
            matrix_cores(N > 8);
        }
        return chain_choices.emplace(key, c).first->second;
    }
};

namespace {

// Launches the GEMM problems of one component and direction, grouped by up to
// GEMM_MAX_PROBLEMS destinations per launch and GEMM_MAX_PAIRS products per destination.
// Rows of frames [t0, t1) only.
// finish: the component whose program these products can finish (CompPlan::in_products), or NULL; *finished is set if they did.
hipError_t run_gemms(rnn_graph* g, const std::vector<GemmProblemPlan>& probs, bool backward, hipStream_t s, int t0, int t1,
                     const CompPlan* finish = nullptr, bool* finished = nullptr) {
    // t0, t1: internal frames
    const int64_t F = (int64_t)g->Ti() * g->N, HN = (int64_t)g->hist() * g->N;
    const int64_t r0 = (int64_t)t0 * g->N, rows = (int64_t)(t1 - t0) * g->N;
    if (probs.empty() || rows <= 0) return hipSuccess;
    const int prof = g->prof.begin(backward ? RNN_PROF_GEMM_BWD : RNN_PROF_GEMM_FWD, s);
    int64_t n_launch = 0;
    GemmGroup grp;
    grp.n_problems = grp.n_pairs = 0;
    auto flush = [&]() -> hipError_t {
        if (grp.n_problems == 0) return hipSuccess;
        // Few output tiles and a long contraction (huge input layers): split the contraction over
        // more workgroups, which add their parts atomically into the zeroed destination.
        int64_t tiles = 0; int kmax = 0;
        for (int i = 0; i < grp.n_problems; ++i) tiles += (int64_t)((grp.p[i].M + 127) / 128) * ((grp.p[i].N + 127) / 128);
        for (int q = 0; q < grp.n_pairs; ++q) kmax = std::max(kmax, grp.pair[q].K);
        int split = 1;
        if (tiles < 256) split = (int)std::max<int64_t>(1, std::min<int64_t>(std::min<int64_t>(16, kmax / 512), (512 + tiles - 1) / tiles));
        for (int i = 0; i < grp.n_problems; ++i) grp.p[i].min_split = split;
        plan_gemm_group(backward ? GEMM_NN : GEMM_NT, grp, g->deterministic);
        // one unsplit product, all of its pairs in this launch and none of them a gather (below): the node's program is done where it is
        // stored.  (2048 rows of 20,000 columns: the program's launch took 210 us, two passes over 164 MB.)
        if (finish && finish->in_products && grp.n_problems == 1 && grp.n_pairs == (int)probs[0].pairs.size() && grp.p[0].split == 1 && !grp.p[0].accumulate) {
            grp.p[0].bias = finish->products_bias >= 0 ? g->weights + finish->products_bias : nullptr;
            grp.p[0].act = finish->products_act;
            *finished = true;
        }
        for (int i = 0; i < grp.n_problems; ++i) {
            if (grp.p[i].split == 1 || grp.p[i].accumulate) continue;
            hipError_t e = launch_fill(grp.p[i].C, (int64_t)grp.p[i].M * grp.p[i].ldc, 0.0f, s);
            if (e != hipSuccess) return e;
            ++n_launch;
        }
        hipError_t e = launch_gemm_group(backward ? GEMM_NN : GEMM_NT, grp, s);
        grp.n_problems = grp.n_pairs = 0; ++n_launch;
        return e;
    };
    for (const auto& pp : probs) {
        GemmProblem* gp = nullptr;
        bool first = true;
        for (const GemmPairPlan& pr : pp.pairs) {
            if (g->is_onehot(pr.a_buf)) continue;      // products with a one-hot source are column gathers, done after the GEMMs (below)
            if (grp.n_pairs == GEMM_MAX_PAIRS || (!gp && grp.n_problems == GEMM_MAX_PROBLEMS)) {
                hipError_t e = flush();
                if (e != hipSuccess) return e;
                gp = nullptr;
            }
            if (!gp) {
                gp = &grp.p[grp.n_problems++];
                std::memset(gp, 0, sizeof(*gp));
                gp->C = g->buf(pp.c_buf) + r0 * pp.n; gp->ldc = pp.n; gp->M = (int)rows; gp->N = pp.n;
                gp->window_M = g->T * g->N;
                gp->first_pair = grp.n_pairs; gp->accumulate = first ? 0 : 1;      // (more pairs than one launch takes: the next one adds)
                first = false;
            }
            GemmPair& o = grp.pair[grp.n_pairs++];
            ++gp->n_pairs;
            o.A = g->buf(pr.a_buf); o.B = g->weights + pr.b_w_off; o.K = pr.k_len; o.lda = pr.k_len;
            o.ldb = backward ? pp.n : pr.k_len;
            o.a_row_off = (int)r0 + (backward ? pr.delay : -pr.delay) * g->N; o.a_rows = (int)F;
            // an input read in place has the window's frames only: its row 0 is internal row HN
            if (g->caller_input(pr.a_buf)) { o.a_row_off -= (int)HN; o.a_rows = (int)(F - HN); }
        }
    }
    {
        hipError_t e = flush();
        if (e != hipSuccess) return e;
    }
    if (!backward)
        for (const auto& pp : probs) {
            bool first = true;
            for (const GemmPairPlan& pr : pp.pairs) if (!g->is_onehot(pr.a_buf)) first = false;      // the GEMMs have written C
            for (const GemmPairPlan& pr : pp.pairs) {
                if (!g->is_onehot(pr.a_buf)) continue;
                // the caller's indices [T][N] (row 0 = internal row HN), or, for an input with delayed
                // connections, the library's copy with history frames in front
                const int32_t* hist_idx = g->onehot_history(pr.a_buf);
                hipError_t e = hist_idx ? launch_onehot_gather(g->buf(pp.c_buf), g->weights + pr.b_w_off, hist_idx, pp.n, pr.k_len, r0, rows,
                                                               (int64_t)pr.delay * g->N, F, !first, s)
                                        : launch_onehot_gather(g->buf(pp.c_buf), g->weights + pr.b_w_off, g->onehot[pr.a_buf], pp.n, pr.k_len, r0, rows,
                                                               HN + (int64_t)pr.delay * g->N, F - HN, !first, s);
                if (e != hipSuccess) return e;
                first = false; ++n_launch;
            }
        }
    g->prof.end(prof, n_launch, s);
    return hipSuccess;
}

XcdMap g_xcd_map[64];
bool g_xcd_local = true;       // RNNG_XCD_LOCAL=0: always write exchanged tensors through

// scratch: SYNC_BYTES of device memory that may be overwritten
hipError_t ensure_xcd_map(unsigned* scratch, hipStream_t s, const XcdMap** out) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    static XcdMap none;
    if (dev < 0 || dev >= 64) { *out = &none; return hipSuccess; }
    XcdMap& m = g_xcd_map[dev];
    if (!m.known) {
        constexpr int NB = (int)(SYNC_BYTES / 4);
        unsigned host[NB];
        e = launch_xcc_probe(scratch, NB, s);
        if (e == hipSuccess) e = hipMemcpyAsync(host, scratch, sizeof(host), hipMemcpyDeviceToHost, s);
        if (e == hipSuccess) e = hipStreamSynchronize(s);
        if (e != hipSuccess) return e;
        m.ok = true;
        for (int b = 8; b < NB; ++b) m.ok = m.ok && host[b] == host[b % 8];
        m.known = true;
    }
    *out = &m;
    return hipSuccess;
}

// The control word for the XCDs of the next launch that exchanges through an XCD's L2, or -1.
hipError_t xcd_word(rnn_graph* g, hipStream_t s, int* word) {
    *word = -1;
    if (!g_xcd_local || !g->xcd || !g->xcd->ok) return hipSuccess;
    if (g->xcd_words_used == XCD_WORDS) {
        hipError_t e = launch_xcd_words_fold(g->ctrl_ptr(), s);
        if (e != hipSuccess) return e;
        g->xcd_words_used = 0;
    }
    *word = XCD_WORDS_FIRST + g->xcd_words_used++;
    return hipSuccess;
}

// The first of the field words (step_layout.h) of the next matrix-core launch with its stream groups on one XCD each, or -1.  They are zero:
// cleared with what is filled for this launch, or at the start of the call for all of its launches.  (In every call, so also in every replay of
// a captured one.)
hipError_t xcd_field_word(rnn_graph* g, hipStream_t s, int count, int* word) {
    *word = -1;
    if (!g_xcd_local || !g->xcd || !g->xcd->ok) return hipSuccess;
    if (!g->prefilled) g->xcd_fields_used = 0;
    if (g->xcd_fields_used + count > XCD_FIELD_WORDS) {
        hipError_t e = launch_fill(reinterpret_cast<float*>(g->ctrl_ptr() + XCD_FIELD_WORDS_FIRST), XCD_FIELD_WORDS, 0.0f, s);
        if (e != hipSuccess) return e;
        g->xcd_fields_used = 0;
    }
    *word = XCD_FIELD_WORDS_FIRST + g->xcd_fields_used;
    g->xcd_fields_used += count;
    return hipSuccess;
}

// The wave-autonomous kernels and the matrix-core kernels with weights in LDS address a stored
// tensor through one buffer descriptor with 32-bit offsets and park idle lanes 1 GiB beyond:
// every tensor of the window must stay below 1 GiB, its twin (whose idle lanes walk the upper 2 GiB)
// below 2 GiB: a width that is no multiple of 4 has a somewhat larger twin.
bool wave_tensor_sizes_ok(const rnn_graph* g) {
    int64_t frame = 1, twin_frame = 0;
    for (int b = 0; b < g->plan.n_bufs; ++b) {
        if (g->plan.buf_alloc[b] == 3) { if (g->layout.buf_off[b] >= 0) twin_frame = std::max(twin_frame, g->plan.frame_floats(b, g->N)); }
        // the caller's input tensors are never stored by a step kernel
        else if (!g->caller_input(b)) frame = std::max<int64_t>(frame, (int64_t)g->N * g->plan.buf_dim[b]);
    }
    return (int64_t)g->Ti() * frame * 4 < (int64_t(1) << 30) && (int64_t)g->Ti() * twin_frame * 4 < (int64_t(1) << 31);
}

// The wave-autonomous kernels can store through ONE buffer descriptor when everything they store
// lies in a window of at most 2 GiB: the workspace, if it is that small and holds every tensor
// but the caller's inputs (which no step kernel stores).  The kernel variant is the same source
// behind one definition.
bool wave_store_window_ok(const rnn_graph* g) {
    if (!g->use_store_window || g->layout.total > (int64_t(1) << 31)) return false;
    for (int b = 0; b < g->plan.n_bufs; ++b) {
        if (g->caller_input(b)) continue;
        const char* p = reinterpret_cast<const char*>(g->buf(b));
        if (p == nullptr) continue;      // no storage: never stored
        const int64_t bytes = (int64_t)g->Ti() * g->plan.frame_floats(b, g->N) * 4;
        if (p < g->ws || p + bytes > g->ws + g->layout.total) return false;
    }
    return true;
}
// The matrix-core build also loads its element-wise inputs through the window: every tensor that
// the phases' programs gather from must lie in the workspace too (not in a tensor of the caller).
bool gathers_in_workspace(const rnn_graph* g, const std::vector<PhasePlan>& phases) {
    for (const PhasePlan& ph : phases) {
        const int32_t* pw = g->plan.words.data() + ph.prog_off;
        for (int i = 0; i < pw[PG_NGATHER]; ++i) {
            const int32_t* ga = pw + PG_HEADER_WORDS + i * GA_WORDS;
            if (ga[GA_KIND] == GA_KIND_ACC) continue;
            const char* p = reinterpret_cast<const char*>(g->buf(ga[GA_BUF]));
            if (g->caller_input(ga[GA_BUF]) || p == nullptr || p < g->ws || p >= g->ws + g->layout.total) return false;
        }
    }
    return true;
}
const std::string& windowed(const std::string& source, std::string& cache) {
    if (cache.empty()) cache = "#define RNNG_STORE_WINDOW 1\n" + source;
    return cache;
}

// Sentinel prefill of the tensors that workgroups poll during frames [t0, t1).  The wave-autonomous
// kernel polls the interleaved bundle tensors instead of bundled members; the members are filled as
// well, so that a fall-back to another kernel build finds them prepared.
// A kernel with tile-blocked exchange polls the twins and nothing else.
std::vector<int> shared_tensors(const rnn_graph* g, const std::vector<int>& bufs, bool with_bundles, bool twins) {
    std::vector<int> list(bufs);
    if (twins) for (int& b : list) if (g->plan.buf_alloc[g->plan.twin_base + b] == 3) b += g->plan.twin_base;      // (tensors without a twin are polled as they are)
    if (with_bundles)
        for (int b : bufs) {
            const int bi = g->plan.bundle_of[b];
            if (bi >= 0 && std::find(list.begin(), list.end(), g->plan.bundles[bi].ebuf) == list.end()) list.push_back(g->plan.bundles[bi].ebuf);
        }
    return list;
}
void add_range(const rnn_graph* g, FillRanges& fr, int b, int t0, int t1) {
    const int64_t frame = g->plan.frame_floats(b, g->N);
    const bool ragged = g->plan.buf_alloc[b] == 3 && frame != (int64_t)g->N * g->plan.buf_dim[b];
    fr.twin_n[fr.count] = ragged ? g->N : 0; fr.twin_dim[fr.count] = ragged ? g->plan.buf_dim[b] : 0;
    fr.p[fr.count] = g->buf(b) + t0 * frame; fr.n[fr.count] = (t1 - t0) * frame;
    ++fr.count;
}
// fields: the launch's field words (xcd_field_word) are cleared along.
hipError_t fill_shared(rnn_graph* g, const std::vector<int>& bufs, bool with_bundles, int t0, int t1, hipStream_t s, bool twins = false, bool fields = false) {
    if (g->prefilled) return hipSuccess;
    FillRanges fr; fr.count = 0;
    for (int b : shared_tensors(g, bufs, with_bundles, twins)) {
        add_range(g, fr, b, t0, t1);
        if (fr.count == FILL_MAX_RANGES) {
            hipError_t e = launch_fill_sentinel_ranges(fr, s);
            if (e != hipSuccess) return e;
            fr.count = 0;
        }
    }
    return fields ? launch_fill_sentinel_and_clear(fr, nullptr, nullptr, 0, 0, nullptr, 0, g->ctrl_ptr() + XCD_FIELD_WORDS_FIRST, XCD_FIELD_WORDS, s)
                  : launch_fill_sentinel_ranges(fr, s);
}

// The workgroups of a persistent step launch wait for each other's results, so every one that takes
// part must be resident at the same time: at most one per compute unit (each takes most of a CU's
// LDS or registers).  A launch that cannot be co-resident is refused here, before it could hang.
bool launch_fits_device(const rnn_graph* g, int participants, std::string& why) {
    if (participants <= g->max_workgroups()) return true;
    why = "the step kernel needs " + std::to_string(participants) + " co-resident workgroups, the device has " +
          std::to_string(g->max_workgroups()) + " compute units";
    return false;
}

// Result of a step-kernel launch attempt.  A specialised kernel that exists but cannot be compiled,
// loaded or launched is an error (text in `err`), never a silent switch to another build; only
// "there is no such kernel for this component" (or no run-time compiler on this machine) moves on
// to the next build.
struct StepRun { hipError_t e = hipSuccess; bool error = false; int code = RNN_ERR_DEVICE; std::string err; };
StepRun step_error(hipError_t e, const std::string& what, int code = RNN_ERR_DEVICE) {
    StepRun r; r.e = e == hipSuccess ? hipErrorUnknown : e; r.error = true; r.code = code;
    r.err = what + (e != hipSuccess ? std::string(": ") + hipGetErrorString(e) : std::string());
    return r;
}

// t0, t1: internal frames
StepRun run_phases(rnn_graph* g, int comp, bool backward, hipStream_t s, int t0, int t1) {
    const CompPlan& cp = g->plan.comps[comp];
    const PlanView pv = g->view();
    const std::vector<PhasePlan>& phases = backward ? cp.bwd_phases : cp.fwd_phases;
    const int T = g->Ti(), N = g->N;
    StepRun ok;
    if (!cp.recurrent) {
        const int prof = g->prof.begin(RNN_PROF_OTHER, s);
        for (const PhasePlan& ph : phases) {
            hipError_t e = launch_node_program(pv, ph.prog_off, ph.max_dim, ph.quads, g->weights, T, N, t0, t1, s);
            if (e != hipSuccess) return step_error(e, "node program launch");
        }
        g->prof.end(prof, (int64_t)phases.size(), s);
        return ok;
    }
    const int prof = g->prof.begin(backward ? RNN_PROF_STEP_BWD : RNN_PROF_STEP_FWD, s);
    int64_t n_launch = 0;
    int& served = g->served[comp][backward ? 1 : 0];
    // Persistent kernel: all steps in one launch.  First choice is the build specialised at run
    // time for this component; the interpreting build serves components no specialised build
    // takes, or all of them when the run-time compiler is unavailable; stepping with per-frame
    // launches is the last resort.
    StepLaunchPlan lp;
    const int desc_off = backward ? cp.bwd_desc_off : cp.fwd_desc_off;
    rnn_graph::JitChoice* jc = (g->use_jit && jit_available()) ? const_cast<rnn_graph::JitChoice*>(&g->jit_choice(comp, backward, N)) : nullptr;
    const bool have_jit = jc && !jc->source.empty() && !g->framewise &&
                          (!(jc->wave || jc->element_wise || (jc->mstep && !jc->two_d)) || wave_tensor_sizes_ok(g));
    const bool have_interp = !g->framewise && plan_step_launch(g->plan.words.data(), desc_off, N, g->force_step_G, lp);
    const int spin_limit = g->spin_limit;
    // (measured for matrix-core launches per direction; backward loops, with more stores and loads per
    // step, gain 3 %, forward loops lose 4 to 6 %)
    const bool window = have_jit && (jc->wave || (((jc->mstep && !jc->two_d && backward) || jc->element_wise) && gathers_in_workspace(g, phases))) && wave_store_window_ok(g);
    // Element-wise recurrences beyond the register build's streams can also go frame by frame, without code that has to be loaded first: a
    // call that may load none takes that way where nothing has.
    const bool have_fn = have_jit && !(g->no_alloc && jc->element_wise && N > 8 &&
                                       !jit_step_function(window ? windowed(jc->source, jc->source_window) : jc->source, nullptr, false, STEP_LDS_LIMIT));
    if (have_fn) {
        hipError_t fe = fill_shared(g, backward ? cp.bwd_shared_bufs : cp.fwd_shared_bufs, jc->wave, t0, t1, s, jc->blocked, jc->local);
        if (fe != hipSuccess) return step_error(fe, "sentinel fill");
        std::string why;
        hipFunction_t fn = jit_step_function(window ? windowed(jc->source, jc->source_window) : jc->source, &why, !g->no_alloc,
                                             jc->mstep && !jc->two_d ? MSTEP_LDS_LIMIT : STEP_LDS_LIMIT);
        if (!fn) return step_error(hipSuccess, "specialised step kernel unavailable: " + why, g->no_alloc ? RNN_ERR_SEQUENCE : RNN_ERR_DEVICE);
        StepArgs a;
        fill_step_args(a, pv, jc->lp, desc_off, g->weights, g->ctrl_ptr(), T, N, backward, spin_limit, t0, t1);
        if (window) { a.store_base = reinterpret_cast<float*>(g->ws); a.store_bytes = (unsigned)g->layout.total; }
        a.J = jc->J;
        a.twin_base = g->plan.twin_base;
        a.lay = g->layout_at(g->lay.comp[2 * comp + (backward ? 1 : 0)]); a.table_bytes = g->table_bytes();
        if (jc->two_d) {
            if (g->layout.partial_off < 0) return step_error(hipErrorInvalidValue, "partial-sum tensor missing from the workspace");
            a.partial = reinterpret_cast<float*>(g->ws + g->layout.partial_off);
            hipError_t e = launch_fill_sentinel(a.partial + (int64_t)t0 * jc->partial_floats, (int64_t)(t1 - t0) * jc->partial_floats, s);
            if (e != hipSuccess) return step_error(e, "sentinel fill");
        }
        if (jc->stream) {
            a.weight_bytes = (unsigned)(g->plan.n_params * 4);
            a.weights_t = g->weights;
            if (jc->needs_t) {
                // the matrices this direction reads transposed: a transposed copy at the same offsets, made per launch
                if (g->layout.wt_off < 0) return step_error(hipErrorInvalidValue, "transposed weight copy missing from the workspace");
                float* wt = reinterpret_cast<float*>(g->ws + g->layout.wt_off);
                a.weights_t = wt;
                StepLayout lay;
                compute_step_layout(g->plan.words.data(), desc_off, jc->lp.G, 1, 1, lay);      // (one stream: only the task list is needed)
                if (!lay.ok) return step_error(hipErrorInvalidValue, "step layout of a streaming kernel");
                for (int t = 0; t < lay.ph[0].n_tasks; ++t)
                    for (int e2 = 0; e2 < lay.ph[0].task[t].n_edges; ++e2) {
                        const StepEdge& ed = lay.ph[0].task[t].e[e2];
                        if (!ed.transposed) continue;
                        // stored [k_len][n_out]; the kernel streams rows of [n_out][k_len]
                        hipError_t te = launch_transpose(wt + ed.w_off, g->weights + ed.w_off, ed.k_len, lay.ph[0].task[t].n_out, s);
                        if (te != hipSuccess) return step_error(te, "weight transposition");
                    }
            }
        }
        if (jc->local || (jc->wave && jc->lp.xcd_stride == 8)) {
            hipError_t we = jc->local ? xcd_field_word(g, s, xcd_field_words(jc->lp.G, jc->J), &a.xcd_word) : xcd_word(g, s, &a.xcd_word);
            if (we != hipSuccess) return step_error(we, "XCD words");
        }
        StepLaunchPlan lp_all = jc->lp;
        lp_all.G = jc->lp.G * jc->J;       // launch size; a.G stays the number of unit chunks
        if (!jc->element_wise && !launch_fits_device(g, lp_all.G, why)) return step_error(hipSuccess, why);
        if (jc->local) { lp_all.G = mstep_local_blocks(jc->lp.G, jc->J); lp_all.xcd_stride = 1; }
        hipError_t e = jit_launch(fn, a, lp_all, s);
        if (e != hipSuccess) { (void)hipGetLastError(); return step_error(e, "specialised step kernel launch"); }
        served = jc->wave || jc->element_wise ? RNN_BUILD_WAVE : jc->two_d ? RNN_BUILD_MATRIX_2D : jc->stream ? RNN_BUILD_STREAMING : jc->mstep ? RNN_BUILD_MATRIX : RNN_BUILD_LDS;
        g->prof.end(prof, 1, s);
        return ok;
    }
    if (have_interp) {
        std::string why;
        if (!launch_fits_device(g, lp.G, why)) return step_error(hipSuccess, why);
        hipError_t fe = fill_shared(g, backward ? cp.bwd_shared_bufs : cp.fwd_shared_bufs, false, t0, t1, s);
        if (fe != hipSuccess) return step_error(fe, "sentinel fill");
        hipError_t e = launch_recurrent_steps(pv, lp, desc_off, g->weights, g->ctrl_ptr(), T, N, backward, spin_limit, t0, t1, s);
        if (e != hipSuccess) return step_error(e, "interpreting step kernel launch");
        served = RNN_BUILD_INTERPRETED;
        g->prof.end(prof, 1, s);
        return ok;
    }
    for (int step = 0; step < t1 - t0; ++step) {
        const int t = backward ? t1 - 1 - step : t0 + step;
        for (const PhasePlan& ph : phases) {
            if (ph.mv_off >= 0) {
                hipError_t e = launch_step_matvec(pv, ph.mv_off, ph.n_mv_tasks, ph.mv_max_out, g->weights, T, N, t, s);
                if (e != hipSuccess) return step_error(e, "per-frame matrix-vector launch");
                ++n_launch;
            }
            hipError_t e = launch_node_program(pv, ph.prog_off, ph.max_dim, ph.quads, g->weights, T, N, t, t + 1, s);
            if (e != hipSuccess) return step_error(e, "per-frame node program launch");
            ++n_launch;
        }
    }
    served = RNN_BUILD_PER_FRAME;
    g->prof.end(prof, n_launch, s);
    return ok;
}

// All members of a chain in one persistent launch.  e == hipErrorNotSupported without `error`: no
// such kernel for this chain (the caller then runs the members one after another).
StepRun run_chain(rnn_graph* g, int chain, bool backward, hipStream_t s, int t0, int t1) {
    const ChainPlan& ch = g->plan.chains[chain];
    StepRun none; none.e = hipErrorNotSupported;
    if (!g->use_jit || !jit_available()) return none;
    rnn_graph::ChainChoice& cc = const_cast<rnn_graph::ChainChoice&>(g->chain_choice(chain, backward, g->N));
    if (cc.source.empty() || !wave_tensor_sizes_ok(g)) return none;
    bool window = wave_store_window_ok(g) && (!cc.mstep || backward);      // (matrix-core build: backward launches only, as for single components)
    if (cc.mstep && window) for (const CompPlan& m : rnn_graph::chain_members(ch, cc)) window = window && gathers_in_workspace(g, m.bwd_phases);
    std::string why;
    hipFunction_t fn = jit_step_function(window ? windowed(cc.source, cc.source_window) : cc.source, &why, !g->no_alloc,
                                         cc.mstep ? MSTEP_LDS_LIMIT : STEP_LDS_LIMIT);
    if (!fn) return step_error(hipSuccess, "specialised chain step kernel unavailable: " + why, g->no_alloc ? RNN_ERR_SEQUENCE : RNN_ERR_DEVICE);
    const PlanView pv = g->view();
    const int T = g->Ti(), N = g->N;
    const int prof = g->prof.begin(backward ? RNN_PROF_STEP_BWD : RNN_PROF_STEP_FWD, s);
    const std::vector<CompPlan>& members = rnn_graph::chain_members(ch, cc);
    {
        std::vector<int> exchanged;      // of all members: one fill launch
        for (const CompPlan& m : members)
            for (int b : backward ? m.bwd_shared_bufs : m.fwd_shared_bufs) exchanged.push_back(b);
        hipError_t e = fill_shared(g, exchanged, !cc.mstep, t0, t1, s, cc.blocked);
        if (e != hipSuccess) return step_error(e, "sentinel fill");
    }
    StepLaunchPlan lp; lp.ok = true; lp.G = 32; lp.NB = step_nb_for(N); lp.lds_bytes = 0; lp.xcd_stride = 8;
    if (cc.mstep) {
        lp.G = 0; lp.NB = 1; lp.lds_bytes = cc.lds_bytes; lp.xcd_stride = 1; lp.threads = cc.threads;
        for (size_t i = 0; i < cc.G.size(); ++i) lp.G += cc.G[i] * cc.J[i];      // launch size
    }
    StepArgs a;
    fill_step_args(a, pv, lp, backward ? members[0].bwd_desc_off : members[0].fwd_desc_off, g->weights, g->ctrl_ptr(),
                   T, N, backward, g->spin_limit, t0, t1);
    if (window) { a.store_base = reinterpret_cast<float*>(g->ws); a.store_bytes = (unsigned)g->layout.total; }
    a.n_groups = (int)members.size();
    a.twin_base = g->plan.twin_base;
    a.table_bytes = g->table_bytes();
    const int first_lay = g->lay.chain[2 * chain + (backward ? 1 : 0)];
    for (int i = 0; i < a.n_groups; ++i) {
        a.grp_desc_off[i] = backward ? members[i].bwd_desc_off : members[i].fwd_desc_off;
        a.grp_G[i] = cc.G[i];
        a.grp_lay[i] = g->layout_at(first_lay < 0 ? -1 : first_lay + i);
        if (cc.mstep) {
            a.grp_J[i] = cc.J[i];
            a.grp_first[i] = i == 0 ? 0 : a.grp_first[i - 1] + cc.G[i - 1] * cc.J[i - 1];
        }
    }
    if (!cc.mstep) {
        hipError_t we = xcd_word(g, s, &a.xcd_word);
        if (we != hipSuccess) return step_error(we, "XCD words");
    }
    int participants = 0;
    for (size_t i = 0; i < cc.G.size(); ++i) participants += cc.G[i] * (cc.mstep ? cc.J[i] : 1);
    if (!launch_fits_device(g, participants, why)) return step_error(hipSuccess, why);
    hipError_t e = jit_launch(fn, a, lp, s);
    if (e != hipSuccess) { (void)hipGetLastError(); return step_error(e, "specialised chain step kernel launch"); }
    for (int c = ch.first; c <= ch.last; ++c) g->served[c][backward ? 1 : 0] = (cc.mstep ? RNN_BUILD_MATRIX : RNN_BUILD_WAVE) | RNN_BUILD_CHAIN | (cc.split ? RNN_BUILD_HELPERS : 0);
    g->prof.end(prof, 1, s);
    StepRun ok;
    return ok;
}

// The tensors that all step launches of a direction poll during frames [t0, t1), if they are few and small: a call fills them with its first
// launch, together with what it clears, instead of with one launch per step launch.  Only where all that the call touches is far less than the
// 256 MiB memory-side cache: what is filled must still be there when it is polled (Elman 38,000-512-20,000, 2,048 frames, whose products
// move 400 MB before the step loop: 5.00 -> 5.69 ms).  Apart / together, us forward + backward: 64 units, one stream, 64 frames (1 MiB) 70 + 61 / 69 + 60, 256 units, 64 streams,
// 4 frames (9 MiB) 44 + 34 / 44 + 31, 16 frames (29 MiB) 62 + 63 / 63 + 62, 64 frames (111 MiB) 136 + 166 / 137 + 164: on both sides of the limits the difference is a per cent.
bool all_shared(rnn_graph* g, bool backward, int t0, int t1, FillRanges& fr) {
    fr.count = 0;
    if (g->framewise) return false;
    int64_t floats = 0;
    auto add = [&](const std::vector<int>& list) {
        for (int b : list) {
            if (fr.count == FILL_MAX_RANGES) return false;
            add_range(g, fr, b, t0, t1);
            floats += fr.n[fr.count - 1];
        }
        return floats <= (4 << 20);
    };
    const Plan& P = g->plan;
    int64_t touched = g->layout.total + 4 * P.n_params;
    for (int k : P.input_nodes) if (!g->is_onehot(k)) touched += (int64_t)g->T * g->N * P.xnodes[k].dim * 4;
    if (touched > (64 << 20)) return false;
    const bool jit = g->use_jit && jit_available();
    for (size_t c = 0; c < P.comps.size(); ++c) {
        const CompPlan& cp = P.comps[c];
        if (!cp.recurrent || !(backward ? cp.has_bwd_program : cp.has_fwd_program)) continue;
        if (cp.chain >= 0 && jit && wave_tensor_sizes_ok(g)) {
            const ChainPlan& ch = P.chains[cp.chain];
            const rnn_graph::ChainChoice& cc = g->chain_choice(cp.chain, backward, g->N);
            if (!cc.source.empty()) {
                if ((int)c != ch.first) continue;
                std::vector<int> exchanged;
                for (const CompPlan& m : rnn_graph::chain_members(ch, cc))
                    for (int b : backward ? m.bwd_shared_bufs : m.fwd_shared_bufs) exchanged.push_back(b);
                if (!add(shared_tensors(g, exchanged, !cc.mstep, cc.blocked))) return false;
                continue;
            }
        }
        const std::vector<int>& bufs = backward ? cp.bwd_shared_bufs : cp.fwd_shared_bufs;
        const rnn_graph::JitChoice* jc = jit ? &g->jit_choice((int)c, backward, g->N) : nullptr;
        if (jc && !jc->source.empty() && (!(jc->wave || jc->element_wise || (jc->mstep && !jc->two_d)) || wave_tensor_sizes_ok(g))) {
            if (!add(shared_tensors(g, bufs, jc->wave, jc->blocked))) return false;
        } else {
            return false;      // (other builds fill their own)
        }
    }
    return true;
}

}  // namespace

extern "C" {

const char* rnn_last_error(void) { return g_last_error.c_str(); }

int rnn_graph_create(const rnn_node_desc* nodes, int32_t n_nodes, const rnn_edge_desc* edges, int32_t n_edges,
                     rnn_graph** out) {
    if (!out) return fail(RNN_ERR_INVALID_ARGUMENT, "out is NULL");
    *out = nullptr;
    if (!nodes || n_nodes <= 0 || n_edges < 0 || (n_edges > 0 && !edges))
        return fail(RNN_ERR_INVALID_ARGUMENT, "node / edge list missing");
    std::vector<GNode> ns(n_nodes); std::vector<GEdge> es(n_edges);
    for (int i = 0; i < n_nodes; ++i) ns[i] = GNode{nodes[i].kind, nodes[i].act, nodes[i].dim, nodes[i].has_bias != 0, nodes[i].is_output};
    for (int i = 0; i < n_edges; ++i) es[i] = GEdge{edges[i].src, edges[i].dst, edges[i].delay, edges[i].wkind};
    rnn_graph* g = new (std::nothrow) rnn_graph();
    if (!g) return fail(RNN_ERR_NO_MEMORY, "out of host memory");
    std::string err;
    if (!build_plan(ns, es, g->plan, err)) { delete g; return fail(RNN_ERR_INVALID_GRAPH, err); }
    g->served.assign(g->plan.comps.size(), std::array<int, 2>{0, 0});
    g->grad_groups.reserve(g->plan.grad_gemms.size() / GEMM_MAX_PROBLEMS + 1);
    g->grad_owned.reserve(g->plan.grad_gemms.size());
    if (const char* env = std::getenv("RNNG_SPIN_LIMIT")) g->spin_limit = std::max(1, std::atoi(env));
    if (const char* env = std::getenv("RNNG_MSTEP_LOCAL")) g->local_env = std::atoi(env);
    if (const char* env = std::getenv("RNNG_STEP_WORKGROUPS")) g->force_step_G = std::atoi(env);
    if (const char* env = std::getenv("RNNG_STEP_STREAM_GROUPS")) g->force_step_J = std::atoi(env);
    if (const char* env = std::getenv("RNNG_CHAIN")) g->use_chains = std::atoi(env) != 0;
    if (const char* env = std::getenv("RNNG_STEP_BUILD")) g->prefer_streaming = std::string(env) == "stream";
    if (const char* env = std::getenv("RNNG_SCHEDULE")) g->framewise = std::string(env) == "framewise";
    if (const char* env = std::getenv("RNNG_LAYOUT_SKEW")) g_layout_skew = std::atoll(env) / 256 * 256;
    if (const char* env = std::getenv("RNNG_BUNDLE"))
        if (std::atoi(env) == 0) g->plan.bundle_of.assign(g->plan.bundle_of.size(), -1);      // tuning aid: no exchange bundles
    if (const char* env = std::getenv("RNNG_JIT")) g->use_jit = std::atoi(env) != 0;
    if (const char* env = std::getenv("RNNG_STORE_WINDOW")) g->use_store_window = std::atoi(env) != 0;
    {
        const char* env = std::getenv("RNNG_XCD_LOCAL");
        g_xcd_local = env ? std::atoi(env) != 0 : true;
    }
    *out = g;
    return RNN_OK;
}

void rnn_graph_destroy(rnn_graph* g) { delete g; }

int rnn_graph_schedule(const rnn_graph* g, int32_t* node_comp, int32_t* node_level, int32_t* comp_level,
                       int32_t* comp_recurrent, int32_t* edge_class, int32_t* n_comps) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    const Schedule& S = g->plan.sched;
    const int K = (int)g->plan.nodes.size(), M = (int)g->plan.edges.size();
    for (int v = 0; v < K; ++v) {
        if (node_comp) node_comp[v] = S.node_comp[v];
        if (node_level) node_level[v] = S.node_level[v];
        if (comp_level) comp_level[v] = S.comp_level[S.node_comp[v]];
        if (comp_recurrent) comp_recurrent[v] = S.comp_recurrent[S.node_comp[v]];
    }
    if (edge_class) for (int m = 0; m < M; ++m) edge_class[m] = S.edge_class[m];
    if (n_comps) *n_comps = S.n_comps;
    return RNN_OK;
}

int64_t rnn_param_count(const rnn_graph* g) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    return g->plan.n_params;
}

int rnn_edge_param_offset(const rnn_graph* g, int32_t edge, int64_t* off, int64_t* len) {
    if (!g || !off || !len) return fail(RNN_ERR_INVALID_ARGUMENT, "NULL argument");
    if (edge < 0 || edge >= (int)g->plan.edges.size()) return fail(RNN_ERR_INVALID_ARGUMENT, "edge index out of range");
    *off = g->plan.edge_off[edge]; *len = g->plan.edge_len[edge];
    return RNN_OK;
}

int rnn_bias_param_offset(const rnn_graph* g, int32_t node, int64_t* off, int64_t* len) {
    if (!g || !off || !len) return fail(RNN_ERR_INVALID_ARGUMENT, "NULL argument");
    if (node < 0 || node >= (int)g->plan.nodes.size()) return fail(RNN_ERR_INVALID_ARGUMENT, "node index out of range");
    *off = g->plan.bias_off[node]; *len = g->plan.bias_len[node];
    return RNN_OK;
}

int64_t rnn_workspace_bytes(const rnn_graph* g, int32_t T, int32_t N) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (T <= 0 || N <= 0) return fail(RNN_ERR_INVALID_ARGUMENT, "T and N must be positive");
    if ((int64_t)(T + g->plan.hist) * N >= (int64_t(1) << 31)) return fail(RNN_ERR_INVALID_ARGUMENT, "T * N exceeds 2^31 - 1");
    return const_cast<rnn_graph*>(g)->layout_for(T, N).total;
}

namespace {

// Waits for the stream, then reads the control words of the current window: E_total (to *loss if
// given) and the flags the kernels raise.  A raised flag means the window's results are invalid.
int read_control(rnn_graph* g, double* loss, hipStream_t s) {
    unsigned char back[SYNC_BYTES];
    hipError_t e = hipMemcpyAsync(back, g->loss_ptr(), sizeof(back), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail_hip(e, "control word read-back");
    if (loss) std::memcpy(loss, back, sizeof(double));
    unsigned flag; std::memcpy(&flag, back + 16, 4);
    for (int i = 0; i < g->xcd_words_used; ++i) {
        unsigned w; std::memcpy(&w, back + 16 + 4 * (XCD_WORDS_FIRST + i), 4);
        if (xcd_word_split(w)) flag = 2;
    }
    if (flag == 3) return fail(RNN_ERR_INVALID_ARGUMENT, "a target class index is not below the output layer's width (that frame was left out)");
    if (flag == 2) return fail(RNN_ERR_DEVICE, "the workgroups of a recurrent layer ran on several XCDs (results are invalid; RNNG_XCD_LOCAL=0 avoids the assumption)");
    if (flag) return fail(RNN_ERR_DEVICE, "a recurrent step kernel ran into its wait limit (results are invalid)");
    return RNN_OK;
}

// Forward pass over internal frames [t0, t1) of the current window: components in schedule order.
int forward_frames(rnn_graph* g, int t0, int t1, hipStream_t s) {
    const Plan& P = g->plan;
    const int N = g->N;
    hipError_t e;
    int chain_done_to = -1;   // components up to this index were run as a chain
    for (const CompPlan& cp : P.comps) {
        if (!cp.has_fwd_program) continue;
        const int c = (int)(&cp - P.comps.data());
        if (c <= chain_done_to) continue;
        if (!g->framewise && cp.chain >= 0 && P.chains[cp.chain].first == c && !g->chain_choice(cp.chain, false, N).source.empty()) {
            const ChainPlan& ch = P.chains[cp.chain];
            for (const CompPlan& m : ch.members) {
                e = run_gemms(g, m.fwd_gemms, false, s, t0, t1);
                if (e != hipSuccess) return fail_hip(e, "forward GEMM");
            }
            const StepRun r = run_chain(g, cp.chain, false, s, t0, t1);
            if (r.error) return fail(r.code, "forward: " + r.err);
            if (r.e == hipSuccess) { chain_done_to = ch.last; continue; }
        }
        bool finished = false;
        e = run_gemms(g, cp.fwd_gemms, false, s, t0, t1, &cp, &finished);
        if (e != hipSuccess) return fail_hip(e, "forward GEMM");
        if (!finished) {
            const StepRun r = run_phases(g, c, false, s, t0, t1);
            if (r.error) return fail(r.code, "forward: " + r.err);
        }
        if (cp.softmax_node >= 0) {
            const int dim = P.xnodes[cp.softmax_node].dim;
            e = launch_softmax_rows(g->buf(P.ybuf(cp.softmax_node)) + (int64_t)t0 * N * dim, (int64_t)(t1 - t0) * N, dim, s);
            if (e != hipSuccess) return fail_hip(e, "softmax");
        }
    }
    return RNN_OK;
}

}  // namespace

int rnn_forward_range(rnn_graph* g, const float* d_weights, const float* const* d_inputs, int32_t T, int32_t N,
                      int32_t t_begin, int32_t t_end, void* d_workspace, int64_t ws_bytes, void* hip_stream) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (!d_weights || !d_inputs) return fail(RNN_ERR_INVALID_ARGUMENT, "weights / inputs pointer is NULL");
    if (T <= 0 || N <= 0) return fail(RNN_ERR_INVALID_ARGUMENT, "T and N must be positive");
    if ((int64_t)(T + g->plan.hist) * N >= (int64_t(1) << 31)) return fail(RNN_ERR_INVALID_ARGUMENT, "T * N exceeds 2^31 - 1");
    if (t_begin < 0 || t_end > T || t_begin >= t_end) return fail(RNN_ERR_INVALID_ARGUMENT, "frame range must satisfy 0 <= t_begin < t_end <= T");
    const Plan& P = g->plan;
    for (size_t i = 0; i < P.input_nodes.size(); ++i)
        if (!d_inputs[i] && !g->is_onehot(P.input_nodes[i])) return fail(RNN_ERR_INVALID_ARGUMENT, "an input tensor pointer is NULL");
    if (!d_workspace) return fail(RNN_ERR_WORKSPACE, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(d_workspace) & 255) return fail(RNN_ERR_WORKSPACE, "workspace is not 256-byte aligned");
    if (ws_bytes < g->layout_for(T, N).total)
        return fail(RNN_ERR_WORKSPACE, "workspace too small: need " + std::to_string(g->layout_for(T, N).total) + " bytes");
    if (g->cu_count == 0) {
        // The step kernels' launch shapes depend on how many workgroups the device keeps resident.
        int dev = 0, cus = 0;
        hipError_t qe = hipGetDevice(&dev);
        if (qe == hipSuccess) qe = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (qe != hipSuccess || cus <= 0) return fail_hip(qe, "device query");
        if (cus != g->max_workgroups()) g->drop_choices();      // chosen for a whole device
        g->cu_count = cus;
    }
    Layout L = g->layout_for(T, N);
    if (ws_bytes < L.total) return fail(RNN_ERR_WORKSPACE, "workspace too small: need " + std::to_string(L.total) + " bytes");
    if (t_begin > 0) {
        // the earlier frames must be there: same window shape and workspace, computed up to t_begin
        if (g->ws != static_cast<char*>(d_workspace) || g->T != T || g->N != N || g->fwd_upto < t_begin)
            return fail(RNN_ERR_SEQUENCE, "frames before t_begin have not been computed in this workspace");
    }
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    g->fwd_done = g->bptt_done = g->prefilled = false;

    g->T = T; g->N = N; g->ws = static_cast<char*>(d_workspace); g->layout = L; g->weights = d_weights;
    g->inputs.assign(P.xnodes.size(), nullptr);
    for (size_t i = 0; i < P.input_nodes.size(); ++i) g->inputs[P.input_nodes[i]] = d_inputs[i];

    // plan tables: buffer pointers, widths, program words, layouts of the step launches
    const bool sizes_ok = wave_tensor_sizes_ok(g);
    if (g->lay.N != N || g->lay.sizes_ok != sizes_ok) g->lay = g->step_layouts(N, sizes_ok);
    const int64_t blob_bytes = L.lay_off + (int64_t)g->lay.words.size() * 4;
    // A later piece of a window finds the tables where its first one put them, as it finds that one's frames, unless an address has changed
    // (one new frame of 2 x 512 LSTM units: 52.8 us with the upload, 41.3 without).
    std::vector<char>& blob = g->blob;
    bool there = t_begin > 0 && g->tables_there && (int64_t)blob.size() == blob_bytes;
    if ((int64_t)blob.size() != blob_bytes) blob.assign(blob_bytes, 0);
    auto put = [&](int64_t off, const void* p, size_t bytes) {
        if (bytes == 0 || (there && std::memcmp(&blob[off], p, bytes) == 0)) return;
        there = false;
        std::memcpy(&blob[off], p, bytes);
    };
    put(L.lay_off, g->lay.words.data(), g->lay.words.size() * 4);
    for (int b = 0; b < P.n_bufs; ++b) {
        float* p = g->buf(b);
        put(L.table_off + 8 * (int64_t)b, &p, 8);
    }
    put(L.dims_off, P.buf_dim.data(), (size_t)P.n_bufs * 4);
    for (int b = 0; b < P.n_bufs; ++b) {
        const int64_t frame = ((P.buf_alloc[b] == 1 || P.buf_alloc[b] == 3) && L.buf_off[b] >= 0) ? P.frame_floats(b, N) : 0;
        put(L.frames_off + 8 * (int64_t)b, &frame, 8);
    }
    put(L.words_off, P.words.data(), P.words.size() * 4);
    hipError_t e = hipSuccess;
    if (!there) {
        // (without allocations: as kernel arguments, which need no staging buffer of the runtime's)
        e = g->no_alloc ? launch_upload_words(reinterpret_cast<uint32_t*>(g->ws), reinterpret_cast<const uint32_t*>(blob.data()), blob_bytes / 4, s)
                        : hipMemcpyAsync(g->ws, blob.data(), (size_t)blob_bytes, hipMemcpyHostToDevice, s);
        g->tables_there = e == hipSuccess;
    }
    if (e != hipSuccess) return fail_hip(e, "plan table upload");
    if (!g->xcd) {
        e = ensure_xcd_map(reinterpret_cast<unsigned*>(g->ws + L.sync_off), s, &g->xcd);
        if (e != hipSuccess) return fail_hip(e, "XCD probe");
    }
    const int H = P.hist;
    if (t_begin == 0) {
        // A new window: the control words (loss, error flags) start at zero, and so do the history
        // frames in front of every frame tensor (the state before a fresh window is zero).  Pieces
        // of a window computed later keep the flags an earlier piece has raised.
        g->xcd_words_used = 0;
        FillRanges fr;
        const bool few = all_shared(g, false, H, H + t_end, fr);
        if (few) e = launch_fill_sentinel_and_clear(fr, g->view().buf_ptr, reinterpret_cast<const int64_t*>(g->ws + L.frames_off), H > 0 ? P.n_bufs : 0, H,
                                                    reinterpret_cast<unsigned*>(g->ws + L.sync_off), (int)(SYNC_BYTES / 4), nullptr, 0, s);
        else e = launch_zero_history(g->view().buf_ptr, reinterpret_cast<const int64_t*>(g->ws + L.frames_off), P.n_bufs, H,
                                reinterpret_cast<unsigned*>(g->ws + L.sync_off), (int)(SYNC_BYTES / 4), s);
        if (e != hipSuccess) return fail_hip(e, "window reset");
        g->prefilled = few;
        g->xcd_fields_used = 0;
    }
    // one-hot inputs with delayed connections: their class indices likewise (-1, the zero vector, in a fresh window's history)
    for (size_t i = 0; i < P.input_nodes.size(); ++i) {
        const int k = P.input_nodes[i];
        int32_t* hist_idx = g->is_onehot(k) ? g->onehot_history(k) : nullptr;
        if (!hist_idx) continue;
        if (t_begin == 0 && H > 0) {
            e = launch_fill_sentinel(reinterpret_cast<float*>(hist_idx), (int64_t)H * N, s);      // all bits set = -1
            if (e != hipSuccess) return fail_hip(e, "index history reset");
        }
        e = hipMemcpyAsync(hist_idx + (int64_t)(H + t_begin) * N, g->onehot[k] + (int64_t)t_begin * N, (size_t)(t_end - t_begin) * N * sizeof(int32_t),
                           hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return fail_hip(e, "index copy");
    }
    // inputs that are not read in place: the new frames go behind the history frames of their copy
    for (size_t i = 0; i < P.input_nodes.size(); ++i) {
        const int k = P.input_nodes[i];
        if (!P.input_staged[k] || g->is_onehot(k)) continue;
        const int64_t fr = (int64_t)N * P.xnodes[k].dim;
        e = hipMemcpyAsync(g->buf(P.ybuf(k)) + (int64_t)(H + t_begin) * fr, d_inputs[i] + (int64_t)t_begin * fr,
                           (size_t)(t_end - t_begin) * fr * sizeof(float), hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return fail_hip(e, "input copy");
    }

    if (g->framewise) {
        for (int t = t_begin; t < t_end; ++t) {
            const int rc = forward_frames(g, H + t, H + t + 1, s);
            if (rc != RNN_OK) return rc;
        }
    } else {
        const int rc = forward_frames(g, H + t_begin, H + t_end, s);
        g->prefilled = false;
        if (rc != RNN_OK) return rc;
    }
    g->fwd_upto = t_end;
    g->fwd_done = t_end == T;
    return RNN_OK;
}

int rnn_forward(rnn_graph* g, const float* d_weights, const float* const* d_inputs, int32_t T, int32_t N,
                void* d_workspace, int64_t ws_bytes, void* hip_stream) {
    return rnn_forward_range(g, d_weights, d_inputs, T, N, 0, T, d_workspace, ws_bytes, hip_stream);
}

// ---- rnn_forward_static: the workspace of callers that cannot allocate -----------------------
namespace {
// Part of the library image: every GPU the library runs on holds its own copy of this array, at
// its own address, until the process ends.  In host code the name is only a handle for
// hipGetSymbolAddress; all device work goes through the address that call returns.
static __device__ __align__(256) unsigned char scratch[RNN_STATIC_WORKSPACE_BYTES];
constexpr int STATIC_MAX_DEVICES = 64;
// per device: address of that GPU's copy (nullptr: not asked yet); [1]: of the large array, for windows that
// fit RNN_STATIC_WORKSPACE_BYTES but for what its limit leaves out
void* g_scratch_ptr[2][STATIC_MAX_DEVICES];
std::mutex g_scratch_mutex;
}  // namespace

int rnn_forward_static(rnn_graph* g, const float* d_weights, const float* const* d_inputs, float* const* d_outputs,
                       int32_t T, int32_t N, void* hip_stream) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (!d_outputs) return fail(RNN_ERR_INVALID_ARGUMENT, "outputs pointer is NULL");
    const Plan& P = g->plan;
    for (size_t i = 0; i < P.output_nodes.size(); ++i)
        if (!d_outputs[i]) return fail(RNN_ERR_INVALID_ARGUMENT, "an output tensor pointer is NULL");
    if (T <= 0 || N <= 0) return fail(RNN_ERR_INVALID_ARGUMENT, "T and N must be positive");
    if (g->prof.mask != 0) return fail(RNN_ERR_SEQUENCE, "kernel-class timing creates events: switch it off for rnn_forward_static");
    const int64_t total = g->layout_for(T, N).total, need = total - g->layout_for(T, N).uncounted_bytes;
    const bool large = total > (int64_t)RNN_STATIC_WORKSPACE_BYTES;
    if (need > (int64_t)RNN_STATIC_WORKSPACE_BYTES)
        return fail(RNN_ERR_WORKSPACE, "the window needs " + std::to_string(need) + " bytes of workspace, the static workspace holds " +
                                           std::to_string((int64_t)RNN_STATIC_WORKSPACE_BYTES));
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
    if (dev < 0 || dev >= STATIC_MAX_DEVICES) return fail(RNN_ERR_DEVICE, "device index beyond the static workspace table");
    void* ws = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[large][dev]) {
            // once per device, with that device current: where this GPU keeps its copy of the array
            void* p = nullptr;
            e = large ? static_large_workspace(&p) : hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
            if (e != hipSuccess || !p) return fail_hip(e, "hipGetSymbolAddress(static workspace)");
            g_scratch_ptr[large][dev] = p;
        }
        ws = g_scratch_ptr[large][dev];
    }
    g->no_alloc = true;
    const int rc = rnn_forward_range(g, d_weights, d_inputs, T, N, 0, T, ws, large ? STATIC_LARGE_BYTES : (int64_t)RNN_STATIC_WORKSPACE_BYTES, hip_stream);
    g->no_alloc = false;
    if (rc != RNN_OK) return rc;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    for (size_t i = 0; i < P.output_nodes.size(); ++i) {
        const int k = P.output_nodes[i];
        e = launch_copy(d_outputs[i], g->frame0(P.ybuf(k)), (int64_t)T * N * P.nodes[k].dim, s);
        if (e != hipSuccess) return fail_hip(e, "output copy");
    }
    return RNN_OK;
}

int rnn_set_onehot_input(rnn_graph* g, int32_t input, const int32_t* d_indices) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    const Plan& P = g->plan;
    if (input < 0 || input >= (int)P.input_nodes.size()) return fail(RNN_ERR_INVALID_ARGUMENT, "input index out of range");
    const int k = P.input_nodes[input];
    if (d_indices)
        for (const GEdge& e : P.xedges)
            if (e.src == k && e.wkind != W_FULL)
                return fail(RNN_ERR_INVALID_ARGUMENT, "a one-hot input may only have full connections");
    g->onehot.resize(P.xnodes.size(), nullptr);
    g->onehot[k] = d_indices;
    g->fwd_done = g->bptt_done = false; g->fwd_upto = 0;
    return RNN_OK;
}

int rnn_shift_window(rnn_graph* g, int32_t frames, void* hip_stream) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (!g->ws || g->fwd_upto != g->T) return fail(RNN_ERR_SEQUENCE, "rnn_shift_window needs a completely computed window");
    if (frames <= 0 || frames >= g->T) return fail(RNN_ERR_INVALID_ARGUMENT, "frames must lie in [1, T - 1]");
    const Plan& P = g->plan;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int Ti = g->Ti();
    // y(t) <- y(t + frames) for every stored frame, the history frames in front of the window
    // included: they then hold the frames right before the new window start.
    ShiftTensors st;
    st.count = 0;
    auto shift = [&](void* p, int64_t frame_words) -> hipError_t {
        st.p[st.count] = p; st.frame_words[st.count] = frame_words;
        if (++st.count < SHIFT_MAX_TENSORS) return hipSuccess;
        const hipError_t e = launch_shift_frames(st, frames, Ti, s);
        st.count = 0;
        return e;
    };
    hipError_t e = hipSuccess;
    for (size_t k = 0; k < P.xnodes.size() && e == hipSuccess; ++k) {
        const int b = P.ybuf((int)k);
        if (g->layout.buf_off[b] < 0) continue;      // an input read in place: the caller shifts it
        e = shift(g->buf(b), P.frame_floats(b, g->N));
        const int twin = P.twin_base + b;      // its tile-blocked twin
        if (e == hipSuccess && P.twin_base >= 0 && g->layout.buf_off[twin] >= 0) e = shift(g->buf(twin), P.frame_floats(twin, g->N));
    }
    for (size_t k = 0; k < P.xnodes.size() && e == hipSuccess; ++k) {
        int32_t* hist_idx = g->is_onehot((int)k) ? g->onehot_history((int)k) : nullptr;
        if (hist_idx) e = shift(hist_idx, g->N);
    }
    // interleaved exchange tensors of forward activations move along with their members
    for (const BundlePlan& bp : P.bundles)
        if (e == hipSuccess && bp.members[0] < (int)P.xnodes.size() && g->layout.buf_off[bp.ebuf] >= 0) e = shift(g->buf(bp.ebuf), P.frame_floats(bp.ebuf, g->N));
    if (e == hipSuccess) e = launch_shift_frames(st, frames, Ti, s);
    if (e != hipSuccess) return fail_hip(e, "window shift");
    g->fwd_upto = g->T - frames;
    g->fwd_done = g->bptt_done = false;
    return RNN_OK;
}

int rnn_output(const rnn_graph* g, int32_t node, const float** d_y) {
    if (!g || !d_y) return fail(RNN_ERR_INVALID_ARGUMENT, "NULL argument");
    if (node < 0 || node >= (int)g->plan.nodes.size()) return fail(RNN_ERR_INVALID_ARGUMENT, "node index out of range");
    if (!g->fwd_done) return fail(RNN_ERR_SEQUENCE, "rnn_output before rnn_forward");
    const int b = g->plan.ybuf(node);
    *d_y = g->plan.nodes[node].kind == NODE_INPUT ? g->inputs[b] : g->frame0(b);
    return RNN_OK;
}

int rnn_bptt(rnn_graph* g, const float* d_weights, const void* const* d_targets, void* hip_stream) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (!g->fwd_done) return fail(RNN_ERR_SEQUENCE, "rnn_bptt before rnn_forward");
    g->bptt_done = false;
    if (!d_weights || !d_targets) return fail(RNN_ERR_INVALID_ARGUMENT, "weights / targets pointer is NULL");
    const Plan& P = g->plan;
    for (size_t i = 0; i < P.output_nodes.size(); ++i)
        if (!d_targets[i]) return fail(RNN_ERR_INVALID_ARGUMENT, "a target tensor pointer is NULL");
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    g->weights = d_weights;
    const int T = g->T, N = g->N, H = g->hist();
    FillRanges fr;
    g->prefilled = false;
    const bool few = all_shared(g, true, H, H + T, fr);
    hipError_t e = few ? launch_fill_sentinel_and_clear(fr, nullptr, nullptr, 0, 0, reinterpret_cast<unsigned*>(g->loss_ptr()), 2,
                                                        g->ctrl_ptr() + XCD_FIELD_WORDS_FIRST, XCD_FIELD_WORDS, s)
                       : launch_fill(reinterpret_cast<float*>(g->loss_ptr()), 2, 0.0f, s);
    if (e != hipSuccess) return fail_hip(e, "loss reset");
    g->prefilled = few;
    g->xcd_fields_used = 0;
    // the output deltas of all frames first (they depend on the forward pass only)
    for (const CompPlan& cp : P.comps) {
        const int k = cp.softmax_node >= 0 ? cp.softmax_node : cp.sqerr_node;
        if (k < 0) continue;
        size_t oi = 0;
        while (oi < P.output_nodes.size() && P.output_nodes[oi] != k) ++oi;
        if (cp.softmax_node >= 0)
            e = launch_softmax_ce_delta(g->frame0(P.ybuf(k)), static_cast<const int32_t*>(d_targets[oi]), g->frame0(P.dbuf(k)), g->loss_ptr(),
                                        g->ctrl_ptr(), (int64_t)T * N, P.xnodes[k].dim, s);
        else
            e = launch_squared_error_delta(g->frame0(P.ybuf(k)), static_cast<const float*>(d_targets[oi]), g->frame0(P.dbuf(k)), g->loss_ptr(),
                                           (int64_t)T * N * P.xnodes[k].dim, P.xnodes[k].act, s);
        if (e != hipSuccess) return fail_hip(e, "output delta");
    }
    auto backward_frames = [&](int t0, int t1) -> int {
        for (int c = (int)P.comps.size() - 1; c >= 0; --c) {
            const CompPlan& cp = P.comps[c];
            if (cp.softmax_node >= 0 || cp.sqerr_node >= 0 || !cp.has_bwd_program) continue;
            if (!g->framewise && cp.chain >= 0 && P.chains[cp.chain].last == c && !g->chain_choice(cp.chain, true, N).source.empty()) {
                const ChainPlan& ch = P.chains[cp.chain];
                for (const CompPlan& m : ch.members) {
                    e = run_gemms(g, m.bwd_gemms, true, s, t0, t1);
                    if (e != hipSuccess) return fail_hip(e, "backward GEMM");
                }
                const StepRun r = run_chain(g, cp.chain, true, s, t0, t1);
                if (r.error) return fail(RNN_ERR_DEVICE, "backward: " + r.err);
                if (r.e == hipSuccess) { c = ch.first; continue; }
            }
            e = run_gemms(g, cp.bwd_gemms, true, s, t0, t1);
            if (e != hipSuccess) return fail_hip(e, "backward GEMM");
            const StepRun r = run_phases(g, c, true, s, t0, t1);
            if (r.error) return fail(RNN_ERR_DEVICE, "backward: " + r.err);
        }
        return RNN_OK;
    };
    // Errors are back-propagated through the window's own frames only (Section 2.2: while t > t0');
    // the history frames in front are read (y of earlier frames), never written.
    if (g->framewise) {
        for (int t = T - 1; t >= 0; --t) {
            const int rc = backward_frames(H + t, H + t + 1);
            if (rc != RNN_OK) return rc;
        }
    } else {
        const int rc = backward_frames(H, H + T);
        g->prefilled = false;
        if (rc != RNN_OK) return rc;
    }
    g->bptt_done = true;
    return RNN_OK;
}

int rnn_state_grad(const rnn_graph* g, int32_t node, const float** d_ds) {
    if (!g || !d_ds) return fail(RNN_ERR_INVALID_ARGUMENT, "NULL argument");
    if (node < 0 || node >= (int)g->plan.nodes.size()) return fail(RNN_ERR_INVALID_ARGUMENT, "node index out of range");
    if (g->plan.nodes[node].kind == NODE_INPUT) return fail(RNN_ERR_INVALID_ARGUMENT, "input nodes have no state gradient");
    if (!g->bptt_done) return fail(RNN_ERR_SEQUENCE, "rnn_state_grad before rnn_bptt");
    *d_ds = g->frame0(g->plan.dbuf(node));
    return RNN_OK;
}

int rnn_grads(rnn_graph* g, float* d_grads, double* loss, void* hip_stream) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (!g->bptt_done) return fail(RNN_ERR_SEQUENCE, "rnn_grads before rnn_bptt");
    if (!d_grads) return fail(RNN_ERR_INVALID_ARGUMENT, "gradient pointer is NULL");
    const Plan& P = g->plan;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    const int T = g->T, N = g->N, H = g->hist();
    const int64_t F = (int64_t)T * N;      // the window's own frames: the sums run over t0' < t <= t1

    // Weight-gradient GEMMs: the contraction runs over frames, its parts x tiles in one row of workgroups.  A block that one
    // unsplit product writes is stored, not added to zeros: blocks of at least OWN_MIN floats are
    // left out of the zero fill (smaller ones are not worth another fill launch for what lies between them).
    // Filling and adding moved each such block twice more.  This call with blocks from 1 / 2^18 / 2^20 / 2^22 / 2^24 floats
    // on stored, and with none, us: 1 x 1024 LSTM (blocks of 2^20), N = 64 443 / 419 / 418 / 418 / 418 / 419; 1 x 2048, N = 16
    // 429 / 406 / 409 / 408 / 414 / 415; 1 x 4096, N = 16 754 / 719 / 724 / 724 / 726 / 808; Elman 38,000-512-20,000
    // 354 / 340 / 330 / 330 / 330 / 340.
    constexpr int64_t OWN_MIN = 1 << 20;
    std::vector<std::pair<int64_t, int64_t>>& owned = g->grad_owned;
    owned.clear();
    auto own = [&](int64_t off, int64_t len) { if (len >= OWN_MIN) owned.emplace_back(off, len); };
    auto in_rows = [&](const GradGemmPlan& gg) {
        const int64_t rows = g->onehot_history(gg.src_buf) ? F : F - (int64_t)gg.delay * N;
        return !g->deterministic && rows > 0 && onehot_grad_in_rows(gg.n_dst, gg.n_src, rows) && gg.sole;
    };
    std::vector<GemmGroup>& groups = g->grad_groups;
    groups.clear();
    int64_t tiles = 0, n_launch = 0;
    int since = 0;      // first problem of the current eight
    // Eight products together have at least as many parts as make 1,024 workgroups of 128 x 128 (and 128 frames each).
    auto eight = [&]() {
        GemmGroup& grp = groups.back();
        for (int i = since; i < grp.n_problems; ++i)
            grp.p[i].min_split = (int)std::max<int64_t>(1, std::min<int64_t>((1024 + tiles - 1) / tiles, (F + 127) / 128));
        since = grp.n_problems; tiles = 0;
    };
    for (const GradGemmPlan& gg : P.grad_gemms) {
        if (g->is_onehot(gg.src_buf)) {
            if (in_rows(gg)) own(gg.w_off, (int64_t)gg.n_dst * gg.n_src);
            continue;
        }
        if (groups.empty() || groups.back().n_problems == GEMM_MAX_PROBLEMS) {
            groups.emplace_back();
            groups.back().n_problems = groups.back().n_pairs = since = 0;
        }
        GemmGroup& grp = groups.back();
        GemmProblem& gp = grp.p[grp.n_problems++];
        gp.C = d_grads + gg.w_off; gp.ldc = gg.n_src; gp.M = gp.window_M = gg.n_dst; gp.N = gg.n_src;
        gp.first_pair = grp.n_pairs; gp.n_pairs = 1; gp.accumulate = gg.sole ? 0 : 1;      // where several connections share a block all add
        GemmPair& o = grp.pair[grp.n_pairs++];
        // eps_m(t) of every frame of the window against y_src(t - d); for the window's first d
        // frames that is a history frame (the real activation of a frame before the window)
        o.A = g->frame0(gg.dst_buf); o.lda = gg.n_dst;
        o.B = g->frame0(gg.src_buf) - (int64_t)gg.delay * N * gg.n_src; o.ldb = gg.n_src; o.K = (int)F; o.a_row_off = 0; o.a_rows = (int)F;
        tiles += (int64_t)((gg.n_dst + 127) / 128) * ((gg.n_src + 127) / 128);
        if (grp.n_problems - since == 8) eight();
    }
    for (GemmGroup& grp : groups) {
        if (&grp == &groups.back() && tiles > 0) eight();
        plan_gemm_group(GEMM_TN, grp, g->deterministic);
        for (int i = 0; i < grp.n_problems; ++i)
            if (grp.p[i].split == 1 && !grp.p[i].accumulate) own(grp.p[i].C - d_grads, (int64_t)grp.p[i].M * grp.p[i].N);
    }

    hipError_t e = hipSuccess;
    std::sort(owned.begin(), owned.end());
    int64_t filled = 0;
    for (const auto& o : owned) {
        e = launch_fill(d_grads + filled, o.first - filled, 0.0f, s);
        if (e != hipSuccess) return fail_hip(e, "gradient reset");
        filled = o.first + o.second;
    }
    e = launch_fill(d_grads + filled, P.n_params - filled, 0.0f, s);
    if (e != hipSuccess) return fail_hip(e, "gradient reset");

    const int prof = g->prof.begin(RNN_PROF_GEMM_GRAD, s);
    for (const GradGemmPlan& gg : P.grad_gemms) {
        if (!g->is_onehot(gg.src_buf)) continue;      // scatter-add instead of a GEMM over a one-hot matrix
        // with history: every frame of the window against the class of frame t - d, which may lie in the history
        const int32_t* hist_idx = g->onehot_history(gg.src_buf);
        const int32_t* idx = hist_idx ? hist_idx + (int64_t)(H - gg.delay) * N : g->onehot[gg.src_buf];
        const int64_t shift = hist_idx ? 0 : (int64_t)gg.delay * N;
        if (F - shift <= 0) continue;
        if (in_rows(gg)) e = launch_onehot_grad_rows(d_grads + gg.w_off, g->frame0(gg.dst_buf), idx, gg.n_dst, gg.n_src, shift, F, s);
        else e = launch_onehot_scatter(d_grads + gg.w_off, g->frame0(gg.dst_buf), idx, gg.n_dst, gg.n_src, shift, F, g->deterministic, s);
        if (e != hipSuccess) return fail_hip(e, "one-hot weight gradient");
        ++n_launch;
    }
    for (const GemmGroup& gr : groups) {
        e = launch_gemm_group(GEMM_TN, gr, s);
        if (e != hipSuccess) return fail_hip(e, "gradient GEMM");
        ++n_launch;
    }
    g->prof.end(prof, n_launch, s);
    e = launch_colsum(g->view(), P.colsum_off, P.n_colsum, P.colsum_max_dim, g->weights, d_grads, H + T, N, H, g->deterministic, s);
    if (e != hipSuccess) return fail_hip(e, "diagonal / bias gradient");
    if (loss) return read_control(g, loss, s);
    return RNN_OK;
}

int rnn_set_deterministic(rnn_graph* g, int32_t on) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    g->deterministic = on != 0;
    return RNN_OK;
}

int rnn_check(rnn_graph* g, void* hip_stream) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (!g->ws) return fail(RNN_ERR_SEQUENCE, "no window yet");
    return read_control(g, nullptr, static_cast<hipStream_t>(hip_stream));
}

int rnn_step_build(const rnn_graph* g, int32_t node, int32_t backward, int32_t* build) {
    if (!g || !build) return fail(RNN_ERR_INVALID_ARGUMENT, "NULL argument");
    if (node < 0 || node >= (int)g->plan.nodes.size()) return fail(RNN_ERR_INVALID_ARGUMENT, "node index out of range");
    const int c = g->plan.xsched.node_comp[node];
    *build = g->plan.comps[c].recurrent ? g->served[c][backward ? 1 : 0] : RNN_BUILD_NONE;
    return RNN_OK;
}

int rnn_specialise(rnn_graph* g, int32_t N) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (N <= 0) return fail(RNN_ERR_INVALID_ARGUMENT, "N must be positive");
    if (!g->use_jit || !jit_available()) return 0;
    int n = 0;
    for (size_t c = 0; c < g->plan.comps.size(); ++c) {
        const CompPlan& cp = g->plan.comps[c];
        if (!cp.recurrent) continue;
        for (int backward = 0; backward < 2; ++backward) {
            if (backward ? !cp.has_bwd_program : !cp.has_fwd_program) continue;
            std::string log;
            const rnn_graph::JitChoice& jc = g->jit_choice((int)c, backward != 0, N);
            if (jc.source.empty()) continue;
            if (!jit_compile(jc.source, &log))
                return fail(RNN_ERR_DEVICE, "step kernel specialisation failed: " + log);
            ++n;
        }
    }
    for (size_t ci = 0; ci < g->plan.chains.size(); ++ci)
        for (int backward = 0; backward < 2; ++backward) {
            const rnn_graph::ChainChoice& cc = g->chain_choice((int)ci, backward != 0, N);
            if (cc.source.empty()) continue;
            std::string log;
            if (!jit_compile(cc.source, &log))
                return fail(RNN_ERR_DEVICE, "chain step kernel specialisation failed: " + log);
            ++n;
        }
    return n;
}

int rnn_plan_work(const rnn_graph* g, int32_t T, int32_t N, int64_t* flops, int64_t* step_bytes) {
    if (!g || !flops || !step_bytes) return fail(RNN_ERR_INVALID_ARGUMENT, "NULL argument");
    if (T <= 0 || N <= 0) return fail(RNN_ERR_INVALID_ARGUMENT, "T and N must be positive");
    const Plan& P = g->plan;
    const int64_t F = (int64_t)T * N;
    for (int i = 0; i < 5; ++i) flops[i] = 0;
    step_bytes[0] = step_bytes[1] = 0;
    // diagonal weights inside recurrent nodes (peepholes) are touched once per step as well
    std::vector<int64_t> diag(P.comps.size(), 0);
    for (size_t m = 0; m < P.xedges.size(); ++m)
        if (P.xedges[m].wkind == W_DIAG && P.xsched.edge_class[m] != EDGE_BATCHED)
            diag[P.xsched.node_comp[P.xedges[m].dst]] += P.xnodes[P.xedges[m].dst].dim;
    for (size_t c = 0; c < P.comps.size(); ++c) {
        for (int d = 0; d < 2; ++d) {
            // the lowering that ran: as a member of a chain launch, or on its own
            const CompPlan* cp = &P.comps[c];
            if (cp->chain >= 0 && (g->served[c][d] & RNN_BUILD_CHAIN)) cp = &P.chains[cp->chain].members[c - P.chains[cp->chain].first];
            for (const GemmProblemPlan& gp : d ? cp->bwd_gemms : cp->fwd_gemms)
                for (const GemmPairPlan& pr : gp.pairs)
                    if (!g->is_onehot(pr.a_buf)) flops[d] += 2 * (int64_t)gp.n * pr.k_len * F;
            if (cp->recurrent) {
                flops[3 + d] += 2 * cp->step_weight_floats * F;
                step_bytes[d] += 4 * (cp->step_weight_floats + diag[c]);
            }
        }
    }
    for (const GradGemmPlan& gg : P.grad_gemms)
        if (!g->is_onehot(gg.src_buf)) flops[2] += 2 * (int64_t)gg.n_dst * gg.n_src * F;
    return RNN_OK;
}

int rnn_debug_read_control(rnn_graph* g, void* out, int32_t bytes) {
    if (!g || !out) return fail(RNN_ERR_INVALID_ARGUMENT, "NULL argument");
    if (!g->ws) return fail(RNN_ERR_SEQUENCE, "no window yet");
    if (bytes <= 0 || bytes > (int32_t)SYNC_BYTES) return fail(RNN_ERR_INVALID_ARGUMENT, "at most 1024 bytes");
    hipError_t e = hipDeviceSynchronize();
    if (e == hipSuccess) e = hipMemcpy(out, g->ws + g->layout.sync_off, (size_t)bytes, hipMemcpyDeviceToHost);
    if (e != hipSuccess) return fail_hip(e, "control word read-back");
    return RNN_OK;
}

int rnn_profile_enable(rnn_graph* g, int32_t class_mask) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    g->prof.mask = class_mask & ((1 << RNN_PROF_CLASSES) - 1);
    return RNN_OK;
}

int rnn_profile_read(rnn_graph* g, int32_t cls, double* ms, int64_t* launches) {
    if (!g) return fail(RNN_ERR_INVALID_ARGUMENT, "graph is NULL");
    if (cls < 0 || cls >= RNN_PROF_CLASSES) return fail(RNN_ERR_INVALID_ARGUMENT, "unknown kernel class");
    double total = 0.0; int64_t n = 0;
    std::vector<Profiler::Rec> keep;
    for (Profiler::Rec& r : g->prof.recs) {
        if (r.cls != cls) { keep.push_back(r); continue; }
        hipError_t e = hipEventSynchronize(r.b);
        float t = 0.0f;
        if (e == hipSuccess) e = hipEventElapsedTime(&t, r.a, r.b);
        g->prof.pool.push_back(r.a); g->prof.pool.push_back(r.b);
        if (e != hipSuccess) { g->prof.recs.swap(keep); return fail_hip(e, "event read"); }
        total += t; n += r.launches;
    }
    g->prof.recs.swap(keep);
    if (ms) *ms = total;
    if (launches) *launches = n;
    return RNN_OK;
}

}  // extern "C"
