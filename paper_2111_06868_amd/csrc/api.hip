// extern "C" entry points declared in include/sv.h: states, gates, fusion,
// circuits, reductions, adjoint gradients and timing.
#include <hip/hip_runtime.h>

#include <atomic>
#include <fstream>
#include <mutex>
#include <string>
#include <thread>
#include <unordered_map>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>

#include "runtime.h"

namespace sv {
const char *last_error_cstr();
int stats_enable(int on);
int stats_reset();
int stats_query(int cls, int64_t *launches, double *total_ms);
}  // namespace sv

using namespace sv;

namespace {

constexpr int kVersion = 1;

size_t amp_bytes(int dtype) { return dtype == SV_C64 ? 8 : 16; }

int check_state(const sv_state *s)
{
    if (!s) return fail(SV_ERR_ARG, "NULL state handle");
    return SV_OK;
}

int select_device(const sv_state *s)
{
    SV_HIP(hipSetDevice(s->device));
    return SV_OK;
}

// Make `to` wait for the work already enqueued on `from`.
int stream_after(hipStream_t to, hipStream_t from)
{
    if (to == from) return SV_OK;
    hipEvent_t e;
    SV_HIP(hipEventCreateWithFlags(&e, hipEventDisableTiming));
    SV_HIP(hipEventRecord(e, from));
    SV_HIP(hipStreamWaitEvent(to, e, 0));
    SV_HIP(hipEventDestroy(e));
    return SV_OK;
}

int check_precision(const sv_state *s, int precision)
{
    if (precision < SV_PREC_FP32 || precision > SV_PREC_SPLIT_BF16X3) return fail(SV_ERR_ARG, "unknown precision %d", precision);
    if ((s->dtype == SV_C128) != (precision == SV_PREC_FP64))
        return fail(SV_ERR_ARG, "precision %d does not match the state's amplitude type", precision);
    return SV_OK;
}

int validate_gates(const sv_gate *g, int G, int n)
{
    if (G < 0) return fail(SV_ERR_ARG, "negative gate count");
    if (G > 0 && !g) return fail(SV_ERR_ARG, "NULL gate array");
    for (int i = 0; i < G; ++i) {
        int rc = check_gate_shape(g[i]);
        if (!rc) rc = check_gate_qubits(g[i], n);
        if (rc) {
            std::string msg = std::string("gate ") + std::to_string(i) + ": " + last_error_cstr();
            return fail(rc, "%s", msg.c_str());
        }
    }
    return SV_OK;
}

// Upload `bytes` staged bytes and enqueue `launches`; the arena and staging
// buffers are reused only after the previous user of the arena finished.
int run_launches(sv_state *s, std::vector<Launch> &launches, bool use_graph)
{
    SV_HIP(hipEventSynchronize(s->arena_free));
    const size_t bytes = pack_operands(launches, s->dtype, s->stage);
    if (bytes == size_t(-1)) return fail(SV_ERR_HIP, "pinned staging allocation failed");
    if (bytes) {
        SV_HIP(s->arena.ensure(bytes));
        SV_HIP(hipMemcpyAsync(s->arena.p, s->stage.p, bytes, hipMemcpyHostToDevice, s->stream));
    }
    if (!use_graph) {
        int rc = enqueue(launches, s->dtype, s->buf, s->n, s->arena.p, s->stream);
        SV_HIP(hipEventRecord(s->arena_free, s->stream));
        return rc;
    }
    // Capture the launches, then reuse the state's instantiated graph when the
    // new one has the same topology (hipGraphExecUpdate takes the new kernel
    // arguments: matrices, operand addresses), else instantiate anew.  The
    // previous launch of that graph has finished: arena_free was synchronised.
    if (!s->capture_stream) SV_HIP(hipStreamCreateWithFlags(&s->capture_stream, hipStreamNonBlocking));
    hipGraph_t graph = nullptr;
    SV_HIP(hipStreamBeginCapture(s->capture_stream, hipStreamCaptureModeThreadLocal));
    timing_suspend(true);
    int rc = enqueue(launches, s->dtype, s->buf, s->n, s->arena.p, s->capture_stream);
    timing_suspend(false);
    hipError_t e = hipStreamEndCapture(s->capture_stream, &graph);
    if (rc) {
        if (graph) (void)hipGraphDestroy(graph);
        return rc;
    }
    if (e != hipSuccess) return fail(SV_ERR_HIP, "graph capture: %s", hipGetErrorString(e));
    bool updated = false;
    if (s->graph_exec) {
        hipGraphNode_t bad = nullptr;
        hipGraphExecUpdateResult res = hipGraphExecUpdateError;
        updated = hipGraphExecUpdate(s->graph_exec, graph, &bad, &res) == hipSuccess && res == hipGraphExecUpdateSuccess;
        if (!updated) {
            (void)hipGetLastError();  // a refused update is not an error of this call
            (void)hipGraphExecDestroy(s->graph_exec);
            s->graph_exec = nullptr;
        }
    }
    if (!updated) e = hipGraphInstantiate(&s->graph_exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e == hipSuccess) e = hipGraphLaunch(s->graph_exec, s->stream);
    if (e == hipSuccess) e = hipEventRecord(s->arena_free, s->stream);
    if (e != hipSuccess) {
        if (s->graph_exec) (void)hipGraphExecDestroy(s->graph_exec);
        s->graph_exec = nullptr;
        return fail(SV_ERR_HIP, "graph launch: %s", hipGetErrorString(e));
    }
    ++s->graph_launches;
    if (updated) ++s->graph_updates;
    return SV_OK;
}

int blocks_to_launches(const std::vector<Block> &blocks, const sv_state *s, int precision, int rule,
                       std::vector<Launch> &out, bool own_blocks = false)
{
    if (rule == SV_RULE_TILED) {
        group_tile_passes(blocks, s->n, precision, out);
        return SV_OK;
    }
    out.clear();
    out.reserve(blocks.size());
    for (const auto &b : blocks) {
        Launch L;
        L.k = b.k;
        std::copy(b.q, b.q + SV_MAX_K, L.q);
        L.path = choose_path(s->dtype, precision, b.k, b.q, s->n);
        L.m = b.m;
        out.push_back(std::move(L));
    }
    if (own_blocks) return SV_OK;
    if (int rc = group_dense_passes(out, s->n, precision)) return rc;
    return group_gate_passes(out, s->n, s->dtype);
}

// Dense blocks of four and more qubits cost a pass over the state each.  In FP32
// and FP64 a plan that has some runs as tile passes of the same gates instead
// (in an order that keeps every qubit's own), where those are priced lower.
// Eight cycles on a two-row ladder, k = 4, dense blocks against tile passes:
// FP32 139 to 113 us at 14 qubits, 280 to 191 at 20 and 1316 to 627 at 24, FP64
// 496 to 132, 802 to 240 and 3520 to 1491, so from the smallest state a tile
// takes.
// The 16-bit splits keep their blocks (group_dense_passes for FP16), since they
// round the state once a block, and blocks of at most three qubits share passes as they
// are (group_gate_passes).
bool takes_tiles(int rule, int precision, int n)
{
    return (rule == SV_RULE_PAPER || rule == SV_RULE_ENHANCED) && n >= tile_min_qubits(precision) &&
           (precision == SV_PREC_FP32 || precision == SV_PREC_SPLIT_BF16X3 || precision == SV_PREC_FP64);
}
bool tiles_are_cheaper(const std::vector<Block> &blocks, const std::vector<Block> &tiled, int n, int precision)
{
    const CostTable cost = lookup_costs(n, precision, nullptr);
    return tiled_plan_cost(tiled, n, precision, cost) < plan_cost(blocks, cost) - 1e-12;
}
// Whether a plan has blocks that tile passes would replace, and no gate that
// is wider than theirs.
bool may_be_tiles(const sv_gate *g, int G, const std::vector<Block> &blocks)
{
    bool wide = false;
    for (const auto &b : blocks) wide = wide || b.k >= 4;
    for (int i = 0; i < G; ++i) wide = wide && g[i].k <= 4;
    return wide;
}
// The tile passes of the gates of a plan (positions and members, no matrices),
// or none where they are ruled out.
int gates_as_tiles(const sv_gate *g, int G, int n, int precision, const std::vector<Block> &blocks,
                   std::vector<Block> &tiled)
{
    tiled.clear();
    if (!may_be_tiles(g, G, blocks)) return SV_OK;
    return fuse_gates(g, G, n, 4, SV_RULE_TILED, default_costs(), tiled, false, precision);
}
// The tile passes of a kept plan's gates, once for all threads that apply it:
// a program that only reads a plan does not pay for them.
int plan_tiles(const sv_plan *p)
{
    std::call_once(p->tiles_formed, [p] {
        p->tiles_rc = fuse_gates(p->gates.data(), int(p->gates.size()), p->n, 4, SV_RULE_TILED, default_costs(), p->tiled,
                                 true, p->precision);
    });
    return p->tiles_rc;
}

int choose_plan_uncached(const sv_gate *g, int G, int n, int dtype, int precision, int rule, int max_k, bool found,
                         const CostTable &cost, int kmin, int kcap, int *out_rule, int *out_k);

// Resolve (rule, max_k) requests: max_k = -1 picks k by the cost table;
// SV_RULE_AUTO also picks between the enhanced and the tiled plan.  Candidate
// plans are priced on block positions only (no matrices are formed).
int choose_plan(const sv_gate *g, int G, int n, int dtype, int precision, int rule, int max_k, int *out_rule,
                int *out_k)
{
    bool found = false;
    const CostTable cost = lookup_costs(n, precision, &found);
    int kmin = 1;
    for (int i = 0; i < G; ++i) kmin = std::max(kmin, g[i].k);
    const int kcap = max_k > 0 ? max_k : SV_MAX_K;
    if (max_k > 0 && rule != SV_RULE_AUTO) {
        *out_rule = rule;
        *out_k = max_k;
        return SV_OK;
    }
    // The choice depends on the gates' positions and the cost table only, so
    // it is remembered per circuit structure (a circuit re-run with new
    // angles is not re-priced).  A stale or colliding entry can only name
    // another valid (rule, k), and one below the widest gate is recomputed.
    uint64_t key = 1469598103934665603ull;
    auto mix = [&key](uint64_t v) { key = (key ^ v) * 1099511628211ull; };
    mix(uint64_t(n));
    mix(uint64_t(dtype));
    mix(uint64_t(precision));
    mix(uint64_t(rule));
    mix(uint64_t(max_k + 8));
    mix(cost_version());
    mix(uint64_t(tile_union_limit()));
    mix(uint64_t(tile_pass_bits(precision)) | uint64_t(tile_pass_capacity(precision)) << 8);
    mix(uint64_t(G));
    for (int i = 0; i < G; ++i) {
        mix(uint64_t(g[i].kind) | uint64_t(g[i].k) << 8);
        for (int j = 0; j < g[i].k; ++j) mix(uint64_t(g[i].q[j]));
    }
    static std::mutex memo_mu;
    static std::unordered_map<uint64_t, std::pair<int, int>> memo;
    {
        std::lock_guard<std::mutex> lk(memo_mu);
        auto it = memo.find(key);
        if (it != memo.end() && it->second.second >= kmin) {
            *out_rule = it->second.first;
            *out_k = it->second.second;
            return SV_OK;
        }
    }
    const int rc = choose_plan_uncached(g, G, n, dtype, precision, rule, max_k, found, cost, kmin, kcap, out_rule,
                                        out_k);
    if (!rc) {
        std::lock_guard<std::mutex> lk(memo_mu);
        if (memo.size() > 4096) memo.clear();
        memo[key] = {*out_rule, *out_k};
    }
    return rc;
}

int choose_plan_uncached(const sv_gate *g, int G, int n, int dtype, int precision, int rule, int max_k, bool found,
                         const CostTable &cost, int kmin, int kcap, int *out_rule, int *out_k)
{
    std::vector<int> rules;
    if (rule == SV_RULE_AUTO) {
        rules.push_back(SV_RULE_ENHANCED);
        if (n >= tile_min_qubits(precision)) rules.push_back(SV_RULE_TILED);
    } else {
        rules.push_back(rule == SV_RULE_NONE ? SV_RULE_PAPER : rule);
    }
    double best = 1e300;
    int best_rule = rules[0], best_k = std::min(kmin, kcap);
    for (int r : rules) {
        const int khi = std::min(kcap, r == SV_RULE_TILED ? 4 : SV_MAX_K);
        for (int k = kmin; k <= khi; ++k) {
            if (!found && k == SV_MAX_K) break;  // untuned: stay below the MFMA-bound size
            std::vector<Block> blocks;
            if (int rc = fuse_gates(g, G, n, k, r, cost, blocks, false, precision)) return rc;
            const double c = r == SV_RULE_TILED ? tiled_plan_cost(blocks, n, precision, cost) : plan_cost(blocks, cost);
            if (c < best - 1e-12) {
                best = c;
                best_rule = r;
                best_k = k;
            }
        }
    }
    *out_rule = rule == SV_RULE_NONE ? SV_RULE_NONE : best_rule;
    *out_k = best_k;
    return SV_OK;
}

int pauli_tables(sv_state *s, const sv_pauli_sum *H, int n, PauliUse use, dev::PauliDev &P);

}  // namespace

// ============================================================== misc
extern "C" const char *sv_last_error(void) { return last_error_cstr(); }
extern "C" int sv_version(void) { return kVersion; }

// ============================================================== states
extern "C" int sv_alloc(int n, int dtype, void *dev_buf, size_t bytes, void *hip_stream, sv_state **out)
{
    clear_error();
    if (!out) return fail(SV_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (dtype != SV_C64 && dtype != SV_C128) return fail(SV_ERR_ARG, "unknown amplitude type %d", dtype);
    const int nmax = dtype == SV_C64 ? SV_MAX_QUBITS_C64 : SV_MAX_QUBITS_C128;
    if (n < 1 || n > nmax) return fail(SV_ERR_ARG, "n = %d outside 1..%d", n, nmax);
    const size_t need = (size_t(1) << n) * amp_bytes(dtype);
    if (dev_buf) {
        if (bytes < need) return fail(SV_ERR_SIZE, "buffer of %zu bytes < %zu needed for %d qubits", bytes, need, n);
        if (reinterpret_cast<uintptr_t>(dev_buf) % 256) return fail(SV_ERR_ARG, "device buffer not 256-byte aligned");
    }
    sv_state *s = new sv_state;
    s->n = n;
    s->dtype = dtype;
    s->stream = static_cast<hipStream_t>(hip_stream);
    hipError_t e = hipGetDevice(&s->device);
    if (e == hipSuccess) e = hipEventCreateWithFlags(&s->arena_free, hipEventDisableTiming);
    if (e == hipSuccess && !dev_buf) {
        e = hipMalloc(&s->buf, need);
        s->owns = e == hipSuccess;
        s->bytes = need;
    } else {
        s->buf = dev_buf;
        s->bytes = bytes;
    }
    if (e == hipSuccess) e = s->red.ensure(sizeof(double) * (2 * dev::kRedBlocks + 64));
    if (e == hipSuccess) e = s->red_host.ensure(sizeof(double) * 64);
    if (e == hipSuccess) e = dev::launch_fill_basis(dtype, s->buf, n, 0, s->stream);
    if (e != hipSuccess) {
        int rc = fail(SV_ERR_HIP, "sv_alloc: %s", hipGetErrorString(e));
        sv_free(s);
        return rc;
    }
    // the first state of the process installs a saved tuning cache, if any
    static std::once_flag cache_once;
    std::call_once(cache_once, [&] {
        const char *path = std::getenv("SV_TUNE_CACHE");
        if (path && *path && std::ifstream(path).good()) (void)load_tuning(path, s->device, nullptr);
        clear_error();
    });
    *out = s;
    return SV_OK;
}

extern "C" int sv_free(sv_state *s)
{
    if (!s) return SV_OK;
    (void)hipSetDevice(s->device);
    (void)hipStreamSynchronize(s->stream);
    if (s->owns && s->buf) (void)hipFree(s->buf);
    if (s->graph_exec) (void)hipGraphExecDestroy(s->graph_exec);
    if (s->capture_stream) (void)hipStreamDestroy(s->capture_stream);
    if (s->arena_free) (void)hipEventDestroy(s->arena_free);
    delete s;
    return SV_OK;
}

extern "C" int sv_info(const sv_state *s, int *n, int *dtype, void **dev_ptr)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (n) *n = s->n;
    if (dtype) *dtype = s->dtype;
    if (dev_ptr) *dev_ptr = s->buf;
    return SV_OK;
}

extern "C" int sv_set_product(sv_state *s, const char *tokens)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (!tokens) return fail(SV_ERR_ARG, "NULL tokens");
    const size_t len = std::strlen(tokens);
    if (len != 1 && len != size_t(s->n))
        return fail(SV_ERR_ARG, "initial state needs 1 or %d tokens, got %zu", s->n, len);
    double amps[4 * SV_MAX_QUBITS_C64];
    const double r = 0.70710678118654752440;
    for (int j = 0; j < s->n; ++j) {
        const char c = len == 1 ? tokens[0] : tokens[j];
        const int p = s->n - 1 - j;  // token j describes position n-1-j
        double *a = amps + 4 * p;
        switch (c) {
        case '0': a[0] = 1; a[1] = 0; a[2] = 0; a[3] = 0; break;
        case '1': a[0] = 0; a[1] = 0; a[2] = 1; a[3] = 0; break;
        case '+': a[0] = r; a[1] = 0; a[2] = r; a[3] = 0; break;
        case '-': a[0] = r; a[1] = 0; a[2] = -r; a[3] = 0; break;
        default: return fail(SV_ERR_ARG, "initial-state token '%c' is not one of 0 1 + -", c);
        }
    }
    if (int rc = select_device(s)) return rc;
    SV_HIP(dev::launch_product(s->dtype, s->buf, s->n, amps, s->stream));
    return SV_OK;
}

extern "C" int sv_set_basis(sv_state *s, uint64_t index)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (index >> s->n) return fail(SV_ERR_ARG, "basis index %llu >= 2^%d", (unsigned long long)index, s->n);
    if (int rc = select_device(s)) return rc;
    SV_HIP(dev::launch_fill_basis(s->dtype, s->buf, s->n, index, s->stream));
    return SV_OK;
}

extern "C" int sv_read(sv_state *s, uint64_t first, uint64_t count, void *host)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    const uint64_t N = uint64_t(1) << s->n;
    if (first > N || count > N - first) return fail(SV_ERR_ARG, "range [%llu, +%llu) outside the state", (unsigned long long)first, (unsigned long long)count);
    if (count && !host) return fail(SV_ERR_ARG, "NULL host buffer");
    if (int rc = select_device(s)) return rc;
    const size_t ab = amp_bytes(s->dtype);
    if (count) SV_HIP(hipMemcpyAsync(host, static_cast<char *>(s->buf) + first * ab, count * ab, hipMemcpyDeviceToHost, s->stream));
    SV_HIP(hipStreamSynchronize(s->stream));
    return SV_OK;
}

extern "C" int sv_write(sv_state *s, uint64_t first, uint64_t count, const void *host)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    const uint64_t N = uint64_t(1) << s->n;
    if (first > N || count > N - first) return fail(SV_ERR_ARG, "range outside the state");
    if (count && !host) return fail(SV_ERR_ARG, "NULL host buffer");
    if (int rc = select_device(s)) return rc;
    const size_t ab = amp_bytes(s->dtype);
    if (count) SV_HIP(hipMemcpyAsync(static_cast<char *>(s->buf) + first * ab, host, count * ab, hipMemcpyHostToDevice, s->stream));
    SV_HIP(hipStreamSynchronize(s->stream));
    return SV_OK;
}

extern "C" int sv_copy(sv_state *dst, sv_state *src)
{
    clear_error();
    if (!dst || !src) return fail(SV_ERR_ARG, "NULL state handle");
    if (dst->n != src->n) return fail(SV_ERR_ARG, "qubit counts differ (%d vs %d)", dst->n, src->n);
    if (int rc = select_device(dst)) return rc;
    if (int rc = stream_after(dst->stream, src->stream)) return rc;
    SV_HIP(dev::launch_convert(src->dtype, src->buf, dst->dtype, dst->buf, uint64_t(1) << dst->n, dst->stream));
    return SV_OK;
}

extern "C" int sv_synchronize(sv_state *s)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (int rc = select_device(s)) return rc;
    SV_HIP(hipStreamSynchronize(s->stream));
    return SV_OK;
}

// ============================================================== gates
extern "C" int sv_gate_matrix(const sv_gate *g, double *out)
{
    clear_error();
    if (!g || !out) return fail(SV_ERR_ARG, "NULL argument");
    std::vector<cd> m;
    if (int rc = gate_matrix_abi(*g, m)) return rc;
    for (size_t i = 0; i < m.size(); ++i) {
        out[2 * i] = m[i].real();
        out[2 * i + 1] = m[i].imag();
    }
    return SV_OK;
}

namespace {
int apply_gate_impl(sv_state *s, const sv_gate *g);
}

extern "C" int sv_apply_gate(sv_state *s, const sv_gate *g)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (int rc = validate_gates(g, 1, s->n)) return rc;
    return apply_gate_impl(s, g);
}

namespace {
int apply_gate_impl(sv_state *s, const sv_gate *g)
{
    Launch L;
    L.k = g->k;
    int sq[SV_MAX_K];
    if (int rc = gate_matrix_canonical(*g, L.m, sq)) return rc;
    std::fill(L.q, L.q + SV_MAX_K, 0);
    std::copy(sq, sq + g->k, L.q);
    const int prec = s->dtype == SV_C64 ? SV_PREC_FP32 : SV_PREC_FP64;
    L.path = choose_path(s->dtype, prec, L.k, L.q, s->n);
    std::vector<Launch> v;
    v.push_back(std::move(L));
    if (int rc = select_device(s)) return rc;
    return run_launches(s, v, false);
}
}  // namespace

// ============================================================== fusion
namespace {

// precision < 0: FP32 cost tables, tile passes sized for operands of any precision
int fuse_plan(const sv_gate *g, int G, int n, int max_k, int rule, int precision, sv_plan **out)
{
    if (!out) return fail(SV_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (n < 1 || n > SV_MAX_QUBITS_C64) return fail(SV_ERR_ARG, "n = %d outside 1..%d", n, SV_MAX_QUBITS_C64);
    if (precision < -1 || precision > SV_PREC_SPLIT_BF16X3) return fail(SV_ERR_ARG, "precision %d", precision);
    if (int rc = validate_gates(g, G, n)) return rc;
    if (rule < SV_RULE_PAPER || rule > SV_RULE_AUTO) return fail(SV_ERR_ARG, "unknown fusion rule %d", rule);
    const int cost_prec = precision < 0 ? SV_PREC_FP32 : precision;
    if (max_k == -1 || rule == SV_RULE_AUTO) {
        if (max_k != -1 && (max_k < 1 || max_k > SV_MAX_K)) return fail(SV_ERR_ARG, "max_k %d", max_k);
        if (int rc = choose_plan(g, G, n, SV_C64, cost_prec, rule, max_k, &rule, &max_k)) return rc;
    }
    auto *p = new sv_plan;
    p->n = n;
    p->max_k = max_k;
    p->rule = rule;
    int rc = fuse_gates(g, G, n, max_k, rule, lookup_costs(n, cost_prec, nullptr), p->blocks, true, precision);
    if (rc) {
        delete p;
        return rc;
    }
    p->precision = precision;
    if (takes_tiles(rule, cost_prec, n) && may_be_tiles(g, G, p->blocks)) {
        p->gates.assign(g, g + G);
        size_t at = 0;
        for (int i = 0; i < G; ++i)
            if (g[i].kind == SV_G_MATRIX) at += size_t(2) << (2 * g[i].k);
        p->matrices.resize(at);
        at = 0;
        for (sv_gate &x : p->gates)
            if (x.kind == SV_G_MATRIX) {
                const size_t count = size_t(2) << (2 * x.k);
                x.m = static_cast<const double *>(std::memcpy(p->matrices.data() + at, x.m, count * sizeof(double)));
                at += count;
            }
    }
    *out = p;
    return SV_OK;
}

}  // namespace

extern "C" int sv_fuse(const sv_gate *g, int G, int n, int max_k, int rule, sv_plan **out)
{
    clear_error();
    return fuse_plan(g, G, n, max_k, rule, -1, out);
}

extern "C" int sv_fuse_prec(const sv_gate *g, int G, int n, int max_k, int rule, int precision, sv_plan **out)
{
    clear_error();
    if (precision < 0) return fail(SV_ERR_ARG, "precision %d", precision);
    return fuse_plan(g, G, n, max_k, rule, precision, out);
}

extern "C" int sv_plan_free(sv_plan *p)
{
    delete p;
    return SV_OK;
}

extern "C" int sv_plan_num_blocks(const sv_plan *p, int *out)
{
    clear_error();
    if (!p || !out) return fail(SV_ERR_ARG, "NULL argument");
    *out = int(p->blocks.size());
    return SV_OK;
}

extern "C" int sv_plan_max_k(const sv_plan *p, int *out)
{
    clear_error();
    if (!p || !out) return fail(SV_ERR_ARG, "NULL argument");
    *out = p->max_k;
    return SV_OK;
}

extern "C" int sv_plan_rule(const sv_plan *p, int *out)
{
    clear_error();
    if (!p || !out) return fail(SV_ERR_ARG, "NULL argument");
    *out = p->rule;
    return SV_OK;
}

extern "C" int sv_plan_block(const sv_plan *p, int b, int32_t *k, int32_t *q, int32_t *n_members)
{
    clear_error();
    if (!p) return fail(SV_ERR_ARG, "NULL plan");
    if (b < 0 || b >= int(p->blocks.size())) return fail(SV_ERR_ARG, "block %d out of range", b);
    const Block &B = p->blocks[b];
    if (k) *k = B.k;
    if (q)
        for (int j = 0; j < SV_MAX_K; ++j) q[j] = j < B.k ? B.q[j] : -1;
    if (n_members) *n_members = int(B.members.size());
    return SV_OK;
}

extern "C" int sv_plan_own_blocks(sv_plan *p, int on)
{
    clear_error();
    if (!p) return fail(SV_ERR_ARG, "NULL argument");
    p->own_blocks = on != 0;
    return SV_OK;
}

extern "C" int sv_plan_block_pass(const sv_plan *p, int b, int32_t *pass)
{
    clear_error();
    if (!p || !pass) return fail(SV_ERR_ARG, "NULL argument");
    if (b < 0 || b >= int(p->blocks.size())) return fail(SV_ERR_ARG, "block %d out of range", b);
    *pass = p->blocks[b].pass;
    return SV_OK;
}

extern "C" int sv_plan_block_members(const sv_plan *p, int b, int32_t *members)
{
    clear_error();
    if (!p || !members) return fail(SV_ERR_ARG, "NULL argument");
    if (b < 0 || b >= int(p->blocks.size())) return fail(SV_ERR_ARG, "block %d out of range", b);
    const Block &B = p->blocks[b];
    std::copy(B.members.begin(), B.members.end(), members);
    return SV_OK;
}

extern "C" int sv_plan_block_matrix(const sv_plan *p, int b, double *m)
{
    clear_error();
    if (!p || !m) return fail(SV_ERR_ARG, "NULL argument");
    if (b < 0 || b >= int(p->blocks.size())) return fail(SV_ERR_ARG, "block %d out of range", b);
    const Block &B = p->blocks[b];
    std::vector<cd> abi;
    reverse_local_bits(B.m, B.k, abi);
    for (size_t i = 0; i < abi.size(); ++i) {
        m[2 * i] = abi[i].real();
        m[2 * i + 1] = abi[i].imag();
    }
    return SV_OK;
}

extern "C" int sv_apply_plan(sv_state *s, const sv_plan *p, int precision, int use_graph)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (!p) return fail(SV_ERR_ARG, "NULL plan");
    if (int rc = check_precision(s, precision)) return rc;
    for (const auto &b : p->blocks)
        for (int j = 0; j < b.k; ++j)
            if (b.q[j] >= s->n) return fail(SV_ERR_QUBIT, "plan position %d outside a %d-qubit state", b.q[j], s->n);
    if (precision == SV_PREC_SPLIT_FP16)
        for (size_t i = 0; i < p->blocks.size(); ++i) {
            std::string what = "plan block " + std::to_string(i);
            if (int rc = check_unitary(p->blocks[i].m, p->blocks[i].k, what.c_str())) return rc;
        }
    std::vector<Launch> L;
    bool tiles = !p->own_blocks && !p->gates.empty() && takes_tiles(p->rule, precision, s->n);
    if (tiles) {
        if (int rc = plan_tiles(p)) return rc;
        tiles = tiles_are_cheaper(p->blocks, p->tiled, s->n, precision);
    }
    if (int rc = blocks_to_launches(tiles ? p->tiled : p->blocks, s, precision, tiles ? SV_RULE_TILED : p->rule, L,
                                    p->own_blocks))
        return rc;
    if (int rc = select_device(s)) return rc;
    return run_launches(s, L, use_graph != 0);
}

// ============================================================== circuits
namespace {

// Fuse and apply a validated state's circuit (sv_run_circuit, sv_dm_run).
// basis >= 0: the state first becomes |basis> (sv_run_circuit_basis): the
// first launch produces it itself when it is a tile pass, else it is filled.
int run_circuit_impl(sv_state *s, const sv_gate *g, int G, const sv_run_opts *o, int64_t basis = -1)
{
    sv_run_opts d;
    d.max_k = SV_MAX_K;
    d.precision = s->dtype == SV_C64 ? SV_PREC_FP32 : SV_PREC_FP64;
    d.rule = SV_RULE_NONE;
    d.use_graph = 0;
    if (!o) o = &d;
    if (int rc = check_precision(s, o->precision)) return rc;
    if (int rc = validate_gates(g, G, s->n)) return rc;
    if (o->precision == SV_PREC_SPLIT_FP16)
        if (int rc = check_fp16_gates(g, G)) return rc;
    int max_k = o->max_k, rule = o->rule;
    if (rule < SV_RULE_PAPER || rule > SV_RULE_AUTO) return fail(SV_ERR_ARG, "unknown fusion rule %d", rule);
    if (max_k != -1 && (max_k < 1 || max_k > SV_MAX_K))
        return fail(SV_ERR_ARG, "max_k %d outside 1..%d (or -1)", max_k, SV_MAX_K);
    if (max_k == -1 || rule == SV_RULE_AUTO) {
        if (int rc = choose_plan(g, G, s->n, s->dtype, o->precision, rule, max_k, &rule, &max_k)) return rc;
    }
    std::vector<Block> blocks, tiled;
    if (int rc = fuse_gates(g, G, s->n, max_k, rule, lookup_costs(s->n, o->precision, nullptr), blocks, false,
                            o->precision))
        return rc;
    if (takes_tiles(rule, o->precision, s->n)) {
        if (int rc = gates_as_tiles(g, G, s->n, o->precision, blocks, tiled)) return rc;
        if (!tiled.empty() && tiles_are_cheaper(blocks, tiled, s->n, o->precision)) {
            blocks.swap(tiled);
            rule = SV_RULE_TILED;
        }
    }
    block_matrices(g, blocks);
    std::vector<Launch> L;
    if (int rc = blocks_to_launches(blocks, s, o->precision, rule, L)) return rc;
    if (int rc = select_device(s)) return rc;
    if (basis >= 0) {
        // FP32, FP64 and split-FP16 tile passes start from the basis state
        // themselves; other first launches get it filled in
        if (!L.empty() && (L[0].path == PATH_TILE || L[0].path == PATH_TILE_FP16 || L[0].path == PATH_TILE_FP64))
            L[0].basis = basis;
        else
            SV_HIP(dev::launch_fill_basis(s->dtype, s->buf, s->n, uint64_t(basis), s->stream));
    }
    return run_launches(s, L, o->use_graph != 0);
}

}  // namespace

extern "C" int sv_run_circuit(sv_state *s, const sv_gate *g, int G, const sv_run_opts *o)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    return run_circuit_impl(s, g, G, o);
}

extern "C" int sv_run_circuit_basis(sv_state *s, uint64_t basis, const sv_gate *g, int G, const sv_run_opts *o)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (basis >> s->n) return fail(SV_ERR_ARG, "basis index %llu >= 2^%d", (unsigned long long)basis, s->n);
    return run_circuit_impl(s, g, G, o, int64_t(basis));
}

// The super circuit is rewritten as a regular circuit of 2n positions
// (dm_expand) and run like any other circuit.
extern "C" int sv_dm_run(sv_state *rho, const sv_gate *g, int G, const sv_super_op *ops, int n_ops,
                         const sv_run_opts *o)
{
    clear_error();
    if (int rc = check_state(rho)) return rc;
    if (rho->n % 2) return fail(SV_ERR_ARG, "a density matrix needs an even number of state qubits, got %d", rho->n);
    if (o && o->precision == SV_PREC_SPLIT_FP16)
        return fail(SV_ERR_ARG, "SV_PREC_SPLIT_FP16 is not available for density matrices (super operators may "
                                "raise the 2-norm its tile passes rely on)");
    if (int rc = validate_gates(g, G, rho->n / 2)) return rc;
    std::vector<sv_gate> full;
    std::vector<std::vector<double>> store;
    if (int rc = dm_expand(g, G, rho->n / 2, ops, n_ops, full, store)) return rc;
    return run_circuit_impl(rho, full.data(), int(full.size()), o);
}

// ============================================================== reductions
namespace {

// Where a reduction's last kernel writes its `count` results: pinned host memory,
// so that a result costs no copy on the stream behind it (10 qubits: norm 18.2 to
// 16.3 us, expectation of ten terms 25.9 to 19.4).
int result_slots(sv_state *s, size_t count, double **res)
{
    SV_HIP(s->red_host.ensure(count * sizeof(double)));
    *res = static_cast<double *>(s->red_host.p);
    return SV_OK;
}

int read_result(sv_state *s, const double *res, size_t count, double *out)
{
    SV_HIP(hipStreamSynchronize(s->stream));
    std::memcpy(out, res, count * sizeof(double));
    return SV_OK;
}

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

// Group the terms, stage the tables and upload them into the arena.
// The caller synchronised arena_free and records it after its launches.
int pauli_tables(sv_state *s, const sv_pauli_sum *H, int n, PauliUse use, dev::PauliDev &P)
{
    const size_t total = pauli_table_bytes(H);
    SV_HIP(s->stage.ensure(total));
    SV_HIP(s->arena.ensure(total));
    pauli_table_fill(H, n, s->dtype, use, static_cast<char *>(s->stage.p), static_cast<const char *>(s->arena.p), P);
    SV_HIP(hipMemcpyAsync(s->arena.p, s->stage.p, total, hipMemcpyHostToDevice, s->stream));
    return SV_OK;
}

}  // namespace

namespace sv {

int check_pauli(const sv_pauli_sum *H, int n)
{
    if (!H) return fail(SV_ERR_ARG, "NULL Pauli sum");
    if (H->n_terms < 0 || H->n_terms > SV_MAX_PAULI_TERMS)
        return fail(SV_ERR_ARG, "Pauli sum with %d terms (0..%d)", H->n_terms, SV_MAX_PAULI_TERMS);
    if (H->reserved != 0) return fail(SV_ERR_ARG, "sv_pauli_sum.reserved must be 0");
    if (H->n_terms && (!H->coef || !H->xmask || !H->zmask)) return fail(SV_ERR_ARG, "NULL Pauli arrays");
    const uint64_t bad = n >= 64 ? 0 : ~((uint64_t(1) << n) - 1);
    for (int t = 0; t < H->n_terms; ++t) {
        if ((H->xmask[t] | H->zmask[t]) & bad) return fail(SV_ERR_QUBIT, "Pauli term %d acts beyond qubit %d", t, n - 1);
        if (!std::isfinite(H->coef[t])) return fail(SV_ERR_ARG, "non-finite Pauli coefficient");
    }
    return SV_OK;
}

namespace {

// Byte offsets of the device tables of a Pauli sum with ng groups and nt
// terms: group masks, group offsets, term z masks, coefficients.
struct PauliLayout {
    size_t gx, goff, tz, tc, total;
    PauliLayout(int ng, int nt)
    {
        gx = 0;
        goff = al256(gx + 8 * std::max(ng, 1));
        tz = al256(goff + 4 * (ng + 1));
        tc = al256(tz + 8 * std::max(nt, 1));
        total = al256(tc + 8 * std::max(nt, 1));
    }
};

// The group of a term: its x mask and whether its weight is imaginary.
uint64_t pauli_group(const sv_pauli_sum *H, int t)
{
    return H->xmask[t] | (__builtin_popcountll(H->xmask[t] & H->zmask[t]) & 1 ? dev::kPauliImag : 0);
}

int count_groups(const sv_pauli_sum *H)
{
    std::vector<uint64_t> x(size_t(H->n_terms));
    for (int t = 0; t < H->n_terms; ++t) x[size_t(t)] = pauli_group(H, t);
    std::sort(x.begin(), x.end());
    return int(std::unique(x.begin(), x.end()) - x.begin());
}

}  // namespace

size_t pauli_table_bytes(const sv_pauli_sum *H) { return PauliLayout(count_groups(H), H->n_terms).total; }

void pauli_table_fill(const sv_pauli_sum *H, int n, int dtype, PauliUse use, char *h, const char *d, dev::PauliDev &P)
{
    const int nt = H->n_terms;
    P.n_pass = dev::pauli_passes(n, dtype, P.pass_w);
    std::vector<int> order(nt), pass(nt, 0);
    std::vector<uint64_t> group(nt);
    for (int t = 0; t < nt; ++t) {
        order[t] = t;
        group[t] = pauli_group(H, t);
    }
    {
        std::vector<uint64_t> distinct(group);
        std::sort(distinct.begin(), distinct.end());
        distinct.erase(std::unique(distinct.begin(), distinct.end()), distinct.end());
        dev::pauli_choose(n, dtype, nt, distinct.data(), int(distinct.size()), P);
    }
    // the tiled kernels take the groups by pass; a thread of the others gathers
    // them in the order of their masks
    const bool tiled = use == PAULI_EXPECT ? P.tile_expect : use == PAULI_APPLY && P.tile_apply;
    if (tiled)
        for (int t = 0; t < nt; ++t) pass[t] = dev::pauli_pass_of(H->xmask[t], dtype, P.n_pass, P.pass_w);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) {
        if (pass[a] != pass[b]) return pass[a] < pass[b];
        if (!tiled && H->xmask[a] != H->xmask[b]) return H->xmask[a] < H->xmask[b];
        return group[a] < group[b];
    });
    std::vector<uint64_t> gx;
    std::vector<int32_t> goff;
    for (int p = 0, i = 0; p < P.n_pass; ++p) {
        for (; i < nt && pass[order[i]] == p; ++i)
            if (gx.empty() || group[order[i]] != gx.back()) {
                gx.push_back(group[order[i]]);
                goff.push_back(i);
            }
        P.pass_end[p] = int(gx.size());
    }
    goff.push_back(nt);
    const int ng = int(gx.size());
    const PauliLayout L(ng, nt);
    std::memcpy(h + L.gx, gx.data(), 8 * ng);
    std::memcpy(h + L.goff, goff.data(), 4 * (ng + 1));
    for (int i = 0; i < nt; ++i) {
        const int t = order[i];
        const bool minus = __builtin_popcountll(H->xmask[t] & H->zmask[t]) & 2;  // i^2, i^3
        reinterpret_cast<uint64_t *>(h + L.tz)[i] = H->zmask[t];
        reinterpret_cast<double *>(h + L.tc)[i] = minus ? -H->coef[t] : H->coef[t];
    }
    P.n_groups = ng;
    P.gx = reinterpret_cast<const uint64_t *>(d + L.gx);
    P.goff = reinterpret_cast<const int32_t *>(d + L.goff);
    P.tz = reinterpret_cast<const uint64_t *>(d + L.tz);
    P.tc = reinterpret_cast<const double *>(d + L.tc);
}

}  // namespace sv

extern "C" int sv_norm(sv_state *s, double *out)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (!out) return fail(SV_ERR_ARG, "NULL out");
    if (int rc = select_device(s)) return rc;
    double *part = static_cast<double *>(s->red.p), *res = nullptr;
    if (int rc = result_slots(s, 1, &res)) return rc;
    {
        LaunchTimer t(stat_class(FAM_REDUCE, 1), s->stream);
        SV_HIP(dev::launch_norm(s->dtype, s->buf, s->n, part, res, s->stream));
    }
    return read_result(s, res, 1, out);
}

extern "C" int sv_inner(sv_state *a, sv_state *b, double *re, double *im)
{
    clear_error();
    if (!a || !b || !re || !im) return fail(SV_ERR_ARG, "NULL argument");
    if (a->n != b->n) return fail(SV_ERR_ARG, "qubit counts differ (%d vs %d)", a->n, b->n);
    if (int rc = select_device(b)) return rc;
    if (int rc = stream_after(b->stream, a->stream)) return rc;
    double *part = static_cast<double *>(b->red.p), *res = nullptr;
    if (int rc = result_slots(b, 2, &res)) return rc;
    {
        LaunchTimer t(stat_class(FAM_REDUCE, 2), b->stream);
        SV_HIP(dev::launch_inner(a->dtype, a->buf, b->dtype, b->buf, b->n, part, res, b->stream));
    }
    double v[2];
    if (int rc = read_result(b, res, 2, v)) return rc;
    *re = v[0];
    *im = v[1];
    return SV_OK;
}

extern "C" int sv_expectation(sv_state *s, const sv_pauli_sum *H, double *out)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (!out) return fail(SV_ERR_ARG, "NULL out");
    if (int rc = check_pauli(H, s->n)) return rc;
    if (H->n_terms == 0) {
        *out = 0.0;
        return SV_OK;
    }
    if (int rc = select_device(s)) return rc;
    SV_HIP(hipEventSynchronize(s->arena_free));
    dev::PauliDev P;
    if (int rc = pauli_tables(s, H, s->n, PAULI_EXPECT, P)) return rc;
    double *part = static_cast<double *>(s->red.p), *res = nullptr;
    if (int rc = result_slots(s, 1, &res)) return rc;
    {
        LaunchTimer t(stat_class(FAM_REDUCE, 3), s->stream);
        SV_HIP(dev::launch_pauli_expect(s->dtype, s->buf, s->n, P, part, res, s->stream));
    }
    SV_HIP(hipEventRecord(s->arena_free, s->stream));
    return read_result(s, res, 1, out);
}

extern "C" int sv_dm_expectation(sv_state *rho, const sv_pauli_sum *H, double *out)
{
    clear_error();
    if (int rc = check_state(rho)) return rc;
    if (!out) return fail(SV_ERR_ARG, "NULL out");
    if (rho->n % 2) return fail(SV_ERR_ARG, "a density matrix needs an even number of state qubits, got %d", rho->n);
    const int n = rho->n / 2;
    if (int rc = check_pauli(H, n)) return rc;
    if (H->n_terms == 0) {
        *out = 0.0;
        return SV_OK;
    }
    if (int rc = select_device(rho)) return rc;
    SV_HIP(hipEventSynchronize(rho->arena_free));
    dev::PauliDev P;
    if (int rc = pauli_tables(rho, H, n, PAULI_TRACE, P)) return rc;
    double *part = static_cast<double *>(rho->red.p), *res = nullptr;
    if (int rc = result_slots(rho, 1, &res)) return rc;
    {
        LaunchTimer t(stat_class(FAM_REDUCE, 5), rho->stream);
        SV_HIP(dev::launch_dm_expect(rho->dtype, rho->buf, n, P, part, res, rho->stream));
    }
    SV_HIP(hipEventRecord(rho->arena_free, rho->stream));
    return read_result(rho, res, 1, out);
}

namespace {

// p[i] = ||K_i psi||^2 (FP64; one pass over the state per kMaxKraus
// operators).  Synchronises.
int kraus_weights(sv_state *s, const KrausSet &ks, double *p)
{
    if (int rc = select_device(s)) return rc;
    constexpr int kChunks = (kMaxKrausOps + dev::kMaxKraus - 1) / dev::kMaxKraus;
    SV_HIP(s->red.ensure(sizeof(double) * (size_t(dev::kMaxKraus) * dev::kRedBlocks + dev::kMaxKraus * kChunks)));
    SV_HIP(hipEventSynchronize(s->arena_free));
    const size_t bytes = sizeof(cd) * ks.canon.size();
    SV_HIP(s->stage.ensure(bytes));
    SV_HIP(s->arena.ensure(bytes));
    std::memcpy(s->stage.p, ks.canon.data(), bytes);
    SV_HIP(hipMemcpyAsync(s->arena.p, s->stage.p, bytes, hipMemcpyHostToDevice, s->stream));
    double *part = static_cast<double *>(s->red.p), *res = nullptr;
    if (int rc = result_slots(s, size_t(dev::kMaxKraus) * kChunks, &res)) return rc;
    const size_t D2 = size_t(1) << (2 * ks.k);
    for (int c0 = 0; c0 < ks.n_ops; c0 += dev::kMaxKraus) {
        dev::KrausDev K;
        K.n_ops = std::min(dev::kMaxKraus, ks.n_ops - c0);
        K.k = ks.k;
        for (int j = 0; j < 3; ++j) K.pos[j] = j < ks.k ? ks.sorted_q[j] : 0;
        K.m = static_cast<const double *>(s->arena.p) + 2 * D2 * c0;
        LaunchTimer t(stat_class(FAM_REDUCE, 6), s->stream);
        SV_HIP(dev::launch_kraus_probs(s->dtype, s->buf, s->n, K, part, res + c0, s->stream));
    }
    SV_HIP(hipEventRecord(s->arena_free, s->stream));
    return read_result(s, res, size_t(ks.n_ops), p);
}

// The draw: the first operator of nonzero weight whose running sum exceeds
// u * sum p (zero-weight operators are never taken).
int pick_kraus(const double *p, int n_ops, double u, int *pick, double *total)
{
    double sum = 0.0;
    for (int i = 0; i < n_ops; ++i) sum += p[i];
    if (!(sum > 0.0) || !std::isfinite(sum)) return fail(SV_ERR_ARG, "Kraus outcome weights sum to %g", sum);
    *pick = -1;
    *total = sum;
    double run = 0.0;
    for (int i = 0; i < n_ops; ++i) {
        run += p[i];
        if (p[i] > 0.0) *pick = i;  // the last nonzero one, should rounding leave u * total above every sum
        if (p[i] > 0.0 && u * sum < run) break;
    }
    return SV_OK;
}

// Channels sampled one after another on a state, with no gates in between.
//
// Where K_i^dagger K_i is diagonal for every operator of a channel (damping,
// dephasing, Pauli channels, projective measurement), the outcome weights
// depend on the probabilities of its qubits' basis values only.  One pass
// (launch_weighted_bins) then gives the joint probabilities of up to kMaxBins
// qubits, from which the outcomes of all channels on them are drawn in order;
// and a drawn operator need not be applied before the next pass, which weights
// each amplitude by diag(K^dagger K) / p of it instead, as long as the channels
// act on distinct qubits.  The drawn operators are applied together, as gates,
// by flush() or with the gates that follow them (take()).  Other channels run
// one by one: their weights (kraus_weights), then their operator.
class KrausSampler {
  public:
    explicit KrausSampler(sv_state *s) : s_(s) { clear_weights(); }

    // Channel j of `count` with uniform u[j]: its outcome into picks[j] and
    // the outcome's probability into probs[j] (either may be NULL).
    int run(const KrausSet *ks, int count, const double *u, int32_t *picks, double *probs)
    {
        for (int j = 0; j < count;) {
            int end = j, bits = 0;
            uint64_t used = pending_mask_;
            for (; end < count; ++end) {
                bool flat = true;
                uint64_t mask = 0;
                for (int i = 0; i < ks[end].k; ++i) mask |= uint64_t(1) << ks[end].q[i];
                if ((mask & used) || !diagonal(ks[end], &flat)) break;
                if (!flat && bits + ks[end].k > dev::kMaxBins) break;
                if (!flat) bits += ks[end].k;
                used |= mask;
            }
            if (end > j && weights_factor_) {
                if (int rc = draw_group(ks + j, end - j, u + j, picks ? picks + j : nullptr, probs ? probs + j : nullptr)) return rc;
                j = end;
                continue;
            }
            if (!pending_.empty()) {  // the next channel needs the state itself
                if (int rc = flush()) return rc;
                continue;
            }
            double p[kMaxKrausOps], total = 0.0;
            int pick = -1;
            if (int rc = kraus_weights(s_, ks[j], p)) return rc;
            if (int rc = pick_kraus(p, ks[j].n_ops, u[j], &pick, &total)) return rc;
            add_pending(ks[j], pick, p[pick]);
            if (int rc = flush()) return rc;
            if (picks) picks[j] = pick;
            if (probs) probs[j] = p[pick] / total;
            ++j;
        }
        return SV_OK;
    }

    // Qubits of the widest drawn operator (0 when there is none).
    int widest() const
    {
        int k = 0;
        for (const Pending &p : pending_) k = std::max(k, p.k);
        return k;
    }

    // Applies the drawn operators, fused, in the state's own arithmetic.
    int flush()
    {
        if (pending_.empty()) return SV_OK;
        std::vector<sv_gate> g;
        std::vector<std::vector<double>> keep;
        take(g, keep);
        if (g.size() == 1) return apply_gate_impl(s_, g.data());
        sv_run_opts o;
        o.max_k = 4;
        o.precision = s_->dtype == SV_C64 ? SV_PREC_FP32 : SV_PREC_FP64;
        o.rule = s_->n >= tile_min_qubits(o.precision) ? SV_RULE_TILED : SV_RULE_ENHANCED;
        o.use_graph = 0;
        return run_circuit_impl(s_, g.data(), int(g.size()), &o);
    }

    // The drawn operators as gates (matrices in `keep`), for a caller that
    // applies them before anything else reads the state.
    void take(std::vector<sv_gate> &g, std::vector<std::vector<double>> &keep)
    {
        for (Pending &p : pending_) {
            sv_gate h{};
            h.kind = SV_G_MATRIX;
            h.k = p.k;
            h.param = -1;
            for (int a = 0; a < p.k; ++a) h.q[a] = p.q[a];
            keep.push_back(std::move(p.m));
            h.m = keep.back().data();
            g.push_back(h);
        }
        pending_.clear();
        pending_mask_ = 0;
        clear_weights();
    }

  private:
    struct Pending {
        int k;
        int q[3];
        std::vector<double> m;
    };

    void clear_weights()
    {
        for (auto &w : w_) w[0] = w[1] = 1.0;
        scale_ = 1.0;
        weights_factor_ = true;
    }

    // diag(K_i^dagger K_i) of operator i (ABI order)
    static void diag_of(const KrausSet &ks, int i, double *d)
    {
        const int D = 1 << ks.k;
        const double *m = ks.abi.data() + size_t(2) * D * D * i;
        for (int c = 0; c < D; ++c) {
            d[c] = 0.0;
            for (int r = 0; r < D; ++r) d[c] += m[2 * (r * D + c)] * m[2 * (r * D + c)] + m[2 * (r * D + c) + 1] * m[2 * (r * D + c) + 1];
        }
    }

    // K_i^dagger K_i diagonal for every i: no two columns of K_i meet in a row.
    // *flat: it is a multiple of the identity for every i.
    static bool diagonal(const KrausSet &ks, bool *flat)
    {
        const int D = 1 << ks.k;
        *flat = true;
        for (int i = 0; i < ks.n_ops; ++i) {
            const double *m = ks.abi.data() + size_t(2) * D * D * i;
            for (int r = 0; r < D; ++r) {
                int filled = 0;
                for (int c = 0; c < D; ++c) filled += m[2 * (r * D + c)] != 0.0 || m[2 * (r * D + c) + 1] != 0.0;
                if (filled > 1) return false;
            }
            double d[8];
            diag_of(ks, i, d);
            for (int c = 1; c < D; ++c) *flat = *flat && d[c] == d[0];
        }
        return true;
    }

    void add_pending(const KrausSet &ks, int pick, double p)
    {
        const size_t D = size_t(1) << ks.k;
        const double scale = 1.0 / std::sqrt(p);
        Pending x;
        x.k = ks.k;
        for (int a = 0; a < 3; ++a) x.q[a] = ks.q[a];
        x.m.resize(2 * D * D);
        for (size_t e = 0; e < 2 * D * D; ++e) x.m[e] = ks.abi[2 * D * D * size_t(pick) + e] * scale;
        for (int a = 0; a < ks.k; ++a) pending_mask_ |= uint64_t(1) << ks.q[a];
        pending_.push_back(std::move(x));
    }

    int draw_group(const KrausSet *ks, int count, const double *u, int32_t *picks, double *probs)
    {
        // the qubits whose values matter, in the order of their channels (the
        // first channel's first qubit on the top bit of the joint index)
        int order[dev::kMaxBins], pos[dev::kMaxBins], m = 0;
        for (int j = 0; j < count; ++j) {
            bool flat;
            diagonal(ks[j], &flat);
            for (int a = 0; a < ks[j].k && !flat; ++a) order[m++] = ks[j].q[a];
        }
        std::copy(order, order + m, pos);
        std::sort(pos, pos + m);
        if (int rc = select_device(s_)) return rc;
        SV_HIP(s_->red.ensure(dev::weighted_bins_bytes(s_->n, pos, m)));
        SV_HIP(s_->red_host.ensure(sizeof(double) << m));
        const double *bins = static_cast<const double *>(s_->red_host.p);
        {
            LaunchTimer t(stat_class(FAM_REDUCE, 6), s_->stream);
            SV_HIP(dev::launch_weighted_bins(s_->dtype, s_->buf, s_->n, pos, m, w_, scale_,
                                             static_cast<double *>(s_->red.p), static_cast<double *>(s_->red_host.p),
                                             s_->stream));
        }
        SV_HIP(hipStreamSynchronize(s_->stream));
        // joint probabilities by channel order; channel by channel its top bits
        // are summed out with the drawn operator's weights
        std::vector<double> P(size_t(1) << m);
        for (size_t v = 0; v < P.size(); ++v) {
            size_t b = 0;
            for (int i = 0; i < m; ++i)
                if ((v >> (m - 1 - i)) & 1) b |= size_t(1) << (std::lower_bound(pos, pos + m, order[i]) - pos);
            P[v] = bins[b];
        }
        for (int j = 0; j < count; ++j) {
            bool flat;
            diagonal(ks[j], &flat);
            const size_t D = flat ? 1 : size_t(1) << ks[j].k, rest = P.size() / D;
            double S[8], p[kMaxKrausOps], d[8], total = 0.0;
            for (size_t t = 0; t < D; ++t) {
                S[t] = 0.0;
                for (size_t r = 0; r < rest; ++r) S[t] += P[t * rest + r];
            }
            for (int i = 0; i < ks[j].n_ops; ++i) {
                diag_of(ks[j], i, d);
                p[i] = 0.0;
                for (size_t t = 0; t < D; ++t) p[i] += d[t] * S[t];
            }
            int pick = -1;
            if (int rc = pick_kraus(p, ks[j].n_ops, u[j], &pick, &total)) {
                const std::string msg = last_error_cstr();
                (void)flush();  // the channels before it have acted
                return fail(rc, "%s", msg.c_str());
            }
            diag_of(ks[j], pick, d);
            for (size_t r = 0; r < rest; ++r) {
                double v = 0.0;
                for (size_t t = 0; t < D; ++t) v += d[t] / p[pick] * P[t * rest + r];
                P[r] = v;
            }
            P.resize(rest);
            if (flat) scale_ *= d[0] / p[pick];
            else if (ks[j].k == 1) w_[ks[j].q[0]][0] = d[0] / p[pick], w_[ks[j].q[0]][1] = d[1] / p[pick];
            else weights_factor_ = false;  // not a product over qubits: applied before the next pass
            add_pending(ks[j], pick, p[pick]);
            if (picks) picks[j] = pick;
            if (probs) probs[j] = p[pick] / total;
        }
        return SV_OK;
    }

    sv_state *s_;
    std::vector<Pending> pending_;
    uint64_t pending_mask_ = 0;
    double w_[SV_MAX_QUBITS_C64][2];  // weights of the pending operators by qubit value
    double scale_;                    // and of those that are multiples of a unitary
    bool weights_factor_;
};

}  // namespace

extern "C" int sv_kraus_probabilities(sv_state *s, const sv_super_op *op, double *p_out)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (!op || !p_out) return fail(SV_ERR_ARG, "NULL argument");
    KrausSet ks;
    if (int rc = kraus_canonical(*op, s->n, ks)) return rc;
    if (int rc = kraus_weights(s, ks, p_out)) return rc;
    for (int i = ks.n_ops; i < op->n_left; ++i) p_out[i] = 0.0;
    return SV_OK;
}

extern "C" int sv_apply_kraus_sampled(sv_state *s, const sv_super_op *op, double u, int32_t *chosen,
                                      double *p_chosen)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (!op) return fail(SV_ERR_ARG, "NULL operator");
    if (!(u >= 0.0 && u < 1.0)) return fail(SV_ERR_ARG, "uniform %g outside [0, 1)", u);
    KrausSet ks;
    if (int rc = kraus_canonical(*op, s->n, ks)) return rc;
    KrausSampler sampler(s);
    if (int rc = sampler.run(&ks, 1, &u, chosen, p_chosen)) return rc;
    return sampler.flush();
}

extern "C" int sv_run_trajectory(sv_state *s, const sv_gate *g, int G, const sv_super_op *ops, int n_ops,
                                 const double *uniforms, const sv_run_opts *o, int32_t *outcomes)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (int rc = validate_gates(g, G, s->n)) return rc;
    if (n_ops < 0 || (n_ops && (!ops || !uniforms))) return fail(SV_ERR_ARG, "NULL operator or uniform array");
    for (int j = 0; j < n_ops; ++j) {
        KrausSet ks;
        if (int rc = kraus_canonical(ops[j], s->n, ks)) return rc;
        if (ops[j].after < 0 || ops[j].after > G || (j && ops[j].after < ops[j - 1].after))
            return fail(SV_ERR_ARG, "operator %d: after = %d out of order (0..%d, nondecreasing)", j, ops[j].after, G);
        if (!(uniforms[j] >= 0.0 && uniforms[j] < 1.0))
            return fail(SV_ERR_ARG, "uniform %d = %g outside [0, 1)", j, uniforms[j]);
    }
    // Drawn operators join the gates that follow them where those are fused in
    // FP32 or FP64 (the blocks' matrices are formed in FP64).  The 16-bit splits
    // would hold the operators in fewer bits, and an unfused run would give
    // each operator a pass of its own.
    const bool join = o && o->rule != SV_RULE_NONE &&
                      (o->precision == SV_PREC_FP32 || o->precision == SV_PREC_SPLIT_BF16X3 || o->precision == SV_PREC_FP64);
    KrausSampler sampler(s);
    for (int j = 0, done = 0;;) {
        const int upto = j < n_ops ? ops[j].after : G;
        if (upto > done) {
            std::vector<sv_gate> part;
            std::vector<std::vector<double>> keep;
            if (join && (o->max_k < 0 || o->max_k >= sampler.widest())) sampler.take(part, keep);
            else if (int rc = sampler.flush()) return rc;
            if (part.empty()) {
                if (int rc = run_circuit_impl(s, g + done, upto - done, o)) return rc;
            } else {
                part.insert(part.end(), g + done, g + upto);
                if (int rc = run_circuit_impl(s, part.data(), int(part.size()), o)) return rc;
            }
            done = upto;
        }
        if (j == n_ops) break;
        // channels of one place in the circuit, as long as their matrices stay
        // below 4 MiB (three-qubit depolarizing takes 128 KiB)
        std::vector<KrausSet> ks;
        int end = j;
        for (size_t held = 0; end < n_ops && ops[end].after == upto && held < (size_t(4) << 20); ++end) {
            ks.emplace_back();
            if (int rc = kraus_canonical(ops[end], s->n, ks.back())) return rc;
            held += 2 * sizeof(cd) * ks.back().canon.size();
        }
        std::vector<int32_t> picks(size_t(end - j), -1);
        const int rc = sampler.run(ks.data(), end - j, uniforms + j, picks.data(), nullptr);
        for (int i = 0; outcomes && i < end - j; ++i)
            if (picks[size_t(i)] >= 0) outcomes[j + i] = picks[size_t(i)];
        if (rc) return rc;
        j = end;
    }
    return sampler.flush();
}

// ============================================================== projections, measurement, control
extern "C" int sv_project(sv_state *s, int k, const int32_t *q, uint64_t bits, int renormalize, double *prob)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (k < 1 || k > SV_MAX_K || !q) return fail(SV_ERR_ARG, "projection on %d qubits (1..%d)", k, SV_MAX_K);
    if (bits >> k) return fail(SV_ERR_ARG, "bits 0x%llx exceed %d qubits", (unsigned long long)bits, k);
    sv_gate h{};
    h.kind = SV_G_MATRIX;
    h.k = k;
    h.param = -1;
    for (int j = 0; j < k; ++j) h.q[j] = q[j];
    if (int rc = check_gate_qubits(h, s->n)) return rc;
    // |bits><bits| on q (q[0] the most significant bit of bits)
    const size_t D = size_t(1) << k;
    std::vector<double> m(2 * D * D, 0.0);
    m[2 * (bits * D + bits)] = 1.0;
    h.m = m.data();
    if (int rc = select_device(s)) return rc;
    if (int rc = apply_gate_impl(s, &h)) return rc;
    double p = 0.0;
    if (int rc = sv_norm(s, &p)) return rc;
    if (renormalize) {
        if (!(p > 0.0)) return fail(SV_ERR_ARG, "the projection has probability 0; cannot renormalise");
        const double c = 1.0 / std::sqrt(p);
        const double sc[8] = {c, 0, 0, 0, 0, 0, c, 0};  // c I on q[0]
        sv_gate t{};
        t.kind = SV_G_MATRIX;
        t.k = 1;
        t.q[0] = q[0];
        t.param = -1;
        t.m = sc;
        if (int rc = apply_gate_impl(s, &t)) return rc;
    }
    if (prob) *prob = p;
    return SV_OK;
}

extern "C" int sv_measure(sv_state *s, int k, const int32_t *q, const double *uniforms, uint64_t *bits,
                          double *prob)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (k < 1 || k > s->n || !q || !uniforms) return fail(SV_ERR_ARG, "measurement of %d qubits", k);
    for (int j = 0; j < k; ++j) {
        if (q[j] < 0 || q[j] >= s->n) return fail(SV_ERR_QUBIT, "qubit %d outside 0..%d", q[j], s->n - 1);
        for (int i = 0; i < j; ++i)
            if (q[i] == q[j]) return fail(SV_ERR_QUBIT, "qubit %d repeated", q[j]);
        if (!(uniforms[j] >= 0.0 && uniforms[j] < 1.0))
            return fail(SV_ERR_ARG, "uniform %d = %g outside [0, 1)", j, uniforms[j]);
    }
    // qubit by qubit: the Kraus set {|0><0|, |1><1|} sampled with uniforms[j]
    static const double proj[16] = {1, 0, 0, 0, 0, 0, 0, 0,   // |0><0|
                                    0, 0, 0, 0, 0, 0, 1, 0};  // |1><1|
    std::vector<KrausSet> ks(static_cast<size_t>(k));
    for (int j = 0; j < k; ++j) {
        sv_super_op op{};
        op.after = 0;
        op.k = 1;
        op.q[0] = q[j];
        op.n_left = op.n_right = 2;
        op.left = op.right = proj;
        if (int rc = kraus_canonical(op, s->n, ks[size_t(j)])) return rc;
    }
    std::vector<int32_t> b(static_cast<size_t>(k));
    std::vector<double> pb(static_cast<size_t>(k));
    KrausSampler sampler(s);
    if (int rc = sampler.run(ks.data(), k, uniforms, b.data(), pb.data())) return rc;
    if (int rc = sampler.flush()) return rc;
    uint64_t out = 0;
    double ptot = 1.0;
    for (int j = 0; j < k; ++j) {
        out = (out << 1) | uint64_t(b[size_t(j)]);
        ptot *= pb[size_t(j)];
    }
    if (bits) *bits = out;
    if (prob) *prob = ptot;
    return SV_OK;
}

extern "C" int sv_controlled_gate(const sv_gate *g, int n_c, const int32_t *controls, sv_gate *out, double *m_out)
{
    clear_error();
    if (!g || !out || !m_out || (n_c > 0 && !controls)) return fail(SV_ERR_ARG, "NULL argument");
    if (int rc = check_gate_shape(*g)) return rc;
    if (n_c < 1 || n_c + g->k > SV_MAX_K)
        return fail(SV_ERR_ARG, "%d controls on a %d-qubit gate (at most %d qubits in all)", n_c, g->k, SV_MAX_K);
    sv_gate h{};
    h.kind = SV_G_MATRIX;
    h.k = n_c + g->k;
    h.param = -1;
    for (int j = 0; j < n_c; ++j) h.q[j] = controls[j];
    for (int j = 0; j < g->k; ++j) h.q[n_c + j] = g->q[j];
    if (int rc = check_gate_qubits(h, 64)) return rc;
    std::vector<cd> U;
    if (int rc = gate_matrix_abi(*g, U)) return rc;
    // identity, except the block where every control (the most significant
    // local bits) is 1, which holds U
    const size_t D = size_t(1) << h.k, d = size_t(1) << g->k, off = D - d;
    std::fill(m_out, m_out + 2 * D * D, 0.0);
    for (size_t i = 0; i < off; ++i) m_out[2 * (i * D + i)] = 1.0;
    for (size_t r = 0; r < d; ++r)
        for (size_t c = 0; c < d; ++c) {
            m_out[2 * ((off + r) * D + off + c)] = U[r * d + c].real();
            m_out[2 * ((off + r) * D + off + c) + 1] = U[r * d + c].imag();
        }
    h.m = m_out;
    *out = h;
    return SV_OK;
}

extern "C" int sv_apply_pauli_sum(sv_state *psi, const sv_pauli_sum *H, sv_state *out)
{
    clear_error();
    if (!psi || !out) return fail(SV_ERR_ARG, "NULL state handle");
    if (psi == out) return fail(SV_ERR_ARG, "output must be a different state");
    if (psi->n != out->n || psi->dtype != out->dtype) return fail(SV_ERR_ARG, "states differ in n or type");
    if (int rc = check_pauli(H, psi->n)) return rc;
    if (int rc = select_device(psi)) return rc;
    if (int rc = stream_after(psi->stream, out->stream)) return rc;
    SV_HIP(hipEventSynchronize(psi->arena_free));
    dev::PauliDev P;
    if (H->n_terms == 0) {
        SV_HIP(dev::launch_fill_basis(out->dtype, out->buf, out->n, ~uint64_t(0), psi->stream));
    } else {
        if (int rc = pauli_tables(psi, H, psi->n, PAULI_APPLY, P)) return rc;
        LaunchTimer t(stat_class(FAM_REDUCE, 4), psi->stream);
        SV_HIP(dev::launch_pauli_apply(psi->dtype, psi->buf, out->buf, psi->n, P, psi->stream));
    }
    SV_HIP(hipEventRecord(psi->arena_free, psi->stream));
    if (int rc = stream_after(out->stream, psi->stream)) return rc;
    return SV_OK;
}

// ============================================================== adjoint
namespace {

// One step of the backward sweep (gates are visited from last to first): the
// transition sums of a run's qubits, then the launches that undo its gates and
// those before it up to the next rotation with a parameter.
struct BwdStep {
    int lo = 0, hi = -1;      // the run of one-qubit gates lo..hi (hi: a parameterised one), or empty
    std::vector<int> qubits;  // its qubits with parameterised gates
    int slot = -1;            // the first one's slot
    int first = 0, last = 0;  // the gates it undoes, first down to last
};

// dE/dtheta of the run's parameterised gates from its qubits' sums v (8 doubles
// each: S, Z, A, B), added to grad.  The generator P of a gate is Im <lam| V P
// V^dagger |phi> with V the run's later gates on its qubit.
int run_gradients(const sv_gate *g, const BwdStep &st, const double *v, double *grad)
{
    for (size_t k = 0; k < st.qubits.size(); ++k) {
        auto sum = [&](int i) { return cd(v[8 * k + 2 * i], v[8 * k + 2 * i + 1]); };
        const cd M[2][2] = {{0.5 * (sum(0) + sum(1)), 0.5 * (sum(2) + sum(3))},
                            {0.5 * (sum(2) - sum(3)), 0.5 * (sum(0) - sum(1))}};
        cd V[2][2] = {{1, 0}, {0, 1}};
        for (int t = st.hi; t >= st.lo; --t) {
            if (g[t].q[0] != st.qubits[k]) continue;
            if (g[t].param >= 0) {
                static const cd P[3][2][2] = {{{0, 1}, {1, 0}}, {{0, cd(0, -1)}, {cd(0, 1), 0}}, {{1, 0}, {0, -1}}};
                const cd(&p)[2][2] = P[g[t].kind == SV_G_RX ? 0 : g[t].kind == SV_G_RY ? 1 : 2];
                cd e = 0;  // sum_ab (V P V^dagger)_ab M_ab
                for (int a = 0; a < 2; ++a)
                    for (int b = 0; b < 2; ++b)
                        for (int x = 0; x < 2; ++x)
                            for (int y = 0; y < 2; ++y) e += V[a][x] * p[x][y] * std::conj(V[b][y]) * M[a][b];
                grad[g[t].param] += e.imag();
            }
            std::vector<cd> U;
            if (int rc = gate_matrix_abi(g[t], U)) return rc;
            cd W[2][2];
            for (int a = 0; a < 2; ++a)
                for (int b = 0; b < 2; ++b) W[a][b] = V[a][0] * U[size_t(b)] + V[a][1] * U[size_t(2 + b)];
            std::memcpy(static_cast<void *>(V), W, sizeof V);
        }
    }
    return SV_OK;
}

// The daggers of a run of gates, fused into blocks: tile passes or dense ones.
struct DaggerPlan {
    std::vector<cd> store;    // the daggers' matrices
    std::vector<sv_gate> dg;  // point into store
    int kmax = 1;             // qubits of the widest
    std::vector<Block> blocks;
    bool tiled = false;
};

// The daggers of gates hi, hi-1, .., lo (in that order) of a run.
void form_daggers(const sv_gate *g, int hi, int lo, DaggerPlan &p)
{
    const int cnt = hi - lo + 1;
    std::vector<sv_gate> &dg = p.dg;
    dg.resize(size_t(cnt));
    size_t entries = 0;
    for (int t = lo; t <= hi; ++t) entries += size_t(1) << (2 * g[t].k);
    p.store.resize(entries);
    cd *m = p.store.data();
    for (int t = 0; t < cnt; ++t) {
        const sv_gate &src = g[hi - t];
        const int D = 1 << src.k;
        fill_gate_matrix(src, m);
        for (int r = 0; r < D; ++r) {
            for (int c = 0; c < r; ++c) {
                const cd v = m[r * D + c];
                m[r * D + c] = std::conj(m[c * D + r]);
                m[c * D + r] = std::conj(v);
            }
            m[r * D + r] = std::conj(m[r * D + r]);
        }
        dg[t] = src;
        dg[t].kind = SV_G_MATRIX;
        dg[t].param = -1;
        dg[t].m = reinterpret_cast<const double *>(m);
        p.kmax = std::max(p.kmax, src.k);
        m += D * D;
    }
}

// Whether two runs of gates have the same positions.
bool same_positions(const sv_gate *g, const BwdStep &a, const BwdStep &b)
{
    if (a.first - a.last != b.first - b.last) return false;
    for (int i = a.first, j = b.first; i >= a.last; --i, --j)
        if (g[i].k != g[j].k || !std::equal(g[i].q, g[i].q + g[i].k, g[j].q)) return false;
    return true;
}

// Plan the daggers: positions and members of the blocks, no matrices yet
// (dagger_launches).
int plan_daggers(const sv_state *s, int prec, DaggerPlan &p)
{
    const std::vector<sv_gate> &dg = p.dg;
    const int cnt = int(dg.size()), kmax = p.kmax;
    std::vector<Block> &blocks = p.blocks;
    // gates on at most three qubits: one block, which the register kernel applies
    // to both states at the rate of a copy, and with which a single qubit's sums
    // share a launch (launch_transition_step)
    uint64_t on = 0;
    for (const sv_gate &x : dg)
        for (int j = 0; j < x.k; ++j) on |= uint64_t(1) << x.q[j];
    if (__builtin_popcountll(on) <= 3) {
        blocks.resize(1);
        for (uint64_t m = on; m; m &= m - 1) blocks[0].q[blocks[0].k++] = __builtin_ctzll(m);
        blocks[0].members.resize(size_t(cnt));
        std::iota(blocks[0].members.begin(), blocks[0].members.end(), 0);
        return SV_OK;
    }
    const CostTable cost = lookup_costs(s->n, prec, nullptr);
    // The plan of a run (dense blocks of the cheapest k, or tile passes)
    // depends on its gates' positions and the cost table only; it is
    // remembered per run structure, so a sweep with new angles only forms
    // the block matrices.  A colliding entry can only name another valid plan.
    uint64_t key = 1469598103934665603ull;
    auto mix = [&key](uint64_t v) { key = (key ^ v) * 1099511628211ull; };
    mix(uint64_t(s->n));
    mix(uint64_t(s->dtype));
    mix(uint64_t(prec));
    mix(cost_version());
    mix(uint64_t(tile_union_limit()));
    mix(uint64_t(tile_pass_bits(prec)) | uint64_t(tile_pass_capacity(prec)) << 8);
    mix(uint64_t(cnt));
    for (int t = 0; t < cnt; ++t) {
        mix(uint64_t(dg[t].k));
        for (int j = 0; j < dg[t].k; ++j) mix(uint64_t(dg[t].q[j]));
    }
    static std::mutex memo_mu;
    static std::unordered_map<uint64_t, int> memo;  // k of the dense plan, or 0 for tile passes
    int choice = -1;
    {
        std::lock_guard<std::mutex> lk(memo_mu);
        auto it = memo.find(key);
        if (it != memo.end() && (it->second == 0 ? kmax <= 4 : it->second >= kmax)) choice = it->second;
    }
    if (choice < 0) {
        // block size: the cheapest plan under the cost table (complex64
        // blocks of 4..6 qubits run on MFMA; complex128 stays at 4), or
        // tile passes of <= 4-qubit blocks (one launch for both states per
        // pass) where the cost table prices them lower
        int kbest = std::max(kmax, 4);
        double best = 1e300;
        if (s->dtype == SV_C64 && s->n >= 11) {
            for (int k = std::max(kmax, 4); k <= SV_MAX_K; ++k) {
                if (int rc = fuse_gates(dg.data(), cnt, s->n, k, SV_RULE_ENHANCED, cost, blocks, false)) return rc;
                const double c = plan_cost(blocks, cost);
                if (c < best - 1e-12) {
                    best = c;
                    kbest = k;
                }
            }
        }
        choice = kbest;
        if (kmax <= 4 && s->n >= tile_min_qubits(prec)) {
            if (best > 1e299) {
                if (int rc = fuse_gates(dg.data(), cnt, s->n, kbest, SV_RULE_ENHANCED, cost, blocks, false)) return rc;
                best = plan_cost(blocks, cost);
            }
            if (int rc = fuse_gates(dg.data(), cnt, s->n, 4, SV_RULE_TILED, cost, blocks, false, prec)) return rc;
            if (tiled_plan_cost(blocks, s->n, prec, cost) < best - 1e-12) choice = 0;
        }
        std::lock_guard<std::mutex> lk(memo_mu);
        if (memo.size() > 65536) memo.clear();
        memo[key] = choice;
    }
    p.tiled = choice == 0;
    if (p.tiled) return fuse_gates(dg.data(), cnt, s->n, 4, SV_RULE_TILED, cost, blocks, false, prec);
    return fuse_gates(dg.data(), cnt, s->n, choice, SV_RULE_ENHANCED, cost, blocks, false);
}

// No less than the device operands of a plan's blocks take (operand sizes of
// pack_operands), on whatever path.
size_t operand_bound(const DaggerPlan &p, int prec)
{
    const bool split = prec == SV_PREC_SPLIT_BF16 || prec == SV_PREC_SPLIT_FP16;
    const size_t tile = p.tiled ? 4 * size_t(dev::tile_operand_words(tile_operand_prec(tile_path(prec)))) : 0;
    size_t total = 0;
    for (const auto &b : p.blocks) {
        const size_t D2 = size_t(1) << (2 * b.k), form = dev::real_form_elems(b.k);
        total += 256 + std::max({tile, split ? 6 * form + 512 : 4 * form, 16 * D2});
    }
    return total;
}

// Whether the sums of a step and its launches are one pass: one qubit with
// parameters, one dense block of at most three qubits that holds it.
bool one_pass(const BwdStep &st, const std::vector<Launch> &out)
{
    return st.qubits.size() == 1 && out.size() == 1 && !is_tile_path(out[0].path) && out[0].k <= 3 &&
           std::count(out[0].q, out[0].q + out[0].k, st.qubits[0]);
}

// The launches of a plan, whose blocks' matrices are formed here.
std::vector<Launch> dagger_launches(DaggerPlan &p, const sv_state *s, int prec)
{
    std::vector<Launch> out;
    block_matrices(p.dg.data(), p.blocks);
    if (p.tiled) {
        group_tile_passes(p.blocks, s->n, prec, out);
        return out;
    }
    for (auto &b : p.blocks) {
        Launch L;
        L.k = b.k;
        std::copy(b.q, b.q + SV_MAX_K, L.q);
        L.path = choose_path(s->dtype, prec, b.k, b.q, s->n);
        L.m = std::move(b.m);
        out.push_back(std::move(L));
    }
    return out;
}

}  // namespace

namespace {

int backward_impl(sv_state *psi, sv_state *scratch, const sv_gate *g, int G, const sv_pauli_sum *H, double *grad,
                  int n_params, int prec);

}  // namespace

extern "C" int sv_backward(sv_state *psi, sv_state *scratch, const sv_gate *g, int G, const sv_pauli_sum *H,
                           double *grad, int n_params)
{
    clear_error();
    if (!psi) return fail(SV_ERR_ARG, "NULL state handle");
    return backward_impl(psi, scratch, g, G, H, grad, n_params, psi->dtype == SV_C64 ? SV_PREC_FP32 : SV_PREC_FP64);
}

extern "C" int sv_backward_prec(sv_state *psi, sv_state *scratch, const sv_gate *g, int G, const sv_pauli_sum *H,
                                double *grad, int n_params, int precision)
{
    clear_error();
    if (!psi) return fail(SV_ERR_ARG, "NULL state handle");
    if (int rc = check_precision(psi, precision)) return rc;
    return backward_impl(psi, scratch, g, G, H, grad, n_params, precision);
}

namespace {

int backward_impl(sv_state *psi, sv_state *scratch, const sv_gate *g, int G, const sv_pauli_sum *H, double *grad,
                  int n_params, int prec)
{
    if (!psi || !scratch) return fail(SV_ERR_ARG, "NULL state handle");
    if (psi == scratch) return fail(SV_ERR_ARG, "scratch must be a different state");
    if (psi->n != scratch->n || psi->dtype != scratch->dtype) return fail(SV_ERR_ARG, "states differ in n or type");
    if (n_params < 0 || (n_params > 0 && !grad)) return fail(SV_ERR_ARG, "bad gradient buffer");
    if (int rc = validate_gates(g, G, psi->n)) return rc;
    if (prec == SV_PREC_SPLIT_FP16)
        if (int rc = check_fp16_gates(g, G)) return rc;
    if (int rc = check_pauli(H, psi->n)) return rc;
    for (int i = 0; i < G; ++i)
        if (g[i].param >= n_params) return fail(SV_ERR_ARG, "gate %d: param %d >= n_params %d", i, g[i].param, n_params);

    // plan the sweep: every run of one-qubit gates that ends in a parameterised
    // one shares one pass of transition sums; it is undone together with the
    // gates before it, down to the next parameterised one
    std::vector<BwdStep> steps;
    int slots = 0;
    for (int i = G - 1; i >= 0;) {
        BwdStep st;
        int stop = i;  // the last gate that is not undone in this step
        if (g[i].param >= 0) {
            st.hi = i;
            int j = i;
            uint64_t used = 0;
            for (; j >= 0 && g[j].k == 1; --j)
                if (g[j].param >= 0) used |= uint64_t(1) << g[j].q[0];
            st.lo = j + 1;
            for (uint64_t m = used; m; m &= m - 1) st.qubits.push_back(__builtin_ctzll(m));
            st.slot = slots;
            slots += int(st.qubits.size());
            stop = j;
        }
        while (stop >= 0 && g[stop].param < 0) --stop;
        st.first = i;
        st.last = stop + 1;
        steps.push_back(std::move(st));
        i = stop;
    }
    if (int rc = select_device(psi)) return rc;
    // lam <- H psi on psi's stream
    if (int rc = sv_apply_pauli_sum(psi, H, scratch)) return rc;
    // All that can fail short of a launch comes before the sweep changes psi:
    // the plans of all steps, and room for their operands.  H psi is computed
    // meanwhile.  A step of the same positions as the one before it has that
    // one's plan; the others are independent host work: spread over threads
    // where there are many.
    std::vector<DaggerPlan> plans(steps.size());
    std::vector<size_t> plan_of(steps.size());
    auto spread = [&](size_t from, size_t to, auto &&work) {
        std::atomic<size_t> next(from);
        auto worker = [&]() {
            for (size_t t; (t = next.fetch_add(1)) < to;) work(t);
        };
        unsigned nt = 1;
        if (to - from >= 16)
            nt = std::min(std::max(1u, std::min(8u, std::thread::hardware_concurrency())), unsigned((to - from) / 4));
        std::vector<std::thread> pool;
        for (unsigned t = 1; t < nt; ++t) pool.emplace_back(worker);
        worker();
        for (auto &th : pool) th.join();
    };
    {
        std::vector<int> rcs(steps.size(), SV_OK);
        std::vector<std::string> msgs(steps.size());
        for (size_t t = 0; t < steps.size(); ++t)
            plan_of[t] = t && same_positions(g, steps[t], steps[t - 1]) ? plan_of[t - 1] : t;
        spread(0, steps.size(), [&](size_t t) {
            if (plan_of[t] != t) return;
            form_daggers(g, steps[t].first, steps[t].last, plans[t]);
            rcs[t] = plan_daggers(psi, prec, plans[t]);
            if (rcs[t]) msgs[t] = last_error_cstr();
        });
        for (size_t t = 0; t < steps.size(); ++t)
            if (rcs[t]) return fail(rcs[t], "%s", msgs[t].c_str());
    }
    // The first quarter of the steps is launched before the others' matrices
    // are formed, so that the GPU sweeps meanwhile.  Its operands lie in the
    // scratch state's arena: psi's holds H's tables until then.
    const size_t ahead = (steps.size() + 3) / 4;
    for (sv_state *at : {scratch, psi}) {
        size_t bytes = prec == SV_PREC_SPLIT_FP16 ? 8 * kTileNormSlots + 256 : 0;
        for (size_t t = at == psi ? ahead : 0; t < (at == psi ? steps.size() : ahead); ++t) bytes += operand_bound(plans[plan_of[t]], prec);
        if (bytes > at->stage.cap || bytes > at->arena.cap) SV_HIP(hipEventSynchronize(at->arena_free));
        SV_HIP(at->stage.ensure(bytes));
        SV_HIP(at->arena.ensure(bytes));
    }
    SV_HIP(psi->grad.ensure(sizeof(double) * 8 * size_t(std::max(slots, 1)) * size_t(dev::transition_blocks(psi->n))));
    SV_HIP(psi->red_host.ensure(sizeof(double) * 8 * size_t(std::max(slots, 1))));
    double *part = static_cast<double *>(psi->grad.p);
    auto sweep = [&](size_t from, size_t to, sv_state *at) -> int {
        std::vector<std::vector<Launch>> outs(to - from);
        spread(from, to, [&](size_t t) {
            DaggerPlan p;
            form_daggers(g, steps[t].first, steps[t].last, p);
            p.blocks = plans[plan_of[t]].blocks;
            p.tiled = plans[plan_of[t]].tiled;
            outs[t - from] = dagger_launches(p, psi, prec);
        });
        std::vector<Launch> launches;
        std::vector<size_t> end;  // of each step's launches
        std::vector<char> together;
        for (size_t t = from; t < to; ++t) {
            auto &out = outs[t - from];
            together.push_back(one_pass(steps[t], out));
            if (together.back()) out[0].path = PATH_REG;  // the matrix is an argument
            for (auto &L : out) launches.push_back(std::move(L));
            end.push_back(launches.size());
        }
        // only blocks of other kernels than the register kernel have operands
        const bool operands = std::any_of(launches.begin(), launches.end(), [](const Launch &L) { return L.path != PATH_REG; });
        if (operands) SV_HIP(hipEventSynchronize(at->arena_free));
        const size_t bytes = operands ? pack_operands(launches, psi->dtype, at->stage) : 0;
        if (bytes > at->arena.cap) return fail(SV_ERR_HIP, "operands of %zu bytes in an arena of %zu", bytes, at->arena.cap);
        if (bytes) SV_HIP(hipMemcpyAsync(at->arena.p, at->stage.p, bytes, hipMemcpyHostToDevice, psi->stream));
        for (size_t t = from, l = 0; t < to; l = end[t++ - from]) {
            const BwdStep &st = steps[t];
            const Launch *L = launches.data() + l;
            if (together[t - from]) {
                LaunchTimer timer(stat_class(FAM_ADJOINT, L->k), psi->stream);
                SV_HIP(dev::launch_transition_step(psi->dtype, L->k, L->q, L->m.data(), st.qubits[0], psi->buf,
                                                   scratch->buf, psi->n, part, st.slot, psi->stream));
                continue;
            }
            if (!st.qubits.empty()) {
                LaunchTimer timer(stat_class(FAM_ADJOINT, 3), psi->stream);
                SV_HIP(dev::launch_transitions(psi->dtype, int(st.qubits.size()), st.qubits.data(), psi->buf,
                                               scratch->buf, psi->n, part, st.slot, psi->stream));
            }
            if (int rc = enqueue(launches.data() + l, end[t - from] - l, psi->dtype, psi->buf, psi->n, at->arena.p,
                                 psi->stream, scratch->buf))
                return rc;
        }
        return SV_OK;
    };
    int swept = sweep(0, ahead, scratch);
    // after a failed launch too, nothing may touch the arenas or the scratch
    // state before what is in flight
    SV_HIP(hipEventRecord(scratch->arena_free, psi->stream));
    if (!swept && ahead < steps.size()) swept = sweep(ahead, steps.size(), psi);
    SV_HIP(hipEventRecord(psi->arena_free, psi->stream));
    if (swept) {
        const std::string msg = last_error_cstr();
        (void)stream_after(scratch->stream, psi->stream);
        return fail(swept, "%s", msg.c_str());
    }
    double *sums = static_cast<double *>(psi->red_host.p);
    if (slots) SV_HIP(dev::launch_transitions_final(part, slots, psi->n, sums, psi->stream));
    SV_HIP(hipStreamSynchronize(psi->stream));
    for (const BwdStep &st : steps)
        if (!st.qubits.empty())
            if (int rc = run_gradients(g, st, sums + 8 * size_t(st.slot), grad)) return rc;
    if (int rc = stream_after(scratch->stream, psi->stream)) return rc;
    return SV_OK;
}

}  // namespace

// ============================================================== stats
extern "C" int sv_stats_enable(int on)
{
    clear_error();
    return stats_enable(on);
}
extern "C" int sv_stats_reset(void)
{
    clear_error();
    return stats_reset();
}
extern "C" int sv_stats_query(int cls, int64_t *launches, double *total_ms)
{
    clear_error();
    if (!launches || !total_ms) return fail(SV_ERR_ARG, "NULL argument");
    return stats_query(cls, launches, total_ms);
}

extern "C" int sv_graph_stats(const sv_state *s, int64_t *runs, int64_t *reused)
{
    clear_error();
    if (int rc = check_state(s)) return rc;
    if (runs) *runs = s->graph_launches;
    if (reused) *reused = s->graph_updates;
    return SV_OK;
}
