// Runtime: buffers, launch timing, kernel-path choice, operand packing and
// launch sequencing for fused plans.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <map>

#include "runtime.h"

namespace sv {

// ---------------------------------------------------------------- buffers
hipError_t DevBuf::ensure(size_t bytes)
{
    if (bytes <= cap) return hipSuccess;
    release();
    size_t want = std::max(bytes, size_t(4096));
    hipError_t e = hipMalloc(&p, want);
    if (e != hipSuccess) {
        p = nullptr;
        return e;
    }
    cap = want;
    return hipSuccess;
}

void DevBuf::release()
{
    if (p) (void)hipFree(p);
    p = nullptr;
    cap = 0;
}

hipError_t PinBuf::ensure(size_t bytes)
{
    if (bytes <= cap) return hipSuccess;
    release();
    size_t want = std::max(bytes, size_t(4096));
    hipError_t e = hipHostMalloc(&p, want, hipHostMallocDefault);
    if (e != hipSuccess) {
        p = nullptr;
        return e;
    }
    cap = want;
    return hipSuccess;
}

void PinBuf::release()
{
    if (p) (void)hipHostFree(p);
    p = nullptr;
    cap = 0;
}

// ---------------------------------------------------------------- timing
namespace {
struct Pending {
    int cls;
    int parts[4];
    hipEvent_t a, b;
};
struct StatsState {
    std::mutex mu;
    bool on = false;
    bool suspended = false;
    std::vector<Pending> pending;
    std::vector<hipEvent_t> free_events;
    std::map<int, std::pair<int64_t, double>> totals;
};
StatsState &stats()
{
    static StatsState s;
    return s;
}
hipEvent_t take_event(StatsState &s)
{
    if (!s.free_events.empty()) {
        hipEvent_t e = s.free_events.back();
        s.free_events.pop_back();
        return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
}
// Fold pending launches into the totals (synchronises on their events).
int drain(StatsState &s)
{
    int rc = SV_OK;
    for (auto &p : s.pending) {
        float ms = 0.f;
        hipError_t e = hipEventSynchronize(p.b);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, p.a, p.b);
        if (e != hipSuccess) {
            rc = fail(SV_ERR_HIP, "launch timing: %s", hipGetErrorString(e));
        } else {
            const int sum = p.parts[1] + p.parts[2] + p.parts[3];
            for (int k = sum ? 1 : 0; k <= (sum ? 3 : 0); ++k) {
                if (sum && !p.parts[k]) continue;
                auto &t = s.totals[sum ? stat_class(FAM_REG, k) : p.cls];
                t.first += sum ? p.parts[k] : 1;
                t.second += sum ? ms * p.parts[k] / sum : ms;
            }
        }
        s.free_events.push_back(p.a);
        s.free_events.push_back(p.b);
    }
    s.pending.clear();
    return rc;
}
}  // namespace

LaunchTimer::LaunchTimer(int cls, hipStream_t st, const int *parts) : cls_(cls), st_(st)
{
    for (int k = 1; parts && k <= 3; ++k) parts_[k] = parts[k];
    auto &s = stats();
    std::lock_guard<std::mutex> lk(s.mu);
    if (!s.on || s.suspended) return;
    a_ = take_event(s);
    b_ = take_event(s);
    if (a_ && b_) (void)hipEventRecord(a_, st_);
}

LaunchTimer::~LaunchTimer()
{
    if (!a_ || !b_) return;
    auto &s = stats();
    std::lock_guard<std::mutex> lk(s.mu);
    (void)hipEventRecord(b_, st_);
    s.pending.push_back({cls_, {parts_[0], parts_[1], parts_[2], parts_[3]}, a_, b_});
    if (s.pending.size() > 4096) drain(s);
}

void timing_suspend(bool on)
{
    auto &s = stats();
    std::lock_guard<std::mutex> lk(s.mu);
    s.suspended = on;
}

int stats_enable(int on)
{
    auto &s = stats();
    std::lock_guard<std::mutex> lk(s.mu);
    s.on = on != 0;
    return SV_OK;
}

int stats_reset()
{
    auto &s = stats();
    std::lock_guard<std::mutex> lk(s.mu);
    int rc = drain(s);
    s.totals.clear();
    return rc;
}

int stats_query(int cls, int64_t *launches, double *total_ms)
{
    auto &s = stats();
    std::lock_guard<std::mutex> lk(s.mu);
    int rc = drain(s);
    auto it = s.totals.find(cls);
    *launches = it == s.totals.end() ? 0 : it->second.first;
    *total_ms = it == s.totals.end() ? 0.0 : it->second.second;
    return rc;
}

// ---------------------------------------------------------------- paths
Tuning &tuning()
{
    static Tuning t = [] {
        Tuning x;
        for (int k = 0; k <= SV_MAX_K; ++k) {
            x.reg_grid_cap[k] = 8192;
            x.mfma_tc_log[k] = 6;
            x.mfma_grid_cap[k] = 2048;
            x.split_tc_log[k] = 6;
        }
        x.mfma_tc_log[4] = 7;
        x.split_tc_log[4] = 7;
        x.mfma_tc_log[6] = 5;
        x.split_tc_log[6] = 5;
        x.k4_reg = false;
        x.tile_grid_cap = 256;
        x.tile_bits = 14;
        x.tile_waves = 16;
        if (const char *e = std::getenv("SV_TILE_BITS")) x.tile_bits = std::atoi(e) == 13 ? 13 : 14;
        if (const char *e = std::getenv("SV_TILE_WAVES")) x.tile_waves = std::atoi(e);
        if (!dev::tile_shape_supported(x.tile_bits, x.tile_waves)) x.tile_waves = x.tile_bits == 14 ? 16 : 4;
        if (const char *e = std::getenv("SV_TILE_GRID")) x.tile_grid_cap = std::max(1, std::atoi(e));
        return x;
    }();
    return t;
}

int tile_pass_bits(int precision) { return precision == SV_PREC_FP64 ? dev::kF64MaxUnion : tuning().tile_bits; }

int tile_pass_capacity(int precision)
{
    const Tuning &t = tuning();
    const int prec = precision < 0 ? dev::kTileOperandBF16 : tile_operand_prec(tile_path(precision));
    return dev::tile_max_blocks(t.tile_bits, t.tile_waves, prec);
}

// Below the gate passes, and where MFMA does not reach, the register kernel's
// few threads lose to one output a thread: FP64 k = 3 23 to 6 us, FP32 k = 4
// (at most 8 qubits) 82 to 6.
bool rows_beat_registers(int dtype, int k, int n)
{
    return k >= (dtype == SV_C128 ? 3 : 4) && n < dev::kMinTileQubits;
}

Path choose_path(int dtype, int precision, int k, const int *q, int n)
{
    const bool reg = dev::reg_supported(dtype, k, q, n) && !rows_beat_registers(dtype, k, n);
    if (dtype == SV_C128) return reg ? PATH_REG : PATH_GENERIC;
    if (k >= 4 && dev::mfma_supported(k, n)) {
        if (precision == SV_PREC_SPLIT_BF16) return PATH_SPLIT_BF16;
        if (precision == SV_PREC_SPLIT_FP16) return PATH_SPLIT_FP16;
        if (!(k == 4 && tuning().k4_reg && dev::reg_supported(dtype, k, q, n))) return PATH_MFMA32;
    }
    return reg ? PATH_REG : PATH_GENERIC;
}

int path_family(Path p)
{
    switch (p) {
    case PATH_REG:
    case PATH_GATES: return FAM_REG;
    case PATH_GENERIC: return FAM_GENERIC;
    case PATH_MFMA32: return FAM_MFMA32;
    case PATH_SPLIT_BF16: return FAM_SPLIT_BF16;
    case PATH_TILE: return FAM_TILE;
    case PATH_TILE_BF16: return FAM_TILE_BF16;
    case PATH_TILE_FP16: return FAM_TILE_FP16;
    case PATH_TILE_BF16X3: return FAM_TILE_BF16X3;
    case PATH_TILE_FP64: return FAM_TILE_FP64;
    default: return FAM_SPLIT_FP16;
    }
}

static size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

// The operand of a gate pass (launch_gate_pass): stage ranges, ops, matrices.
static size_t gate_pass_ops_bytes(const Launch &L) { return (4 * dev::kGateHeaderWords + 8 * L.gates.size() + 15) & ~size_t(15); }
static size_t gate_pass_bytes(const Launch &L, int dtype)
{
    return gate_pass_ops_bytes(L) + L.m.size() * 2 * (dtype == SV_C64 ? 4 : 8);
}
template <typename T>
static void pack_gate_pass(const Launch &L, char *h)
{
    uint32_t *w = reinterpret_cast<uint32_t *>(h);
    uint32_t at = 0;
    for (int s = 0; s <= dev::kMaxTileSubBlocks; ++s) {
        w[s] = at;
        if (s < L.k) at += uint32_t(L.stage_gates[size_t(s)]);
    }
    T *m = reinterpret_cast<T *>(h + gate_pass_ops_bytes(L));
    for (size_t i = 0; i < L.m.size(); ++i) {
        m[2 * i] = T(L.m[i].real());
        m[2 * i + 1] = T(L.m[i].imag());
    }
    size_t off = gate_pass_ops_bytes(L) / sizeof(T);
    for (size_t g = 0; g < L.gates.size(); ++g) {
        w[dev::kGateHeaderWords + 2 * g] = uint32_t(L.gates[g].second);
        w[dev::kGateHeaderWords + 2 * g + 1] = uint32_t(off);
        off += size_t(2) << (2 * L.gates[g].first);
    }
}

size_t pack_operands(std::vector<Launch> &launches, int dtype, PinBuf &stage)
{
    // pass 1: sizes
    size_t total = 0;
    for (auto &L : launches) {
        const int D = 1 << L.k;
        switch (L.path) {
        case PATH_REG: break;
        case PATH_GENERIC:
            L.arena_off = total;
            total = align256(total + size_t(D) * D * 2 * (dtype == SV_C64 ? 4 : 8));
            break;
        case PATH_MFMA32:
            L.arena_off = total;
            total = align256(total + dev::real_form_elems(L.k) * 4);
            break;
        case PATH_TILE:
        case PATH_TILE_BF16:
        case PATH_TILE_FP16:
        case PATH_TILE_BF16X3:
        case PATH_TILE_FP64:
            L.arena_off = total;
            total = align256(total + size_t(L.k) * dev::tile_operand_words(tile_operand_prec(L.path)) * 4);
            break;
        case PATH_GATES:
            L.arena_off = total;
            total = align256(total + gate_pass_bytes(L, dtype));
            break;
        default:
            L.arena_off = total;
            total = align256(total + dev::real_form_elems(L.k) * 2);
            L.arena_off2 = total;
            total = align256(total + dev::real_form_elems(L.k) * 2);
            L.arena_off3 = total;
            total = align256(total + dev::real_form_elems(L.k) * 2);
            break;
        }
    }
    // one region for the norm partials of the run's split-FP16 tile passes
    bool fp16_tiles = false;
    for (const auto &L : launches) fp16_tiles = fp16_tiles || L.path == PATH_TILE_FP16;
    if (fp16_tiles) {
        for (auto &L : launches)
            if (L.path == PATH_TILE_FP16) L.norm_off = total;
        total = align256(total + sizeof(double) * kTileNormSlots);
    }
    if (total == 0) return 0;
    if (stage.ensure(total) != hipSuccess) return size_t(-1);
    char *h = static_cast<char *>(stage.p);
    for (auto &L : launches) {
        const int D = 1 << L.k;
        switch (L.path) {
        case PATH_REG: break;
        case PATH_GENERIC:
            if (dtype == SV_C64) {
                float *f = reinterpret_cast<float *>(h + L.arena_off);
                for (int i = 0; i < D * D; ++i) {
                    f[2 * i] = float(L.m[i].real());
                    f[2 * i + 1] = float(L.m[i].imag());
                }
            } else {
                double *f = reinterpret_cast<double *>(h + L.arena_off);
                for (int i = 0; i < D * D; ++i) {
                    f[2 * i] = L.m[i].real();
                    f[2 * i + 1] = L.m[i].imag();
                }
            }
            break;
        case PATH_MFMA32:
            dev::pack_real_form_f32(L.m.data(), L.k, reinterpret_cast<float *>(h + L.arena_off));
            break;
        case PATH_TILE:
        case PATH_TILE_BF16:
        case PATH_TILE_FP16:
        case PATH_TILE_BF16X3:
        case PATH_TILE_FP64:
            for (int sb = 0; sb < L.k; ++sb)
                dev::pack_tile_operand(L.m.data() + 256 * sb, tile_operand_prec(L.path),
                                       reinterpret_cast<uint32_t *>(h + L.arena_off) +
                                           dev::tile_operand_words(tile_operand_prec(L.path)) * sb);
            break;
        case PATH_GATES:
            if (dtype == SV_C64) pack_gate_pass<float>(L, h + L.arena_off);
            else pack_gate_pass<double>(L, h + L.arena_off);
            break;
        default: {
            uint16_t *const parts[3] = {reinterpret_cast<uint16_t *>(h + L.arena_off),
                                        reinterpret_cast<uint16_t *>(h + L.arena_off2),
                                        reinterpret_cast<uint16_t *>(h + L.arena_off3)};
            dev::pack_real_form_split(L.m.data(), L.k, L.path == PATH_SPLIT_FP16, parts);
            break;
        }
        }
    }
    return total;
}

// Canonical 16 x 16 matrix of a block on positions q[0..k-1] (ascending)
// padded with identity on the extra positions of p4 (ascending, 4 entries).
static void pad_to_four(const Block &b, const int *p4, cd *out)
{
    if (b.k == 4) {
        std::copy(b.m.begin(), b.m.end(), out);
        return;
    }
    int own[16], rest[16];  // each padded index's bits of b, and its other bits
    for (int r = 0; r < 16; ++r) {
        own[r] = 0;
        rest[r] = r;
        for (int j = 0; j < 4; ++j)
            for (int i = 0; i < b.k; ++i)
                if (b.q[i] == p4[j] && ((r >> j) & 1)) {
                    own[r] |= 1 << i;
                    rest[r] &= ~(1 << j);
                }
    }
    const int D = 1 << b.k;
    for (int r = 0; r < 16; ++r)
        for (int c = 0; c < 16; ++c) out[r * 16 + c] = rest[r] == rest[c] ? b.m[size_t(own[r]) * D + own[c]] : cd(0);
}

static uint64_t mask_of(const Block &b)
{
    uint64_t m = 0;
    for (int j = 0; j < b.k; ++j) m |= uint64_t(1) << b.q[j];
    return m;
}

Path tile_path(int precision)
{
    if (precision == SV_PREC_SPLIT_BF16) return PATH_TILE_BF16;
    if (precision == SV_PREC_SPLIT_FP16) return PATH_TILE_FP16;
    if (precision == SV_PREC_SPLIT_BF16X3) return PATH_TILE_BF16X3;
    if (precision == SV_PREC_FP64) return PATH_TILE_FP64;
    return PATH_TILE;
}

int tile_operand_prec(int path)
{
    return path == PATH_TILE_BF16     ? dev::kTileOperandBF16
           : path == PATH_TILE_FP16   ? dev::kTileOperandF16
           : path == PATH_TILE_BF16X3 ? dev::kTileOperandBF16X3
           : path == PATH_TILE_FP64   ? dev::kTileOperandF64
                                      : dev::kTileOperandF32;
}

// The positions of tile_pass_blocks' padded blocks.
static void tile_pass_positions(const Block *const *blocks, int count, int n, int (*sub_pos)[4])
{
    uint64_t um = 0;
    for (int i = 0; i < count; ++i) um |= mask_of(*blocks[i]);
    // the union gets at least 4 positions (lowest free ones)
    for (int p = 0; p < n && __builtin_popcountll(um) < 4; ++p) um |= uint64_t(1) << p;
    for (int sb = 0; sb < count; ++sb) {
        uint64_t pm = mask_of(*blocks[sb]);
        for (int p = 0; p < 64 && __builtin_popcountll(pm) < 4; ++p)
            if (((um >> p) & 1) && !((pm >> p) & 1)) pm |= uint64_t(1) << p;
        int c = 0;
        for (int p = 0; p < 64; ++p)
            if ((pm >> p) & 1) sub_pos[sb][c++] = p;
    }
}

void tile_pass_blocks(const Block *const *blocks, int count, int n, int (*sub_pos)[4], std::vector<cd> &mats)
{
    tile_pass_positions(blocks, count, n, sub_pos);
    mats.resize(size_t(256) * count);
    for (int sb = 0; sb < count; ++sb) pad_to_four(*blocks[sb], sub_pos[sb], mats.data() + 256 * sb);
}

void group_tile_passes(const std::vector<Block> &blocks, int n, int precision, std::vector<Launch> &out)
{
    out.clear();
    const CostTable cost = lookup_costs(n, precision, nullptr);
    const bool fp64 = precision == SV_PREC_FP64;
    for (const auto &grp : tile_groups(blocks, n, precision))
        for (size_t at = 0; at < grp.size();) {
            // a pass planned for another arithmetic or another tile shape may
            // cover more positions than a tile holds now: as many of its blocks
            // as fit (position 0 lies in every tile of complex64, and FP64's
            // count leaves it out)
            size_t end = at;
            for (uint64_t u = fp64 ? 0 : 1; end < grp.size(); ++end) {
                u |= mask_of(blocks[grp[end]]);
                if (end > at && __builtin_popcountll(u) > tile_pass_bits(precision)) break;
            }
            // a block alone: its own dense launch, or a tile pass of one block
            // where that is priced lower
            const Block &b0 = blocks[grp[at]];
            Launch L;
            if (end - at == 1 && !(lone_block_may_tile(b0.k, n) && cost.tile[1] < cost.ms[b0.k])) {
                L.k = b0.k;
                std::copy(b0.q, b0.q + SV_MAX_K, L.q);
                L.path = choose_path(fp64 ? SV_C128 : SV_C64, precision, b0.k, b0.q, n);
                L.m = b0.m;
            } else {
                L.path = tile_path(precision);
                L.k = int(end - at);
                std::fill(L.q, L.q + SV_MAX_K, 0);
                std::vector<const Block *> bp;
                for (size_t i = at; i < end; ++i) bp.push_back(&blocks[grp[i]]);
                tile_pass_blocks(bp.data(), L.k, n, L.sub_pos, L.m);
            }
            out.push_back(std::move(L));
            at = end;
        }
}

int group_dense_passes(std::vector<Launch> &launches, int n, int precision)
{
    if (n < dev::kMinTileQubits) return SV_OK;
    auto takes = [](const Launch &L) { return L.k == 4 && L.path == PATH_SPLIT_FP16; };
    const CostTable cost = lookup_costs(n, precision, nullptr);
    std::vector<Launch> out, passes;
    for (size_t at = 0; at < launches.size();) {
        size_t end = at;
        while (end < launches.size() && takes(launches[end])) ++end;
        if (end - at < 2) {
            out.push_back(std::move(launches[at++]));
            continue;
        }
        std::vector<sv_gate> g(end - at);
        for (size_t i = at; i < end; ++i) {
            sv_gate &x = g[i - at];
            x.kind = SV_G_MATRIX;
            x.k = 4;
            for (int j = 0; j < 4; ++j) x.q[j] = launches[i].q[3 - j];  // canonical order: the lowest position is the lowest bit
            x.param = -1;
            x.m = reinterpret_cast<const double *>(launches[i].m.data());
        }
        std::vector<Block> blocks;
        if (int rc = fuse_gates(g.data(), int(g.size()), n, 4, SV_RULE_TILED, cost, blocks, true, precision)) return rc;
        if (tiled_plan_cost(blocks, n, precision, cost) < cost.ms[4] * double(end - at) - 1e-12) {
            group_tile_passes(blocks, n, precision, passes);
            for (auto &L : passes) out.push_back(std::move(L));
        } else {
            for (size_t i = at; i < end; ++i) out.push_back(std::move(launches[i]));
        }
        at = end;
    }
    launches.swap(out);
    return SV_OK;
}

int group_gate_passes(std::vector<Launch> &launches, int n, int dtype)
{
    if (n < dev::kMinTileQubits) return SV_OK;
    const int precision = dtype == SV_C64 ? SV_PREC_FP32 : SV_PREC_FP64;
    auto small = [](const Launch &L) { return L.path == PATH_REG && L.k <= 3; };
    // Below 20 qubits a launch is host time, and a pass takes more of it than a
    // gate does: 11 us more than the first launch, against what a further gate in
    // the pass saves, about 3, 2 and 4 us for one, two and three qubits
    // (complex128, whose register kernel is slower: 4, 4 and 11).  16 qubits,
    // launches against passes: two H 17 and 23 us, four 25 and 25, eight 38 and
    // 31; three FSIM 24 and 28, six 37 and 36, ten 54 and 48.
    const int gain[4] = {0, dtype == SV_C64 ? 3 : 4, dtype == SV_C64 ? 2 : 4, dtype == SV_C64 ? 4 : 11};
    auto worth = [&](int sum) { return n >= 20 || sum >= 11; };
    int longest = 0, run = 0, count = 0;
    for (const Launch &L : launches) {
        run = small(L) ? run + gain[L.k] : 0;
        count = small(L) ? count + 1 : 0;
        if (count >= 2) longest = std::max(longest, run);
    }
    if (longest == 0 || !worth(longest)) return SV_OK;
    std::vector<Launch> out;
    for (size_t at = 0; at < launches.size();) {
        size_t end = at;
        int saved = 0;
        uint64_t on = 0;
        for (; end < launches.size() && small(launches[end]); ++end) {
            saved += gain[launches[end].k];
            for (int j = 0; j < launches[end].k; ++j) on |= uint64_t(1) << launches[end].q[j];
        }
        // planning costs as well: more positions than a pass takes are two passes
        if (end - at < 2 || !worth(__builtin_popcountll(on) > tile_union_limit() ? saved / 2 : saved)) {
            do out.push_back(std::move(launches[at++]));
            while (at < end);
            continue;
        }
        // stages and passes of the run: blocks of <= 4 positions in tile passes
        std::vector<sv_gate> g(end - at);
        for (size_t i = at; i < end; ++i) {
            g[i - at].k = launches[i].k;
            std::copy(launches[i].q, launches[i].q + launches[i].k, g[i - at].q);
        }
        std::vector<Block> blocks;
        if (int rc = fuse_gates(g.data(), int(g.size()), n, 4, SV_RULE_TILED, default_costs(), blocks, false, precision)) return rc;
        const size_t cap = size_t(dev::tile_max_blocks(14, 8, dev::kTileOperandF32));
        for (const auto &grp : tile_groups(blocks, n, precision))
            for (size_t c = 0; c < grp.size(); c += cap) {
                const size_t stop = std::min(grp.size(), c + cap);
                size_t count = 0;
                int pass_saved = 0;
                for (size_t i = c; i < stop; ++i)
                    for (int mem : blocks[grp[i]].members) ++count, pass_saved += gain[launches[at + size_t(mem)].k];
                if (count == 1 || !worth(pass_saved)) {  // the gates alone
                    for (size_t i = c; i < stop; ++i)
                        for (int mem : blocks[grp[i]].members) out.push_back(std::move(launches[at + size_t(mem)]));
                    continue;
                }
                Launch P;
                P.path = PATH_GATES;
                P.k = int(stop - c);
                std::fill(P.q, P.q + SV_MAX_K, 0);
                std::vector<const Block *> bp;
                for (size_t i = c; i < stop; ++i) bp.push_back(&blocks[grp[i]]);
                tile_pass_positions(bp.data(), P.k, n, P.sub_pos);
                for (int s = 0; s < P.k; ++s) {
                    P.stage_gates.push_back(int(bp[size_t(s)]->members.size()));
                    for (int mem : bp[size_t(s)]->members) {
                        const Launch &G = launches[at + size_t(mem)];
                        int b[3] = {0, 0, 0};
                        for (int j = 0; j < G.k; ++j)
                            while (P.sub_pos[s][b[j]] != G.q[j]) ++b[j];
                        P.gates.push_back({G.k, dev::gate_code(G.k, b)});
                        P.m.insert(P.m.end(), G.m.begin(), G.m.end());
                    }
                }
                out.push_back(std::move(P));
            }
        at = end;
    }
    launches.swap(out);
    return SV_OK;
}

// The launch shape of blocks [first, first + m) of a tile pass over one state,
// or two.  A state of few tiles leaves CUs idle, and a workgroup's time is that
// of its blocks one after another: smaller tiles spread the state over more
// CUs with fewer waves each.  Tiles of 2^12 up to 256 of them, else 2^13, else
// the shape that is set; a pass of more positions than the small tile has
// takes the next one.  Seven blocks, (14, 16) against the small shape: FP32 at 14
// qubits 27.8 to 19.0 us, at 20 30.5 to 20.9, at 21 (2^13) 32.7 to 24.5; FP16 at 20 26.4
// to 18.9; FP64 (virtual position 0, 2^14 units of 8 bytes) at 20 45.9 to 30.3; one
// size further on the small tiles lose (FP32, 22 qubits: 35.9 to 39.7).  States of
// 10 and 11 qubits are one tile of 2^10 or 2^11, where a launch for every block
// costs more (eight cycles on a ladder, dense blocks against tiles: FP32 at 10
// qubits 124 to 76 us, at 12 152 to 79, FP64 375 to 67 and 425 to 87).  A shape
// other than the default is kept: the caller or the tuner chose it.
struct TileShape {
    int bits, waves;
};
static TileShape tile_shape_for(const Launch &L, int first, int m, int n, bool two)
{
    const Tuning &T = tuning();
    const bool f64 = L.path == PATH_TILE_FP64;
    if (!f64 && n >= dev::kMinTileQubits && (T.tile_bits != 14 || T.tile_waves != 16)) return {T.tile_bits, T.tile_waves};
    uint64_t u = 1;  // position 0 is in every tile
    for (int s = first; s < first + m; ++s)
        for (int j = 0; j < 4; ++j) u |= uint64_t(1) << (L.sub_pos[s][j] + (f64 ? 1 : 0));
    const int small = n + (f64 ? 1 : 0) + (two ? 1 : 0) - 8;  // 2^8 tiles
    const int bits = std::max(std::max(small, std::min(12, n + (f64 ? 1 : 0))), __builtin_popcountll(u));
    if (bits <= 12) return {bits, 1 << (bits - 10)};
    if (bits == 13) return {13, 8};
    return f64 ? TileShape{dev::kF64TileBits, dev::kF64TileWaves} : TileShape{T.tile_bits, T.tile_waves};
}

// How many blocks of a tile pass, from the first one on, share one launch, and
// the launch's shape: no more than the set shape holds in LDS, which is what
// passes are planned for, and no more than the shape they then take, whose own
// limit may be lower ((13, 8) holds 16 FP32 blocks, (12, 4) 11).
static int tile_chunk(const Launch &L, int first, int n, bool two, TileShape &shape)
{
    const Tuning &T = tuning();
    const int prec = tile_operand_prec(L.path);
    int m = std::min(dev::tile_max_blocks(T.tile_bits, T.tile_waves, prec), L.k - first);
    shape = tile_shape_for(L, first, m, n, two);
    for (int fit; (fit = dev::tile_max_blocks(shape.bits, shape.waves, prec)) < m;) {
        m = fit;
        shape = tile_shape_for(L, first, m, n, two);  // fewer positions may take a smaller shape
    }
    return m;
}

int enqueue(const std::vector<Launch> &launches, int dtype, void *psi, int n, const void *arena, hipStream_t st)
{
    return enqueue(launches.data(), launches.size(), dtype, psi, n, arena, st);
}

int enqueue(const Launch *first, size_t count, int dtype, void *psi, int n, const void *arena, hipStream_t st,
            void *psi2)
{
    const char *A = static_cast<const char *>(arena);
    const Tuning &T = tuning();
    // split-FP16 tile passes of one state: the first writes the norm partials,
    // the later ones take their scale from them (unitary blocks keep the norm,
    // so it is one scale for all of them), and from the second of them to the
    // last the state stays in HBM times that scale: the second scales it at
    // copy-in, the last unscales it at copy-out, the ones between copy it as
    // it is.  Launches in between act on it linearly; the state is plain again
    // when this call's launches end.
    int norm_launches = 0;  // split-FP16 tile launches of this call that take part
    if (!psi2)
        for (const Launch *it = first; it != first + count; ++it)
            if (it->path == PATH_TILE_FP16) {
                TileShape shape;
                for (int c = 0; c < it->k; c += tile_chunk(*it, c, n, false, shape)) ++norm_launches;
            }
    int norm_grid = 0, norm_done = 0;
    for (const Launch *it = first; it != first + count; ++it) {
        const Launch &L = *it;
        if (psi2 && L.path != PATH_REG && L.path != PATH_GENERIC && L.path != PATH_MFMA32 && L.path != PATH_GATES &&
            !is_tile_path(L.path)) {
            // paths without a second-state launch: one launch per state
            if (int rc = enqueue(it, 1, dtype, psi, n, arena, st)) return rc;
            if (int rc = enqueue(it, 1, dtype, psi2, n, arena, st)) return rc;
            continue;
        }
        if (is_tile_path(L.path)) {
            // one launch per chunk of blocks (tile_chunk)
            const size_t op_bytes = 4 * dev::tile_operand_words(tile_operand_prec(L.path));
            const bool use_norm = L.path == PATH_TILE_FP16 && !psi2;
            for (int c = 0, m = 0; c < L.k; c += m) {
                TileShape shape;
                m = tile_chunk(L, c, n, psi2 != nullptr, shape);
                const int per_cu = L.path == PATH_TILE_FP64 ? 1 : dev::tile_wgs_per_cu(shape.bits, shape.waves);
                const int grid_cap = std::min(kTileNormSlots, T.tile_grid_cap * per_cu);
                dev::TileNorm norm;
                int launched = 0;
                if (use_norm) {
                    double *part = reinterpret_cast<double *>(const_cast<char *>(A) + L.norm_off);
                    if (norm_grid > 0) {
                        norm.in = part;
                        norm.n_in = norm_grid;
                        norm.in_scaled = norm_done >= 2;
                        norm.out_scaled = norm_done + 1 < norm_launches;
                    } else {
                        norm.out = part;
                    }
                }
                if (c == 0 && L.basis >= 0) norm.basis = L.basis;  // reads nothing: the state starts here
                LaunchTimer timer(stat_class(path_family(L.path), m), st);
                hipError_t e = dev::launch_tile_pass(m, L.sub_pos + c, A + L.arena_off + c * op_bytes,
                                                     tile_operand_prec(L.path), psi, n, st, grid_cap, shape.bits,
                                                     shape.waves, psi2, norm, &launched);
                if (e != hipSuccess)
                    return fail(SV_ERR_HIP, "tile pass launch (%d blocks): %s", m, hipGetErrorString(e));
                if (norm.out) norm_grid = launched;
                if (use_norm) ++norm_done;
            }
            continue;
        }
        int parts[4] = {0, 0, 0, 0};
        for (const auto &g : L.gates) ++parts[g.first];
        LaunchTimer timer(stat_class(path_family(L.path), L.k), st, L.path == PATH_GATES ? parts : nullptr);
        hipError_t e = hipSuccess;
        switch (L.path) {
        case PATH_GATES:
            e = dev::launch_gate_pass(L.k, L.sub_pos, A + L.arena_off, dtype, psi, n, st, T.tile_grid_cap, psi2);
            break;
        case PATH_REG: e = dev::launch_reg(dtype, L.k, L.q, L.m.data(), psi, n, st, T.reg_grid_cap[L.k], psi2); break;
        case PATH_GENERIC: e = dev::launch_generic(dtype, L.k, L.q, A + L.arena_off, psi, n, st, psi2); break;
        case PATH_MFMA32:
            e = dev::launch_mfma_f32(L.k, L.q, reinterpret_cast<const float *>(A + L.arena_off), psi, n, st,
                                     T.mfma_tc_log[L.k], T.mfma_grid_cap[L.k], psi2);
            break;
        default: {
            const uint16_t *const parts[3] = {reinterpret_cast<const uint16_t *>(A + L.arena_off),
                                              reinterpret_cast<const uint16_t *>(A + L.arena_off2),
                                              reinterpret_cast<const uint16_t *>(A + L.arena_off3)};
            e = dev::launch_mfma_split(L.k, L.path == PATH_SPLIT_FP16, L.q, parts, psi, n, st,
                                       T.split_tc_log[L.k], T.mfma_grid_cap[L.k]);
            break;
        }
        }
        if (e != hipSuccess) return fail(SV_ERR_HIP, "kernel launch (path %d, k=%d): %s", int(L.path), L.k, hipGetErrorString(e));
    }
    return SV_OK;
}

}  // namespace sv
