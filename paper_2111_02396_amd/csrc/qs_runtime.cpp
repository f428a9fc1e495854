// Host runtime behind include/qs.h: state handles, deferred operations,
// Kraus-branch selection, sampling and the trajectory driver.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <array>
#include <atomic>
#include <condition_variable>
#include <functional>
#include <deque>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include "qs.h"
#include "qs_internal.h"
#include "qs_philox.h"
#include "qs_plan.h"
#include "qs_pool.h"

using qs::cd;

namespace {

thread_local std::string g_last_error;

qs_status fail(qs_status st, const std::string &msg) {
    g_last_error = msg;
    return st;
}

constexpr int kDefaultFuse = 4;
constexpr size_t kArenaHalf = size_t(1) << 18;  // float2 per half of the staging ring (2 MiB)
// The ring of a state that has only staged a few small trajectories at a time.
// Device allocations below 2 MiB cost 1 us, larger ones 12 and as much again to
// free, about a tenth of a request that makes a state for one small trajectory.
constexpr size_t kArenaSmallHalf = size_t(1) << 16;
constexpr double kRenormLogThreshold = -46.0;  // ~1e-20 on the norm squared
// Where a sweep that forms a reduced density matrix writes its workgroup
// records in the state's reduction buffer (past the norm pass's records).
constexpr size_t kRdmRecordOffset = size_t(qs::kMaxReduceBlocks);

// qs_sample_measurements draws up to this many samples straight into pinned
// memory; beyond that one copy at the end is cheaper than 8-byte writes over
// the host link.
constexpr int kPinnedSamples = 4096;

struct PendingOp {
    int k;
    int t[5];
    std::vector<cd> m;
};

}  // namespace

struct qs_state_s {
    int n = 0;
    int device = 0;             // the HIP device current when the state was created
    float2 *amp = nullptr;      // where the amplitudes are now
    float2 *home = nullptr;     // where they live between calls
    bool owns_home = false;
    hipStream_t st = nullptr;
    float2 *scratch = nullptr;  // second state for the conventional method
    double *red_partials = nullptr;
    double *red_out = nullptr;
    double *red_host = nullptr;  // pinned; a reduction whose result the host reads
    double *red_host_dev = nullptr;  // ... ends in it directly, with no copy behind it
    double *samp_sums = nullptr;
    double *samp_incl = nullptr;
    double *samp_norm = nullptr;
    uint64_t *samp_out = nullptr;
    size_t samp_cap = 0;
    uint64_t *samp_host = nullptr;  // pinned, kPinnedSamples; its device address
    uint64_t *samp_host_dev = nullptr;
    double *z_dev = nullptr;  // per-trajectory Z-weight records of the driver
    size_t z_cap = 0;         // records
    // matrix staging: two halves of a pinned host buffer mirrored on the
    // device; a half is refilled only after its last copy has completed
    float2 *arena_dev = nullptr;
    float2 *arena_host = nullptr;
    size_t arena_len = 0;        // float2 per half
    hipEvent_t arena_ev[2] = {};
    bool arena_live[2] = {false, false};
    int arena_half = 0;
    size_t arena_head = 0;       // next free float2 in the current half
    size_t arena_committed = 0;  // first float2 not yet copied
    std::vector<PendingOp> pending;
    bool poisoned = false;
    // trajectory-driver buffers kept across calls (allocated on first use)
    float2 *side_buf = nullptr;      // states beside this one, and sweep records
    size_t side_cap = 0;             // bytes
    int *sel_choice_dev = nullptr;   // an error flag, then the device-side picks [kChoiceCap]
    int *sel_choice_host = nullptr;  // pinned mirror
    double *sel_rdm = nullptr;       // the pending channel's reduced density matrix
    float2 *static_buf = nullptr;    // default-plan matrices
    size_t static_cap = 0;           // float2
    uint64_t static_tag = 0;         // cached plan whose matrices static_buf holds (0: none)
    double *chan_dev = nullptr;      // channels' excess matrices and bounds
    size_t chan_cap = 0;             // doubles
    uint64_t chan_tag = 0;           // cached model and mode whose channels chan_dev holds (0: none)
};

namespace {

const int *tile_slots() {
    static const int slots[6] = {0, qs::tile_mat_slots(1), qs::tile_mat_slots(2),
                                 qs::tile_mat_slots(3), qs::tile_mat_slots(4), qs::tile_mat_slots(5)};
    return slots;
}

qs_status device_fail(qs_state s, hipError_t e, const char *what) {
    if (s) s->poisoned = true;
    return fail(QS_ERR_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

#define QS_HIP(s, expr)                                          \
    do {                                                         \
        hipError_t e_ = (expr);                                  \
        if (e_ != hipSuccess) return device_fail((s), e_, #expr); \
    } while (0)

#define QS_CHECK(expr)                   \
    do {                                 \
        qs_status st_ = (expr);          \
        if (st_ != QS_OK) return st_;    \
    } while (0)

qs_status check_handle(qs_state s) {
    if (!s) return fail(QS_ERR_INVALID_ARGUMENT, "null state handle");
    if (s->poisoned) return fail(QS_ERR_DEVICE, "state handle poisoned by an earlier device error");
    return QS_OK;
}

bool finite_matrix(const double *m, size_t n_doubles) {
    for (size_t i = 0; i < n_doubles; ++i)
        if (!std::isfinite(m[i])) return false;
    return true;
}

qs_status check_targets(int n, int k, const int *t, int kmax) {
    if (k < 1 || k > kmax) return fail(QS_ERR_INVALID_ARGUMENT, "k out of range");
    if (k > n) return fail(QS_ERR_INVALID_ARGUMENT, "more targets than qubits");
    if (!t) return fail(QS_ERR_INVALID_ARGUMENT, "null targets");
    for (int i = 0; i < k; ++i) {
        if (t[i] < 0 || t[i] >= n) return fail(QS_ERR_INVALID_ARGUMENT, "target out of range");
        for (int j = 0; j < i; ++j)
            if (t[i] == t[j]) return fail(QS_ERR_INVALID_ARGUMENT, "duplicate target");
    }
    return QS_OK;
}

// GateDesc (ascending targets, complex64) from a complex128 matrix in the
// caller's target order.
void make_desc(int k, const int *t, const cd *m, qs::GateDesc &g) {
    const int D = 1 << k;
    std::vector<cd> sorted(size_t(D) * D);
    int ts[5];
    qs::to_ascending_order(k, t, m, sorted.data(), ts);
    g.k = k;
    for (int b = 0; b < 5; ++b) g.t[b] = b < k ? ts[b] : 0;
    for (int i = 0; i < D * D; ++i)
        g.m[i] = make_float2(float(sorted[i].real()), float(sorted[i].imag()));
}

// Makes the ring's halves hold `len` float2.  Only where nothing is staged
// and no pending launch reads the ring.
qs_status arena_reserve(qs_state s, size_t len) {
    if (s->arena_len >= len) return QS_OK;
    if (s->arena_dev) {
        QS_HIP(s, hipStreamSynchronize(s->st));
        QS_HIP(s, hipFree(s->arena_dev));
        s->arena_dev = nullptr;
        s->arena_len = 0;
        QS_HIP(s, hipHostFree(s->arena_host));
        s->arena_host = nullptr;
    }
    QS_HIP(s, hipMalloc(&s->arena_dev, sizeof(float2) * 2 * len));
    QS_HIP(s, hipHostMalloc(&s->arena_host, sizeof(float2) * 2 * len, hipHostMallocDefault));
    for (int i = 0; i < 2; ++i) {
        if (!s->arena_ev[i]) QS_HIP(s, hipEventCreateWithFlags(&s->arena_ev[i], hipEventDisableTiming));
        s->arena_live[i] = false;
    }
    s->arena_half = 0;
    s->arena_head = s->arena_committed = 0;
    s->arena_len = len;
    return QS_OK;
}

// Copy everything staged since the last commit to the device (one copy).
qs_status arena_commit(qs_state s) {
    if (s->arena_head == s->arena_committed) return QS_OK;
    const size_t base = size_t(s->arena_half) * s->arena_len;
    QS_HIP(s, hipMemcpyAsync(s->arena_dev + base + s->arena_committed,
                             s->arena_host + base + s->arena_committed,
                             sizeof(float2) * (s->arena_head - s->arena_committed),
                             hipMemcpyHostToDevice, s->st));
    QS_HIP(s, hipEventRecord(s->arena_ev[s->arena_half], s->st));
    s->arena_live[s->arena_half] = true;
    s->arena_committed = s->arena_head;
    return QS_OK;
}

// Whether `count` float2 fit in the current half without switching halves.
bool arena_fits(qs_state s, size_t count) {
    return s->arena_head + count <= s->arena_len;
}

// Reserve `count` float2 of staging; returns the host slot and device address.
// A full half is committed and the other half reused once its copy is done.
qs_status arena_stage(qs_state s, size_t count, float2 **host, const float2 **dev) {
    if (!s->arena_dev) QS_CHECK(arena_reserve(s, kArenaHalf));
    if (count > s->arena_len) return fail(QS_ERR_INVALID_ARGUMENT, "matrix staging request too large");
    if (s->arena_head + count > s->arena_len) {
        QS_CHECK(arena_commit(s));
        s->arena_half ^= 1;
        if (s->arena_live[s->arena_half]) QS_HIP(s, hipEventSynchronize(s->arena_ev[s->arena_half]));
        s->arena_live[s->arena_half] = false;
        s->arena_head = s->arena_committed = 0;
    }
    const size_t base = size_t(s->arena_half) * s->arena_len + s->arena_head;
    *host = s->arena_host + base;
    *dev = s->arena_dev + base;
    s->arena_head += (count + 31) & ~size_t(31);  // 256 B alignment
    if (s->arena_head > s->arena_len) s->arena_head = s->arena_len;
    return QS_OK;
}

qs_status enqueue_desc(qs_state s, const qs::GateDesc &g) {
    const size_t dd = size_t(1) << (2 * g.k);
    float2 *h = nullptr;
    const float2 *d = nullptr;
    if (g.k <= qs::kMaxArgGate) {
        QS_HIP(s, qs::launch_apply_gate(s->amp, s->n, g, nullptr, s->st));
        return QS_OK;
    }
    QS_CHECK(arena_stage(s, dd, &h, &d));
    std::memcpy(h, g.m, sizeof(float2) * dd);
    QS_CHECK(arena_commit(s));
    QS_HIP(s, qs::launch_apply_gate(s->amp, s->n, g, d, s->st));
    return QS_OK;
}

qs_status enqueue_matrix(qs_state s, int k, const int *t, const cd *m) {
    qs::GateDesc g;
    make_desc(k, t, m, g);
    return enqueue_desc(s, g);
}

qs_status flush_pending(qs_state s, int max_fuse = kDefaultFuse) {
    if (s->pending.empty()) return QS_OK;
    std::vector<qs::PlanOp> ops(s->pending.size());
    std::vector<const cd *> mats(s->pending.size());
    for (size_t i = 0; i < s->pending.size(); ++i) {
        ops[i].k = s->pending[i].k;
        for (int j = 0; j < 5; ++j) ops[i].q[j] = s->pending[i].t[j];
        mats[i] = s->pending[i].m.data();
    }
    const auto blocks = qs::fuse_greedy(s->n, ops, max_fuse);
    std::vector<cd> M(1024);
    for (const auto &b : blocks) {
        qs::fused_matrix(b.k, b.q, b.ops, ops, mats, M.data());
        cd c;
        if (qs::is_identity_multiple(1 << b.k, M.data(), 1e-15, &c) && std::abs(c - cd(1.0)) < 1e-15)
            continue;
        QS_CHECK(enqueue_matrix(s, b.k, b.q, M.data()));  // b.q ascending already
    }
    s->pending.clear();
    return QS_OK;
}

qs_status ensure_reduce(qs_state s) {
    if (s->red_partials) return QS_OK;
    QS_HIP(s, hipMalloc(&s->red_partials, sizeof(double) * qs::kMaxReduceBlocks * qs::kMaxReduceWidth));
    QS_HIP(s, hipMalloc(&s->red_out, sizeof(double) * qs::kMaxReduceWidth));
    QS_HIP(s, hipHostMalloc(&s->red_host, sizeof(double) * qs::kMaxReduceWidth, hipHostMallocDefault));
    QS_HIP(s, hipHostGetDevicePointer(reinterpret_cast<void **>(&s->red_host_dev), s->red_host, 0));
    return QS_OK;
}

qs_status ensure_sampling(qs_state s, size_t n_out) {
    if (!s->samp_sums) {
        const int B = std::min(s->n, qs::kSampleBlockBits);
        const size_t nb = size_t(1) << (s->n - B);
        QS_HIP(s, hipMalloc(&s->samp_sums, sizeof(double) * nb));
        QS_HIP(s, hipMalloc(&s->samp_incl, sizeof(double) * nb));
        QS_HIP(s, hipMalloc(&s->samp_norm, sizeof(double) * 2));
    }
    if (n_out > s->samp_cap) {
        if (s->samp_out) QS_HIP(s, hipFree(s->samp_out));
        s->samp_out = nullptr;
        s->samp_cap = 0;
        QS_HIP(s, hipMalloc(&s->samp_out, sizeof(uint64_t) * n_out));
        s->samp_cap = n_out;
    }
    return QS_OK;
}

qs_status ensure_scratch(qs_state s) {
    if (s->scratch) return QS_OK;
    const size_t bytes = sizeof(float2) << s->n;
    size_t free_b = 0, total_b = 0;
    QS_HIP(s, hipMemGetInfo(&free_b, &total_b));
    if (free_b < bytes) return fail(QS_ERR_OUT_OF_MEMORY, "no room for the conventional method's second state");
    hipError_t e = hipMalloc(&s->scratch, bytes);
    if (e != hipSuccess) {
        s->scratch = nullptr;
        (void)hipGetLastError();
        return fail(QS_ERR_OUT_OF_MEMORY, "allocating the second state failed");
    }
    return QS_OK;
}

// Sum of |psi|^2 over the current buffer; synchronises.
qs_status device_norm(qs_state s, double *out) {
    QS_CHECK(ensure_reduce(s));
    QS_HIP(s, qs::launch_norm(s->amp, s->n, s->red_partials, s->red_host_dev, s->st));
    QS_HIP(s, hipStreamSynchronize(s->st));
    *out = s->red_host[0];
    return QS_OK;
}

// R = sum_groups v v^dag over ascending targets ts (k <= 2); synchronises.
// R[j][l] = (red_host[2(jD+l)], red_host[2(jD+l)+1]).
qs_status device_rdm(qs_state s, int k, const int *ts) {
    QS_CHECK(ensure_reduce(s));
    QS_HIP(s, qs::launch_rdm(s->amp, s->n, k, ts, s->red_partials, s->red_host_dev, s->st));
    QS_HIP(s, hipStreamSynchronize(s->st));
    return QS_OK;
}

qs_status ensure_zrecords(qs_state s, size_t records) {
    if (records <= s->z_cap) return QS_OK;
    if (s->z_dev) QS_HIP(s, hipFree(s->z_dev));
    s->z_dev = nullptr;
    s->z_cap = 0;
    QS_HIP(s, hipMalloc(&s->z_dev, sizeof(double) * qs::kZRecord * records));
    s->z_cap = records;
    return QS_OK;
}

// <Z_q> = (N - 2 P1[q]) / N from a Z-weight record {N, P1[0..n-1]}.
qs_status z_from_record(int n, const double *rec, double *z) {
    const double N = rec[0];
    if (!(N > 0.0) || !std::isfinite(N)) return fail(QS_ERR_ZERO_NORM, "state has zero norm");
    for (int q = 0; q < n; ++q) z[q] = (N - 2.0 * rec[1 + q]) / N;
    return QS_OK;
}

// Host record of one channel.
struct ChannelInfo {
    int op = -1;
    int k = 0;
    int t[5] = {};
    int ts[5] = {};     // ascending
    int nk = 0;
    const cd *kraus = nullptr;           // nk consecutive D x D (caller order)
    std::vector<double> pbar;
    bool mixture = false;
    std::vector<char> identity;          // K_i proportional to I
    std::vector<cd> unit;                // mixture: K_i / sqrt(pbar_i)
    std::vector<cd> excess_sorted;       // K_i^dag K_i - pbar_i I, ascending-target order
    int default_pick = 0;
    std::vector<double> log_pbar;        // log of pbar_i (norm^2 shrink bound)
};

void build_channel(int k, const int *t, int nk, const cd *kraus, ChannelInfo &c) {
    const int D = 1 << k;
    c.k = k;
    for (int b = 0; b < k; ++b) c.t[b] = t[b];
    c.nk = nk;
    c.kraus = kraus;
    c.pbar.assign(nk, 0.0);
    bool mix = false;
    qs::kraus_bounds(k, nk, kraus, c.pbar.data(), &mix);
    c.mixture = mix;
    c.identity.assign(nk, 0);
    c.unit.assign(size_t(nk) * D * D, cd(0.0));
    c.excess_sorted.assign(size_t(nk) * D * D, cd(0.0));
    c.log_pbar.assign(nk, 0.0);
    std::vector<cd> G(size_t(D) * D);
    for (int i = 0; i < nk; ++i) {
        const cd *K = kraus + size_t(i) * D * D;
        c.identity[i] = qs::is_identity_multiple(D, K, 1e-14, nullptr) ? 1 : 0;
        if (mix && c.pbar[i] > 0.0) {
            const double f = 1.0 / std::sqrt(c.pbar[i]);
            for (int e = 0; e < D * D; ++e) c.unit[size_t(i) * D * D + e] = K[e] * f;
        }
        qs::gram(D, K, G.data());
        for (int j = 0; j < D; ++j) G[j * D + j] -= c.pbar[i];
        qs::to_ascending_order(k, t, G.data(), c.excess_sorted.data() + size_t(i) * D * D, c.ts);
        c.log_pbar[i] = c.mixture ? 0.0 : (c.pbar[i] > 0.0 ? std::log(c.pbar[i]) : -1e300);
    }
    int best = 0;
    for (int i = 1; i < nk; ++i)
        if (c.pbar[i] > c.pbar[best]) best = i;
    c.default_pick = best;
}

// The conventional rule expressed as Algorithm 2: every bound 0, so no pick
// is made from the bounds and the second loop compares the residual r with
// the full p_i = <psi|K_i^dag K_i|psi>/N in order.
void to_conventional(ChannelInfo &c) {
    const int D = 1 << c.k;
    std::vector<cd> G(size_t(D) * D);
    for (int i = 0; i < c.nk; ++i) {
        c.pbar[i] = 0.0;
        c.log_pbar[i] = 0.0;
        qs::gram(D, c.kraus + size_t(i) * D * D, G.data());
        qs::to_ascending_order(c.k, c.t, G.data(), c.excess_sorted.data() + size_t(i) * D * D, c.ts);
    }
    c.mixture = false;
    c.default_pick = 0;
}

// Matrix to apply for pick i picked from the bounds: nullptr = identity
// (a scalar multiple of I is dropped: normalisation is lazy).
const cd *fast_pick_matrix(const ChannelInfo &c, int i) {
    const int D = 1 << c.k;
    if (c.identity[i]) return nullptr;
    if (c.mixture) return c.unit.data() + size_t(i) * D * D;
    return c.kraus + size_t(i) * D * D;
}

// Algorithm 2, steps 1-11: returns the pick, or -1 with *residual set.
int select_fast(const ChannelInfo &c, double r, double *residual) {
    for (int i = 0; i < c.nk; ++i) {
        if (r < c.pbar[i]) return i;
        r -= c.pbar[i];
    }
    if (c.mixture) {
        for (int i = c.nk - 1; i >= 0; --i)
            if (c.pbar[i] > 0.0) return i;
    }
    *residual = r;
    return -1;
}

// Algorithm 2, steps 13-20, from the FP64 reduced density matrix R (ascending
// target order, R[j][l] = sum v_j conj(v_l)).  Returns the pick and p_i.
int select_slow(const ChannelInfo &c, const double *R, double r, double *p_out, double *N_out) {
    const int D = 1 << c.k;
    double N = 0.0;
    for (int j = 0; j < D; ++j) N += R[2 * (j * D + j)];
    *N_out = N;
    int last_pos = -1, pick = -1;
    double e_pick = 0.0;
    std::vector<double> e(c.nk, 0.0);
    for (int i = 0; i < c.nk; ++i) {
        const cd *M = c.excess_sorted.data() + size_t(i) * D * D;
        double tr = 0.0;  // Re sum_jl M[j][l] R[l][j]
        for (int j = 0; j < D; ++j)
            for (int l = 0; l < D; ++l) {
                const cd m = M[j * D + l];
                const double rr = R[2 * (l * D + j)], ri = R[2 * (l * D + j) + 1];
                tr += m.real() * rr - m.imag() * ri;
            }
        e[i] = tr / N;
        if (e[i] > 0.0) last_pos = i;
        if (r < e[i]) {
            pick = i;
            e_pick = e[i];
            break;
        }
        r -= e[i];
    }
    if (pick < 0) {
        pick = last_pos >= 0 ? last_pos : c.nk - 1;
        e_pick = e[pick];
    }
    *p_out = c.pbar[pick] + e_pick;
    return pick;
}

uint32_t channel_draw_index(uint32_t ordinal) { return ordinal; }

// Conventional method for one channel (Section 3.5): trial i writes K_i psi
// to the second state with its norm; r < p_i keeps it.  On return the
// accepted state is current (buffers swapped).
qs_status naive_channel(qs_state s, const ChannelInfo &c, double r, int *pick_out,
                        double *accepted_norm_out) {
    QS_CHECK(ensure_scratch(s));
    QS_CHECK(ensure_reduce(s));
    const int D = 1 << c.k;
    int last_pos = -1;
    int pick = -1;
    double N = 0.0;
    for (int i = 0; i < c.nk; ++i) {
        qs::GateDesc g;
        make_desc(c.k, c.t, c.kraus + size_t(i) * D * D, g);
        QS_HIP(s, qs::launch_apply_copy_norm(s->amp, s->scratch, s->n, g, s->red_partials, s->red_out, s->st));
        QS_HIP(s, hipMemcpyAsync(s->red_host, s->red_out, 2 * sizeof(double), hipMemcpyDeviceToHost, s->st));
        QS_HIP(s, hipStreamSynchronize(s->st));
        N = s->red_host[1];
        if (!(N > 0.0) || !std::isfinite(N)) return fail(QS_ERR_ZERO_NORM, "state has zero norm");
        const double p = s->red_host[0] / N;
        if (p > 0.0) last_pos = i;
        if (r < p) {
            pick = i;
            *accepted_norm_out = s->red_host[0];
            break;
        }
        r -= p;
    }
    if (pick < 0) {
        if (last_pos < 0) return fail(QS_ERR_ZERO_NORM, "every Kraus operator annihilates the state");
        pick = last_pos;
        qs::GateDesc g;
        make_desc(c.k, c.t, c.kraus + size_t(pick) * D * D, g);
        QS_HIP(s, qs::launch_apply_copy_norm(s->amp, s->scratch, s->n, g, s->red_partials, s->red_out, s->st));
        QS_HIP(s, hipMemcpyAsync(s->red_host, s->red_out, 2 * sizeof(double), hipMemcpyDeviceToHost, s->st));
        QS_HIP(s, hipStreamSynchronize(s->st));
        *accepted_norm_out = s->red_host[0];
    }
    std::swap(s->amp, s->scratch);
    *pick_out = pick;
    return QS_OK;
}

qs_status restore_home(qs_state s) {
    if (s->amp == s->home) return QS_OK;
    QS_HIP(s, qs::launch_copy_state(s->home, s->amp, s->n, s->st));
    s->scratch = s->amp;
    s->amp = s->home;
    return QS_OK;
}

qs_status renormalize_now(qs_state s) {
    double N = 0.0;
    QS_CHECK(device_norm(s, &N));
    if (!(N > 0.0) || !std::isfinite(N)) return fail(QS_ERR_ZERO_NORM, "state has zero norm");
    QS_HIP(s, qs::launch_scale(s->amp, s->n, float(1.0 / std::sqrt(N)), s->st));
    return QS_OK;
}

}  // namespace

// ===================================================================== ABI

extern "C" {

const char *qs_last_error_message(void) { return g_last_error.c_str(); }

const char *qs_version(void) { return "qs-mi355x 0.1"; }

qs_status qs_philox4x32_10(const uint32_t ctr[4], const uint32_t key[2], uint32_t out[4]) {
    if (!ctr || !key || !out) return fail(QS_ERR_INVALID_ARGUMENT, "null argument");
    const qs::PhiloxWords w = qs::philox4x32_10(ctr[0], ctr[1], ctr[2], ctr[3], key[0], key[1]);
    for (int i = 0; i < 4; ++i) out[i] = w.w[i];
    return QS_OK;
}

qs_status qs_kraus_bounds(int k, int n_kraus, const double *kraus, double *pbar_out,
                          int *mixture_out) {
    if (k < 1 || k > qs::kMaxGateQubits || n_kraus < 1 || n_kraus > 64 || !kraus || !pbar_out ||
        !mixture_out)
        return fail(QS_ERR_INVALID_ARGUMENT, "bad arguments");
    const int D = 1 << k;
    if (!finite_matrix(kraus, size_t(n_kraus) * D * D * 2))
        return fail(QS_ERR_INVALID_ARGUMENT, "non-finite Kraus entries");
    bool mix = false;
    qs::kraus_bounds(k, n_kraus, reinterpret_cast<const cd *>(kraus), pbar_out, &mix);
    *mixture_out = mix ? 1 : 0;
    return QS_OK;
}

qs_status qs_create_state(int n_qubits, void *device_buf, size_t buf_bytes, void *hip_stream,
                          qs_state *out) {
    if (!out) return fail(QS_ERR_INVALID_ARGUMENT, "null output handle");
    *out = nullptr;
    if (n_qubits < 1 || n_qubits > qs::kMaxQubits) return fail(QS_ERR_INVALID_ARGUMENT, "n out of range");
    const size_t bytes = sizeof(float2) << n_qubits;
    if (device_buf && buf_bytes < bytes) return fail(QS_ERR_INVALID_ARGUMENT, "buffer smaller than 8*2^n bytes");
    if (device_buf && (reinterpret_cast<uintptr_t>(device_buf) & 15u) != 0)
        return fail(QS_ERR_INVALID_ARGUMENT, "buffer not 16-byte aligned");
    auto *s = new qs_state_s();
    s->n = n_qubits;
    if (hipGetDevice(&s->device) != hipSuccess) s->device = 0;
    s->st = static_cast<hipStream_t>(hip_stream);
    if (device_buf) {
        s->home = static_cast<float2 *>(device_buf);
    } else {
        size_t free_b = 0, total_b = 0;
        hipError_t e = hipMemGetInfo(&free_b, &total_b);
        if (e != hipSuccess) {
            delete s;
            return fail(QS_ERR_DEVICE, std::string("hipMemGetInfo: ") + hipGetErrorString(e));
        }
        if (free_b < bytes) {
            delete s;
            return fail(QS_ERR_OUT_OF_MEMORY, "free device memory below 8*2^n bytes");
        }
        e = hipMalloc(&s->home, bytes);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            delete s;
            return fail(QS_ERR_OUT_OF_MEMORY, std::string("hipMalloc: ") + hipGetErrorString(e));
        }
        s->owns_home = true;
    }
    s->amp = s->home;
    hipError_t e = qs::launch_set_basis(s->amp, s->n, 0, s->st);
    if (e != hipSuccess) {
        if (s->owns_home) (void)hipFree(s->home);
        delete s;
        return fail(QS_ERR_DEVICE, std::string("init: ") + hipGetErrorString(e));
    }
    *out = s;
    return QS_OK;
}

qs_status qs_destroy_state(qs_state s) {
    if (!s) return fail(QS_ERR_INVALID_ARGUMENT, "null state handle");
    (void)hipStreamSynchronize(s->st);
    // {amp, scratch} = {home, second buffer} as a set, whatever swaps happened
    float2 *second = s->amp != s->home ? s->amp : s->scratch;
    if (s->owns_home) (void)hipFree(s->home);
    if (second && second != s->home) (void)hipFree(second);
    if (s->red_partials) (void)hipFree(s->red_partials);
    if (s->red_out) (void)hipFree(s->red_out);
    if (s->red_host) (void)hipHostFree(s->red_host);
    if (s->samp_sums) (void)hipFree(s->samp_sums);
    if (s->samp_incl) (void)hipFree(s->samp_incl);
    if (s->samp_norm) (void)hipFree(s->samp_norm);
    if (s->samp_out) (void)hipFree(s->samp_out);
    if (s->samp_host) (void)hipHostFree(s->samp_host);
    if (s->z_dev) (void)hipFree(s->z_dev);
    if (s->arena_dev) (void)hipFree(s->arena_dev);
    if (s->arena_host) (void)hipHostFree(s->arena_host);
    for (int i = 0; i < 2; ++i)
        if (s->arena_ev[i]) (void)hipEventDestroy(s->arena_ev[i]);
    if (s->side_buf) (void)hipFree(s->side_buf);
    if (s->sel_choice_dev) (void)hipFree(s->sel_choice_dev);
    if (s->sel_choice_host) (void)hipHostFree(s->sel_choice_host);
    if (s->sel_rdm) (void)hipFree(s->sel_rdm);
    if (s->static_buf) (void)hipFree(s->static_buf);
    if (s->chan_dev) (void)hipFree(s->chan_dev);
    delete s;
    return QS_OK;
}

qs_status qs_reset_state(qs_state s) {
    QS_CHECK(check_handle(s));
    s->pending.clear();
    QS_CHECK(restore_home(s));
    QS_HIP(s, qs::launch_set_basis(s->amp, s->n, 0, s->st));
    return QS_OK;
}

qs_status qs_state_device_ptr(qs_state s, void **out) {
    QS_CHECK(check_handle(s));
    if (!out) return fail(QS_ERR_INVALID_ARGUMENT, "null output");
    *out = s->amp;
    return QS_OK;
}

qs_status qs_state_qubits(qs_state s, int *n_out) {
    if (!s || !n_out) return fail(QS_ERR_INVALID_ARGUMENT, "null argument");
    *n_out = s->n;
    return QS_OK;
}

qs_status qs_flush(qs_state s) {
    QS_CHECK(check_handle(s));
    return flush_pending(s);
}

qs_status qs_copy_state_to_host(qs_state s, void *host_out, size_t bytes) {
    QS_CHECK(check_handle(s));
    const size_t need = sizeof(float2) << s->n;
    if (!host_out || bytes < need) return fail(QS_ERR_INVALID_ARGUMENT, "host buffer too small");
    QS_CHECK(flush_pending(s));
    QS_HIP(s, hipStreamSynchronize(s->st));
    QS_HIP(s, hipMemcpy(host_out, s->amp, need, hipMemcpyDeviceToHost));
    return QS_OK;
}

qs_status qs_load_state_from_host(qs_state s, const void *host_in, size_t bytes) {
    QS_CHECK(check_handle(s));
    const size_t need = sizeof(float2) << s->n;
    if (!host_in || bytes < need) return fail(QS_ERR_INVALID_ARGUMENT, "host buffer too small");
    s->pending.clear();
    QS_CHECK(restore_home(s));
    QS_HIP(s, hipStreamSynchronize(s->st));
    QS_HIP(s, hipMemcpy(s->amp, host_in, need, hipMemcpyHostToDevice));
    return QS_OK;
}

qs_status qs_copy_state(qs_state dst, qs_state src) {
    QS_CHECK(check_handle(dst));
    QS_CHECK(check_handle(src));
    if (dst == src) return QS_OK;
    if (dst->n != src->n) return fail(QS_ERR_INVALID_ARGUMENT, "states differ in qubit count");
    if (dst->device != src->device) return fail(QS_ERR_NOT_SUPPORTED, "states on different devices");
    QS_CHECK(flush_pending(src));
    dst->pending.clear();
    QS_CHECK(restore_home(dst));
    hipEvent_t ready = nullptr, done = nullptr;
    struct EvGuard {
        hipEvent_t *a, *b;
        ~EvGuard() {
            if (*a) (void)hipEventDestroy(*a);
            if (*b) (void)hipEventDestroy(*b);
        }
    } guard{&ready, &done};
    const bool two = src->st != dst->st;
    if (two) {
        QS_HIP(dst, hipEventCreateWithFlags(&ready, hipEventDisableTiming));
        QS_HIP(dst, hipEventCreateWithFlags(&done, hipEventDisableTiming));
        QS_HIP(src, hipEventRecord(ready, src->st));
        QS_HIP(dst, hipStreamWaitEvent(dst->st, ready, 0));
    }
    QS_HIP(dst, qs::launch_copy_state(dst->amp, src->amp, dst->n, dst->st));
    if (two) {
        QS_HIP(dst, hipEventRecord(done, dst->st));
        QS_HIP(src, hipStreamWaitEvent(src->st, done, 0));
    }
    return QS_OK;
}

qs_status qs_apply_fused_gate(qs_state s, int k, const int *targets, const double *matrix) {
    QS_CHECK(check_handle(s));
    QS_CHECK(check_targets(s->n, k, targets, qs::kMaxGateQubits));
    if (!matrix) return fail(QS_ERR_INVALID_ARGUMENT, "null matrix");
    const int D = 1 << k;
    if (!finite_matrix(matrix, size_t(D) * D * 2)) return fail(QS_ERR_INVALID_ARGUMENT, "non-finite matrix");
    QS_CHECK(flush_pending(s));
    return enqueue_matrix(s, k, targets, reinterpret_cast<const cd *>(matrix));
}

qs_status qs_apply_channel(qs_state s, int k, const int *targets, int n_kraus,
                           const double *kraus, uint64_t seed, uint32_t traj,
                           uint32_t channel_index, qs_kraus_mode mode, int *chosen_out,
                           int *path_out) {
    QS_CHECK(check_handle(s));
    if (k > qs::kMaxChannelQubits && k <= qs::kMaxGateQubits)
        return fail(QS_ERR_NOT_SUPPORTED, "channels act on at most 2 qubits");
    QS_CHECK(check_targets(s->n, k, targets, qs::kMaxChannelQubits));
    if (n_kraus < 1 || n_kraus > 16 || !kraus) return fail(QS_ERR_INVALID_ARGUMENT, "bad Kraus list");
    if (mode != QS_KRAUS_DELAYED && mode != QS_KRAUS_NAIVE && mode != QS_KRAUS_CONVENTIONAL_INPLACE)
        return fail(QS_ERR_INVALID_ARGUMENT, "bad mode");
    const int D = 1 << k;
    if (!finite_matrix(kraus, size_t(n_kraus) * D * D * 2))
        return fail(QS_ERR_INVALID_ARGUMENT, "non-finite Kraus entries");
    ChannelInfo c;
    build_channel(k, targets, n_kraus, reinterpret_cast<const cd *>(kraus), c);
    if (mode == QS_KRAUS_CONVENTIONAL_INPLACE) to_conventional(c);
    const double r = qs::philox_uniform(seed, channel_draw_index(channel_index), traj, 0,
                                        qs::kStreamChannel);
    int pick = -1, path = 0;
    if (mode == QS_KRAUS_DELAYED || mode == QS_KRAUS_CONVENTIONAL_INPLACE) {
        double residual = 0.0;
        pick = select_fast(c, r, &residual);
        if (pick >= 0) {
            const cd *M = fast_pick_matrix(c, pick);
            if (M) {
                PendingOp op;
                op.k = k;
                for (int b = 0; b < 5; ++b) op.t[b] = b < k ? targets[b] : 0;
                op.m.assign(M, M + D * D);
                s->pending.push_back(std::move(op));
            }
        } else {
            path = 1;
            QS_CHECK(flush_pending(s));
            QS_CHECK(device_rdm(s, k, c.ts));
            double p = 0.0, N = 0.0;
            pick = select_slow(c, s->red_host, residual, &p, &N);
            if (!(N > 0.0) || !std::isfinite(N)) return fail(QS_ERR_ZERO_NORM, "state has zero norm");
            if (!(p > 0.0)) return fail(QS_ERR_ZERO_NORM, "chosen Kraus operator has zero weight");
            const double f = 1.0 / std::sqrt(p * N);
            PendingOp op;
            op.k = k;
            for (int b = 0; b < 5; ++b) op.t[b] = b < k ? targets[b] : 0;
            op.m.resize(D * D);
            const cd *K = c.kraus + size_t(pick) * D * D;
            for (int e = 0; e < D * D; ++e) op.m[e] = K[e] * f;
            s->pending.push_back(std::move(op));
        }
    } else {
        path = 1;
        QS_CHECK(flush_pending(s));
        double accepted = 0.0;
        QS_CHECK(naive_channel(s, c, r, &pick, &accepted));
        if (!(accepted > 0.0)) return fail(QS_ERR_ZERO_NORM, "chosen Kraus operator has zero weight");
        // |psi> <- K_i |psi> / sqrt(p_i) up to the lazily kept norm; rescale
        // only when the stored norm leaves a safe float range
        if (accepted < 1e-20 || accepted > 1e20)
            QS_HIP(s, qs::launch_scale(s->amp, s->n, float(1.0 / std::sqrt(accepted)), s->st));
        if (s->home != s->amp && !s->owns_home) QS_CHECK(restore_home(s));
    }
    if (chosen_out) *chosen_out = pick;
    if (path_out) *path_out = path;
    return QS_OK;
}

qs_status qs_norm(qs_state s, double *norm_sq_out) {
    QS_CHECK(check_handle(s));
    if (!norm_sq_out) return fail(QS_ERR_INVALID_ARGUMENT, "null output");
    QS_CHECK(flush_pending(s));
    return device_norm(s, norm_sq_out);
}

qs_status qs_expectation_z(qs_state s, double *z_out) {
    QS_CHECK(check_handle(s));
    if (!z_out) return fail(QS_ERR_INVALID_ARGUMENT, "null output");
    QS_CHECK(flush_pending(s));
    QS_CHECK(ensure_reduce(s));
    QS_HIP(s, qs::launch_zweights(s->amp, s->n, s->red_partials, s->red_host_dev, s->st));
    QS_HIP(s, hipStreamSynchronize(s->st));
    return z_from_record(s->n, s->red_host, z_out);
}

qs_status qs_expectation(qs_state s, int k, const int *targets, const double *observable,
                         double *value_out) {
    QS_CHECK(check_handle(s));
    if (!targets || !observable || !value_out) return fail(QS_ERR_INVALID_ARGUMENT, "null argument");
    if (k < 1 || k > qs::kMaxChannelQubits)
        return fail(QS_ERR_NOT_SUPPORTED, "observables act on one or two qubits");
    for (int a = 0; a < k; ++a) {
        if (targets[a] < 0 || targets[a] >= s->n) return fail(QS_ERR_INVALID_ARGUMENT, "target out of range");
        for (int b = 0; b < a; ++b)
            if (targets[a] == targets[b]) return fail(QS_ERR_INVALID_ARGUMENT, "repeated target");
    }
    const int D = 1 << k;
    const cd *O = reinterpret_cast<const cd *>(observable);
    double scale = 0.0;
    for (int i = 0; i < D * D; ++i) {
        if (!std::isfinite(O[i].real()) || !std::isfinite(O[i].imag()))
            return fail(QS_ERR_INVALID_ARGUMENT, "observable has a non-finite entry");
        scale = std::max(scale, std::abs(O[i]));
    }
    for (int i = 0; i < D; ++i)
        for (int j = 0; j < D; ++j)
            if (std::abs(O[i * D + j] - std::conj(O[j * D + i])) > 1e-12 * std::max(scale, 1.0))
                return fail(QS_ERR_INVALID_ARGUMENT, "observable is not Hermitian");
    std::vector<cd> Os(size_t(D) * D);
    int ts[qs::kMaxChannelQubits];
    qs::to_ascending_order(k, targets, O, Os.data(), ts);
    QS_CHECK(flush_pending(s));
    QS_CHECK(device_rdm(s, k, ts));
    // <psi|O|psi> = sum_{j,l} O[j][l] R[l][j] with R[l][j] = v_l conj(v_j) summed over groups
    const double *R = s->red_host;
    double N = 0.0, acc = 0.0;
    for (int j = 0; j < D; ++j) {
        N += R[2 * (j * D + j)];
        for (int l = 0; l < D; ++l) {
            const cd r(R[2 * (l * D + j)], R[2 * (l * D + j) + 1]);
            acc += (Os[size_t(j) * D + l] * r).real();
        }
    }
    if (!(N > 0.0) || !std::isfinite(N)) return fail(QS_ERR_ZERO_NORM, "state has zero norm");
    *value_out = acc / N;
    return QS_OK;
}

namespace {

qs_status fill_readout(int n, const double *p0to1, const double *p1to0, qs::ReadoutDesc &ro) {
    std::memset(&ro, 0, sizeof(ro));
    if (!p0to1 && !p1to0) return QS_OK;
    if (!p0to1 || !p1to0) return fail(QS_ERR_INVALID_ARGUMENT, "give both readout arrays or neither");
    for (int q = 0; q < n; ++q) {
        if (!(p0to1[q] >= 0.0 && p0to1[q] <= 1.0 && p1to0[q] >= 0.0 && p1to0[q] <= 1.0))
            return fail(QS_ERR_INVALID_ARGUMENT, "readout probability outside [0, 1]");
        ro.e0[q] = p0to1[q];
        ro.e1[q] = p1to0[q];
    }
    ro.enabled = 1;
    return QS_OK;
}

}  // namespace

qs_status qs_sample_measurements(qs_state s, uint64_t seed, uint32_t traj, int n_samples,
                                 const double *p0to1, const double *p1to0,
                                 uint64_t *bitstrings_out) {
    QS_CHECK(check_handle(s));
    if (n_samples < 0 || (n_samples > 0 && !bitstrings_out))
        return fail(QS_ERR_INVALID_ARGUMENT, "bad sample arguments");
    qs::ReadoutDesc ro;
    QS_CHECK(fill_readout(s->n, p0to1, p1to0, ro));
    QS_CHECK(flush_pending(s));
    QS_CHECK(ensure_sampling(s, size_t(std::max(n_samples, 1))));
    QS_CHECK(ensure_reduce(s));
    if (!s->samp_host) {
        QS_HIP(s, hipHostMalloc(&s->samp_host, sizeof(uint64_t) * kPinnedSamples, hipHostMallocDefault));
        QS_HIP(s, hipHostGetDevicePointer(reinterpret_cast<void **>(&s->samp_host_dev), s->samp_host, 0));
    }
    // few samples are drawn straight into pinned memory; the norm always is
    const bool direct = n_samples <= kPinnedSamples;
    QS_HIP(s, qs::launch_sample(s->amp, s->n, s->samp_sums, s->samp_incl, seed, traj, 0, n_samples, ro,
                                direct ? s->samp_host_dev : s->samp_out, s->samp_norm, s->st, s->red_host_dev));
    QS_HIP(s, hipStreamSynchronize(s->st));
    const double N = s->red_host[0];
    if (!(N > 0.0) || !std::isfinite(N)) return fail(QS_ERR_ZERO_NORM, "state has zero norm");
    if (direct && n_samples > 0)
        std::memcpy(bitstrings_out, s->samp_host, sizeof(uint64_t) * size_t(n_samples));
    else if (n_samples > 0)
        QS_HIP(s, hipMemcpy(bitstrings_out, s->samp_out, sizeof(uint64_t) * n_samples, hipMemcpyDeviceToHost));
    return QS_OK;
}

qs_status qs_sample_measurements_noalloc(qs_state s, uint64_t seed, uint32_t traj, int n_samples,
                                         const double *p0to1, const double *p1to0,
                                         uint64_t *bitstrings_out) {
    QS_CHECK(check_handle(s));
    if (n_samples < 0 || (n_samples > 0 && !bitstrings_out))
        return fail(QS_ERR_INVALID_ARGUMENT, "bad sample arguments");
    if (s->n > qs::kNoAllocMaxQubits)
        return fail(QS_ERR_INVALID_ARGUMENT,
                    "allocation-free sampling takes states of at most 28 qubits");
    if (n_samples > qs::kNoAllocMaxSamples)
        return fail(QS_ERR_INVALID_ARGUMENT,
                    "allocation-free sampling draws at most 65536 samples per call");
    if (!s->pending.empty())
        return fail(QS_ERR_INVALID_ARGUMENT,
                    "deferred operations pending: call qs_flush before allocation-free sampling");
    qs::ReadoutDesc ro;
    QS_CHECK(fill_readout(s->n, p0to1, p1to0, ro));
    double *base = nullptr;
    QS_HIP(s, qs::noalloc_scratch(s->device, &base));
    double *sums = base, *incl = base + qs::kNoAllocBlocks, *norm = base + qs::kNoAllocNormOffset;
    uint64_t *out = reinterpret_cast<uint64_t *>(base + qs::kNoAllocOutOffset);
    QS_HIP(s, qs::launch_sample(s->amp, s->n, sums, incl, seed, traj, 0, n_samples, ro, out, norm,
                                s->st));
    double N = 0.0;
    QS_HIP(s, hipMemcpyAsync(&N, norm, sizeof(double), hipMemcpyDeviceToHost, s->st));
    QS_HIP(s, hipStreamSynchronize(s->st));
    if (!(N > 0.0) || !std::isfinite(N)) return fail(QS_ERR_ZERO_NORM, "state has zero norm");
    if (n_samples > 0) {
        QS_HIP(s, hipMemcpyAsync(bitstrings_out, out, sizeof(uint64_t) * n_samples,
                                 hipMemcpyDeviceToHost, s->st));
        QS_HIP(s, hipStreamSynchronize(s->st));
    }
    return QS_OK;
}

// --------------------------------------------------------------------------
// Trajectory driver.
// --------------------------------------------------------------------------

namespace {

struct CircuitModel {
    int n = 0;
    std::vector<qs::PlanOp> ops;
    std::vector<int> kind;
    std::vector<const cd *> gate_mat;    // gates: matrix; channels: nullptr
    std::vector<double> gate_log_bound;  // log sigma_min^2 of a gate matrix (0 if unitary)
    std::vector<int> channel_of_op;      // -1 for gates
    std::vector<ChannelInfo> channels;
};

qs_status build_model(const qs_circuit *c, CircuitModel &m) {
    if (!c || !c->ops || c->n_ops < 0 || !c->mat_pool || c->pool_len < 0)
        return fail(QS_ERR_INVALID_ARGUMENT, "bad circuit");
    m.n = c->n_qubits;
    const cd *pool = reinterpret_cast<const cd *>(c->mat_pool);
    if (!finite_matrix(c->mat_pool, size_t(c->pool_len) * 2))
        return fail(QS_ERR_INVALID_ARGUMENT, "non-finite matrix entries");
    m.ops.resize(c->n_ops);
    m.kind.resize(c->n_ops);
    m.gate_mat.assign(c->n_ops, nullptr);
    m.gate_log_bound.assign(c->n_ops, 0.0);
    m.channel_of_op.assign(c->n_ops, -1);
    std::vector<cd> G(1024);
    for (int o = 0; o < c->n_ops; ++o) {
        const qs_op &op = c->ops[o];
        const int kmax = op.kind == QS_OP_GATE ? qs::kMaxGateQubits : qs::kMaxChannelQubits;
        if (op.kind != QS_OP_GATE && op.kind != QS_OP_CHANNEL)
            return fail(QS_ERR_INVALID_ARGUMENT, "bad op kind");
        if (op.kind == QS_OP_CHANNEL && op.k > qs::kMaxChannelQubits && op.k <= qs::kMaxGateQubits)
            return fail(QS_ERR_NOT_SUPPORTED, "channels act on at most 2 qubits");
        QS_CHECK(check_targets(m.n, op.k, op.targets, kmax));
        const int D = 1 << op.k;
        const int nm = op.kind == QS_OP_GATE ? 1 : op.n_mats;
        if (nm < 1 || nm > 16 || (op.kind == QS_OP_GATE && op.n_mats != 1))
            return fail(QS_ERR_INVALID_ARGUMENT, "bad matrix count");
        if (op.mat_offset < 0 || op.mat_offset + int64_t(nm) * D * D > c->pool_len)
            return fail(QS_ERR_INVALID_ARGUMENT, "matrix outside the pool");
        m.ops[o].k = op.k;
        for (int b = 0; b < 5; ++b) m.ops[o].q[b] = b < op.k ? op.targets[b] : 0;
        m.kind[o] = op.kind;
        if (op.kind == QS_OP_GATE) {
            m.gate_mat[o] = pool + op.mat_offset;
            qs::gram(D, m.gate_mat[o], G.data());
            if (!qs::is_identity_multiple(D, G.data(), 1e-12, nullptr)) {
                const double lam = qs::hermitian_min_eigenvalue(D, G.data());
                m.gate_log_bound[o] = lam > 0 ? std::log(lam) : -1e300;
            } else {
                const double c0 = G[0].real();
                m.gate_log_bound[o] = c0 > 0 ? std::log(c0) : -1e300;
            }
        } else {
            ChannelInfo ci;
            build_channel(op.k, op.targets, nm, pool + op.mat_offset, ci);
            ci.op = o;
            m.channel_of_op[o] = int(m.channels.size());
            m.channels.push_back(std::move(ci));
        }
    }
    return QS_OK;
}

struct BlockDesc {
    qs::GateDesc g;
    bool identity = false;
    double log_bound = 0.0;
    const float2 *dev = nullptr;  // device copy of g.m, or null:
    size_t static_off = 0;        // a plan's block, at this offset of the call's static matrices
};

// Stage a block's matrix in the arena (committed later, before its launch).
qs_status stage_block(qs_state s, BlockDesc &d) {
    if (d.identity) return QS_OK;
    const size_t dd = size_t(1) << (2 * d.g.k);
    float2 *h = nullptr;
    QS_CHECK(arena_stage(s, dd, &h, &d.dev));
    std::memcpy(h, d.g.m, sizeof(float2) * dd);
    return QS_OK;
}

// Build a GateDesc for members (time-ordered) under the given per-op matrices.
void build_block(const CircuitModel &m, const std::vector<int> &members,
                 const std::vector<const cd *> &mats, std::vector<cd> &tmp, BlockDesc &out) {
    int q[5];
    const int k = qs::union_qubits(members, m.ops, q);
    tmp.resize(size_t(1) << (2 * k));
    qs::fused_matrix(k, q, members, m.ops, mats, tmp.data());
    cd c;
    out.identity = qs::is_identity_multiple(1 << k, tmp.data(), 1e-15, &c) && std::abs(c - cd(1.0)) < 1e-15;
    out.g.k = k;
    for (int b = 0; b < 5; ++b) out.g.t[b] = b < k ? q[b] : 0;
    const int D = 1 << k;
    for (int i = 0; i < D * D; ++i) out.g.m[i] = make_float2(float(tmp[i].real()), float(tmp[i].imag()));
}

// Event pairs around kernel launches, harvested lazily so the host never
// waits on recent work.
// HIP-event timing of the fused-gate sweeps.  One event pair brackets a run
// of sweep launches issued back to back (a segment's units); the run's time is
// divided over its launches, so the per-launch figure carries no event
// overhead of its own.  A bracket is closed before any other kernel is
// launched.  A ring of brackets is harvested as it wraps.
struct KernelTimer {
    std::vector<hipEvent_t> ev;
    std::vector<int> launches;  // per bracket: 0 = not pending
    int pos = 0;
    bool open_now = false;
    int cur = 0;
    double total_ms = 0.0;
    int64_t count = 0;
    // optional: every bracket as (start, end) in ms after `ref` (a completed
    // event), so that brackets of several streams can be merged
    hipEvent_t ref = nullptr;
    std::vector<std::pair<double, double>> *intervals = nullptr;

    ~KernelTimer() {
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
    }
    qs_status init(qs_state s, int cap) {
        ev.assign(size_t(2) * cap, nullptr);
        launches.assign(cap, 0);
        // timing only: no system-scope fence (with one, every record writes
        // back and invalidates the L2, which costs the timed sweeps ~10 %)
        for (auto &e : ev) QS_HIP(s, hipEventCreateWithFlags(&e, hipEventDisableSystemFence));
        return QS_OK;
    }
    qs_status harvest(qs_state s, int slot) {
        if (!launches[slot]) return QS_OK;
        QS_HIP(s, hipEventSynchronize(ev[2 * slot + 1]));
        float ms = 0.f;
        QS_HIP(s, hipEventElapsedTime(&ms, ev[2 * slot], ev[2 * slot + 1]));
        total_ms += ms;
        if (ref && intervals) {
            float t0 = 0.f;
            QS_HIP(s, hipEventElapsedTime(&t0, ref, ev[2 * slot]));
            intervals->emplace_back(double(t0), double(t0) + double(ms));
        }
        count += launches[slot];
        launches[slot] = 0;
        return QS_OK;
    }
    // before a sweep launch
    qs_status open(qs_state s) {
        if (open_now) return QS_OK;
        QS_CHECK(harvest(s, pos));
        QS_HIP(s, hipEventRecord(ev[2 * pos], s->st));
        open_now = true;
        cur = 0;
        return QS_OK;
    }
    // after a sweep launch
    void launched() { ++cur; }
    void launched_n(int k) { cur += k; }
    // before any other kernel, and at the end of a run of sweeps
    qs_status close(qs_state s) {
        if (!open_now) return QS_OK;
        QS_HIP(s, hipEventRecord(ev[2 * pos + 1], s->st));
        launches[pos] = cur;  // a bracket with no launches is never harvested
        pos = (pos + 1) % int(launches.size());
        open_now = false;
        return QS_OK;
    }
    qs_status finish(qs_state s) {
        QS_CHECK(close(s));
        for (int i = 0; i < int(launches.size()); ++i) QS_CHECK(harvest(s, i));
        return QS_OK;
    }
};

// ---- per-circuit plan cache
// The default plan of a circuit (fusion into blocks, their matrices, the tile
// sweep grouping) depends only on the circuit, the mode's channel bounds, the
// widths and the grouping's restarts, so calls that run the same circuit again (one state per call,
// a serving loop, the autotuner's final choice) reuse it instead of fusing
// again.  Keyed by the circuit's model-cache id.
struct PlanKey {
    uint64_t hash;  // model id
    int n, mode, f, tb, restarts;
    bool operator<(const PlanKey &o) const {
        return std::tie(hash, n, mode, f, tb, restarts) <
               std::tie(o.hash, o.n, o.mode, o.f, o.tb, o.restarts);
    }
};

struct TileLayout {
    bool tiled = false;
    int tb = 0;
    int pos[qs::kMaxTileBits] = {};
    int8_t local[qs::kMaxQubits] = {};

    // Tile layout of a sweep: its qubits plus the lowest others up to the tile
    // width (at least 10 bits, and k + 8 for its widest block).
    static TileLayout of(int n, const qs::Sweep &sw, const std::vector<qs::Block> &bl) {
        TileLayout L;
        const auto &bits = sw.bits;
        if (bits.empty() || int(bits.size()) > qs::kMaxTileBits) return L;
        int maxk = 1;
        for (int b : sw.blocks) maxk = std::max(maxk, bl[b].k);
        int tb = std::max<int>(int(bits.size()), std::min(qs::kMaxTileBits, std::max(10, maxk + 8)));
        tb = std::min(tb, n);
        std::vector<char> in(n, 0);
        for (int q : bits) in[q] = 1;
        int cnt = int(bits.size());
        for (int q = 0; q < n && cnt < tb; ++q)
            if (!in[q]) {
                in[q] = 1;
                ++cnt;
            }
        L.tb = tb;
        int i = 0;
        for (int q = 0; q < qs::kMaxQubits; ++q) L.local[q] = -1;
        for (int q = 0; q < n; ++q)
            if (in[q]) {
                L.pos[i] = q;
                L.local[q] = int8_t(i);
                ++i;
            }
        L.tiled = true;
        return L;
    }
};

struct PlanEntry {
    std::vector<qs::Block> blocks;
    std::vector<int> op_block;
    std::vector<BlockDesc> block_desc;  // device copies not set, static offsets are
    std::vector<qs::Sweep> sweeps;
    std::vector<TileLayout> layouts;
    size_t static_len = 0;              // float2 of the blocks' matrices
};

constexpr size_t kPlanCacheEntries = 32;
std::mutex g_plan_mu;
std::map<PlanKey, std::shared_ptr<const PlanEntry>> g_plan_cache;
std::deque<PlanKey> g_plan_fifo;

void plan_lookup(const PlanKey &k, std::shared_ptr<const PlanEntry> *out) {
    std::lock_guard<std::mutex> lock(g_plan_mu);
    auto it = g_plan_cache.find(k);
    *out = it == g_plan_cache.end() ? nullptr : it->second;
}

void plan_insert(const PlanKey &k, std::shared_ptr<const PlanEntry> e) {
    std::lock_guard<std::mutex> lock(g_plan_mu);
    if (g_plan_cache.count(k)) return;
    if (g_plan_fifo.size() >= kPlanCacheEntries) {
        g_plan_cache.erase(g_plan_fifo.front());
        g_plan_fifo.pop_front();
    }
    g_plan_cache[k] = std::move(e);
    g_plan_fifo.push_back(k);
}

// Hash of the circuit's qubit count, op records and matrix pool, eight bytes
// at a time (a cache key only: the model cache below compares the bytes).
uint64_t circuit_hash(const qs_circuit *c) {
    uint64_t h = 0x9e3779b97f4a7c15ull ^ uint64_t(uint32_t(c->n_qubits));
    auto mix = [&h](const void *p, size_t len) {
        const unsigned char *b = static_cast<const unsigned char *>(p);
        size_t i = 0;
        // four chains, so that the multiplications overlap
        uint64_t lane[4] = {h, h ^ 0x9ddfea08eb382d69ull, h ^ 0xc2b2ae3d27d4eb4full, h ^ 0x165667b19e3779f9ull};
        for (; i + 32 <= len; i += 32)
            for (int j = 0; j < 4; ++j) {
                uint64_t w;
                std::memcpy(&w, b + i + 8 * j, 8);
                lane[j] = (lane[j] ^ w) * 0xff51afd7ed558ccdull;
                lane[j] ^= lane[j] >> 32;
            }
        for (int j = 0; j < 4; ++j) h = (h ^ lane[j]) * 0x9fb21c651e98df25ull, h ^= h >> 32;
        for (; i + 8 <= len; i += 8) {
            uint64_t w;
            std::memcpy(&w, b + i, 8);
            h = (h ^ w) * 0xff51afd7ed558ccdull;
            h ^= h >> 32;
        }
        for (; i < len; ++i) h = (h ^ b[i]) * 0x100000001b3ull;
        h ^= uint64_t(len);
    };
    if (c->ops) mix(c->ops, sizeof(qs_op) * size_t(std::max(c->n_ops, 0)));
    if (c->mat_pool) mix(c->mat_pool, sizeof(double) * 2 * size_t(std::max<int64_t>(c->pool_len, 0)));
    return h;
}

// ---- circuit model cache
// A circuit's model (its ops, channel bounds and fast-path matrices) depends
// only on the circuit's bytes, so calls that run the same circuit again reuse
// it.  An entry keeps its own copy of the op records and the matrix pool (the
// model points into that copy, not into the caller's buffers) and is found by
// hash and then compared in full, so two circuits never share an entry.
// Each entry has a unique id; the plan and width caches are keyed by it.
struct ModelEntry {
    uint64_t id = 0;
    uint64_t hash = 0;
    size_t bytes = 0;  // estimate of the host memory held
    int n = 0;
    std::vector<qs_op> ops;
    std::vector<double> pool;
    CircuitModel model;
};

// Bounded by count and by an estimate of the host memory an entry holds
// (a batch of a few hundred distinct circuits must fit, or every call would
// rebuild every model and miss every plan keyed by it).
constexpr size_t kModelCacheEntries = 4096;
constexpr size_t kModelCacheBytes = size_t(512) << 20;
size_t g_model_bytes = 0;
std::mutex g_model_mu;
std::multimap<uint64_t, std::shared_ptr<const ModelEntry>> g_model_cache;
std::deque<std::shared_ptr<const ModelEntry>> g_model_fifo;
uint64_t g_model_next_id = 1;

bool same_circuit(const ModelEntry &e, const qs_circuit *c) {
    const size_t nops = size_t(c->n_ops), npool = size_t(c->pool_len) * 2;
    return e.n == c->n_qubits && e.ops.size() == nops && e.pool.size() == npool &&
           (nops == 0 || std::memcmp(e.ops.data(), c->ops, sizeof(qs_op) * nops) == 0) &&
           (npool == 0 || std::memcmp(e.pool.data(), c->mat_pool, sizeof(double) * npool) == 0);
}

// The model of circuit c, built (and validated) on its first use.
qs_status circuit_model(const qs_circuit *c, std::shared_ptr<const ModelEntry> *out) {
    if (!c || !c->ops || c->n_ops < 0 || !c->mat_pool || c->pool_len < 0)
        return fail(QS_ERR_INVALID_ARGUMENT, "bad circuit");
    const uint64_t h = circuit_hash(c);
    std::vector<std::shared_ptr<const ModelEntry>> alike;
    {
        std::lock_guard<std::mutex> lock(g_model_mu);
        auto range = g_model_cache.equal_range(h);
        for (auto it = range.first; it != range.second; ++it) alike.push_back(it->second);
    }
    for (auto &a : alike)  // compared outside the lock: a batch looks its circuits up on many threads
        if (same_circuit(*a, c)) {
            *out = std::move(a);
            return QS_OK;
        }
    auto e = std::make_shared<ModelEntry>();
    e->hash = h;
    e->n = c->n_qubits;
    e->ops.assign(c->ops, c->ops + c->n_ops);
    e->pool.assign(c->mat_pool, c->mat_pool + size_t(c->pool_len) * 2);
    qs_circuit own = *c;  // the model points into the entry's copies (an empty one holds no pointer)
    if (!e->ops.empty()) own.ops = e->ops.data();
    if (!e->pool.empty()) own.mat_pool = e->pool.data();
    QS_CHECK(build_model(&own, e->model));
    std::lock_guard<std::mutex> lock(g_model_mu);
    auto range = g_model_cache.equal_range(h);  // another thread may have built it meanwhile
    for (auto it = range.first; it != range.second; ++it)
        if (same_circuit(*it->second, c)) {
            *out = it->second;
            return QS_OK;
        }
    e->id = g_model_next_id++;
    e->bytes = sizeof(ModelEntry) + sizeof(qs_op) * e->ops.size() + sizeof(double) * e->pool.size() +
               (sizeof(qs::PlanOp) + 2 * sizeof(int) + sizeof(void *) + sizeof(double)) * e->model.ops.size();
    for (const ChannelInfo &ci : e->model.channels)
        e->bytes += sizeof(ChannelInfo) + sizeof(cd) * (ci.unit.size() + ci.excess_sorted.size()) +
                    (2 * sizeof(double) + 1) * ci.pbar.size();
    while (!g_model_fifo.empty() && (g_model_fifo.size() >= kModelCacheEntries ||
                                     g_model_bytes + e->bytes > kModelCacheBytes)) {
        const auto old = g_model_fifo.front();
        auto r = g_model_cache.equal_range(old->hash);
        for (auto it = r.first; it != r.second; ++it)
            if (it->second == old) {
                g_model_cache.erase(it);
                break;
            }
        g_model_bytes -= old->bytes;
        g_model_fifo.pop_front();
    }
    g_model_cache.emplace(h, e);
    g_model_fifo.push_back(e);
    g_model_bytes += e->bytes;
    *out = std::move(e);
    return QS_OK;
}

// ---- sweep grouping effort and the per-segment cache
// Every sweep saved is one read and one write of the state per trajectory, so
// the default plan's grouping is searched in proportion to the sweep work of
// the call (n_traj states of 2^n amplitudes; about 10 ms for 4096 restarts on
// a 24-qubit plan), and always hard from 26 qubits on, where one trajectory's
// sweeps take tens of milliseconds.  Blocks on disjoint qubits commute but
// round differently, so the grouping is part of the results: the count is a
// part of every key that a plan is kept under, and one of four, so that a
// circuit run with varying trajectory counts has at most four plans.  A
// trajectory whose channels need inner products regroups the blocks of each
// segment between such channels; those groupings are cached per segment.
int plan_restarts(int n, int64_t n_traj) {
    if (n >= 26) return 4096;
    const double w = std::ldexp(double(std::max<int64_t>(n_traj, 1)), n - 20);
    int restarts = 64;
    while (restarts < 4096 && restarts < w) restarts *= 4;
    return restarts;
}
// Below 24 qubits a sweep costs a few microseconds, about as much as a
// dozen restarts on a segment's blocks, and a segment with fewer than 16
// blocks (noisy circuits split into many) seldom groups better than the
// searched greedy grouping: it gets no restarts.
int segment_restarts(int n, size_t blocks) {
    if (n >= 24) return 64;
    if (blocks < 16) return 0;
    return n >= 20 ? 16 : 4;
}
constexpr uint64_t kGroupSeed = 0x243f6a8885a308d3ull;

struct SegKey {
    uint64_t model;  // model id
    int mode, f, tb, start, end;
    bool operator<(const SegKey &o) const {
        return std::tie(model, mode, f, tb, start, end) < std::tie(o.model, o.mode, o.f, o.tb, o.start, o.end);
    }
};
constexpr size_t kSegmentCacheEntries = 16384;
std::mutex g_seg_mu;
std::map<SegKey, std::vector<qs::Sweep>> g_seg_cache;
std::deque<SegKey> g_seg_fifo;

bool segment_lookup(const SegKey &k, std::vector<qs::Sweep> *out) {
    std::lock_guard<std::mutex> lock(g_seg_mu);
    auto it = g_seg_cache.find(k);
    if (it == g_seg_cache.end()) return false;
    *out = it->second;
    return true;
}

void segment_insert(const SegKey &k, const std::vector<qs::Sweep> &sw) {
    std::lock_guard<std::mutex> lock(g_seg_mu);
    if (g_seg_cache.count(k)) return;
    if (g_seg_fifo.size() >= kSegmentCacheEntries) {
        g_seg_cache.erase(g_seg_fifo.front());
        g_seg_fifo.pop_front();
    }
    g_seg_cache.emplace(k, sw);
    g_seg_fifo.push_back(k);
}

// A trajectory's program for the launches that run several side by side: the
// blocks in launch order, cut into sweeps (n > kBatchLdsQubits) and with a
// selection per inner-product channel.  Offsets are float2 in `mats`.
struct TrajPlan {
    struct Gate {
        int k = 0;
        int t[5] = {};                  // ascending index bits
        const float2 *dev = nullptr;    // default matrix, else `off`
        size_t off = 0;
        int sel = -1;                   // the matrix is this selection's outcome
        int before = -1;                // a selection made in front of this block
    };
    struct Cut {
        int pos[qs::kMaxTileBits] = {};
        int g0 = 0, g1 = 0;
        int sel = -1, rdm_q = -1;       // the selection after this sweep, and its qubit
    };
    struct Select {
        int channel = 0;
        double resid = 0.0;
        size_t cand = 0;                // nk x Db x Db complex128
        size_t dst = 0;                 // Db x Db float2 (sweeps)
        int Db = 0;
    };
    bool ok = false;                    // false: the one-by-one path runs it
    int sweeps = 0;                     // sweeps with gates, as the one-by-one path counts them
    std::vector<Gate> gates;
    std::vector<Cut> cuts;
    std::vector<Select> sels;
    std::vector<float2> mats;
};

// Side by side, trajectories of n > kBatchLdsQubits share sweep launches of up
// to this many 2^13-amplitude tiles (64 MiB of states; 512 workgroups are
// resident at once).  Calls of the noisy grid at 256 / 512 / 1024 / 2048 / 4096
// tiles: 20 trajectories of 15 qubits 0.77, 0.62, 0.62, 0.65, 0.66 ms; 64 of 17
// 1.93, 1.47, 1.27, 1.25, 1.28; 20 of 20 3.58, 2.56, 2.09, 1.92, 1.96; 20 of 21
// 4.43, 4.26, 3.61, 3.34, 3.23: beyond 1024 up to a tenth is left at 20 and 21
// qubits, for twice the memory a step.  From 22 qubits on one trajectory fills
// the GPU.
constexpr int kSideTiles = 1024;
constexpr int kSideMaxQubits = 21;
// Samples and Z records a call holds on the device at once.
constexpr int64_t kSampleRecords = int64_t(1) << 22;
constexpr int64_t kZRecords = 4096;

// Expected channels per trajectory that need inner products: for each
// channel that is not a mixture of unitaries, the chance that the draw lands
// past the sum of its bounds (Algorithm 2 resolves every other draw from the
// bounds alone).
double expected_slow_paths(const CircuitModel &m) {
    double e = 0.0;
    for (const ChannelInfo &c : m.channels) {
        if (c.mixture) continue;
        double sum = 0.0;
        for (double x : c.pbar) sum += x;
        e += std::max(0.0, 1.0 - sum);
    }
    return e;
}

// Whether the sweeps of a call of n_traj trajectories are replayed from a HIP
// graph where they can be.
constexpr int kGraphMaxQubits = 22;
bool graph_call(const CircuitModel &m, const qs_traj_params &p, int64_t n_traj) {
    return p.mode == QS_KRAUS_DELAYED && (p.flags & QS_TRAJ_GRAPH) && !(p.flags & QS_TRAJ_NO_GRAPH) &&
           m.n <= kGraphMaxQubits && n_traj >= 2;
}

// Whether n_traj trajectories may run side by side at the default tile width:
// the delayed scheme without kernel timing or graph replay, samples and Z
// records of one flush.  Up to 13 qubits that is all; from 14 qubits on at
// least two trajectories share sweeps, which take gates of at most four qubits
// and inner-product channels of one (what the sweep that forms a reduced
// density matrix takes).  The call alone decides, not what its state did
// before: where the two ways round differently its results would change.
bool side_call(const CircuitModel &m, const qs_traj_params &p, bool z_records, int64_t n_traj) {
    if (p.mode != QS_KRAUS_DELAYED || n_traj < 1 || (p.flags & QS_TRAJ_TIME_KERNELS) || graph_call(m, p, n_traj))
        return false;
    if (n_traj > 1 && p.n_samples > 0 && n_traj > kSampleRecords / p.n_samples) return false;
    if (z_records && n_traj > kZRecords) return false;
    if (m.n <= qs::kBatchLdsQubits) return true;
    if (m.n > kSideMaxQubits || n_traj < 2) return false;
    for (const ChannelInfo &c : m.channels)
        if (!c.mixture && c.k != 1) return false;
    for (const qs::PlanOp &o : m.ops)
        if (o.k > 4) return false;
    return true;
}

struct Runner {
    qs_state s;
    const CircuitModel &m;
    const qs_traj_params &p;
    qs_traj_result &res;
    const int max_fuse;
    const uint64_t chash;  // model id of the call's circuit (0: do not cache the plan)
    // trajectories of the whole call, of which a chunk of a concurrent call runs
    // a part: what decides how results round goes by these, so that they do
    // not depend on the number of states
    const int64_t call_traj;
    bool tuning = false;   // an autotuner trial: default plan only, no channel uploads
    bool one_by_one = false;  // an autotuner trial of trajectories that the call runs so
    // delayed mode: default plan, shared with the cache
    std::vector<const cd *> default_mats;
    std::vector<cd> tmp;
    const std::shared_ptr<const PlanEntry> plan;
    const std::vector<qs::Block> &blocks;
    const std::vector<int> &op_block;
    const std::vector<BlockDesc> &block_desc;
    // tile sweeps over the default plan: the sweep order is the launch order
    const std::vector<qs::Sweep> &sweeps;
    const std::vector<TileLayout> &layouts;
    struct Unit {
        const TileLayout *L;
        std::vector<const BlockDesc *> items;
        int rdm_q = -1;  // >= 0: the sweep also forms the reduced density matrix of this qubit
    };
    int rdm_records = 0;  // workgroup records the last such sweep wrote
    // one sweep of a segment: its layout and (block, op range) members in order
    struct SegSweep {
        const TileLayout *L;
        std::vector<std::array<int, 3>> members;  // block, first op index, end op index
    };
    std::deque<TileLayout> run_layouts;  // those of run_delayed's segments
    // naive mode: gate blocks per inter-channel segment
    std::vector<std::vector<BlockDesc>> naive_segments;
    std::vector<int> rest_ops;  // a slow block's operations after its channel
    std::deque<std::vector<cd>> slow_mats;
    qs::ReadoutDesc ro;
    double log_norm_bound = 0.0;
    double pending_scale = 1.0;     // conventional method: 1/sqrt(p_i N) not yet applied
    KernelTimer timer;
    bool timing = false;
    bool pending_reset = false;     // the state must become |0...0> before its next use
    float2 *static_mats = nullptr;  // default-plan matrices (the state's buffer), uploaded once per call
    // device-side branch selection (delayed mode): per-channel excess
    // matrices and bounds, the picks written by the select kernel, an error flag
    double *chan_buf = nullptr;
    std::vector<const double *> chan_excess, chan_pbar;
    int *dev_error = nullptr;       // error flag, followed by
    int *dev_choice = nullptr;      // [kChoiceCap] picks
    bool selecting = false;         // a selection has been launched
    int *host_choice = nullptr;     // pinned mirror
    double *sel_rdm = nullptr;      // R of the pending channel; a renormalisation
                                    // launched before the select cannot overwrite it
    static constexpr int kChoiceCap = 1 << 16;
    std::vector<std::pair<int64_t, int>> choice_owner;  // (trajectory rel, channel) per slot
    // the pending inner-product channel whose pick decides the next block
    struct PendingSelect {
        bool active = false;
        bool staged = false;
        bool launched = false;
        int op = -1, channel = -1;
        double resid = 0.0;
        qs::SelectArgs args;
    } sel;

    // HIP graph of the default plan's sweeps (delayed mode, small states):
    // each block reads its matrix from a fixed device slot, so one capture
    // serves every trajectory whose channels are all picked from the bounds
    bool graph_wanted = false;
    bool graph_failed = false;
    hipStream_t capture_st = nullptr;      // private non-blocking stream the graph is captured on
    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    int graph_launches = 0;
    int64_t graph_k[6] = {};
    float2 *gtab_dev = nullptr;            // the slots
    std::vector<size_t> gtab_off;          // per block: float2 offset, or kNoSlot (identity)
    std::vector<float2> gtab_host;         // the slots' current contents
    static constexpr int kStages = 4;  // pinned staging copies in flight
    float2 *gtab_stage[kStages] = {};
    hipEvent_t gtab_ev[kStages] = {};
    bool gtab_live[kStages] = {};
    int gtab_half = 0;
    std::vector<char> gdirty_prev;         // blocks the previous replay patched
    static constexpr size_t kNoSlot = ~size_t(0);

    ~Runner() {
        if (gtab_dev) (void)hipStreamSynchronize(s->st);
        if (graph_exec) (void)hipGraphExecDestroy(graph_exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (capture_st) (void)hipStreamDestroy(capture_st);
        if (gtab_dev) (void)hipFree(gtab_dev);
        for (int h = 0; h < kStages; ++h) {
            if (gtab_stage[h]) (void)hipHostFree(gtab_stage[h]);
            if (gtab_ev[h]) (void)hipEventDestroy(gtab_ev[h]);
        }

    }

    // Channels that can need inner products: upload K^dag K - pbar I (ascending
    // target order, complex128) and the bounds once per call.
    qs_status upload_channels() {
        const size_t nch = m.channels.size();
        chan_excess.assign(nch, nullptr);
        chan_pbar.assign(nch, nullptr);
        size_t total = 0;
        for (const auto &c : m.channels)
            if (!c.mixture) total += c.excess_sorted.size() * 2 + c.pbar.size();
        if (total == 0) return QS_OK;  // no channel can need inner products
        if (!s->sel_choice_dev) {
            QS_HIP(s, hipMalloc(&s->sel_choice_dev, sizeof(int) * (kChoiceCap + 1)));
            QS_HIP(s, hipMalloc(&s->sel_rdm, sizeof(double) * qs::kMaxReduceWidth));
            QS_HIP(s, hipHostMalloc(&s->sel_choice_host, sizeof(int) * (kChoiceCap + 1),
                                    hipHostMallocDefault));
        }
        dev_error = s->sel_choice_dev;
        dev_choice = s->sel_choice_dev + 1;
        host_choice = s->sel_choice_host;
        sel_rdm = s->sel_rdm;
        // a cached model's channels are fixed by its id and the mode: the
        // state keeps their tables from one call to the next
        const uint64_t tag = chash ? (chash << 2) | uint64_t(p.mode & 3) : 0;
        const bool have = tag != 0 && tag == s->chan_tag && total <= s->chan_cap;
        std::vector<double> host(have ? 0 : total);
        std::vector<size_t> at(nch, 0);
        size_t pos = 0;
        for (size_t c = 0; c < nch; ++c) {
            const auto &ci = m.channels[c];
            if (ci.mixture) continue;
            at[c] = pos;
            if (have) {
                pos += 2 * ci.excess_sorted.size() + ci.pbar.size();
                continue;
            }
            for (const cd &z : ci.excess_sorted) {
                host[pos++] = z.real();
                host[pos++] = z.imag();
            }
            for (double pb : ci.pbar) host[pos++] = pb;
        }
        if (!have) {
            s->chan_tag = 0;
            if (total > s->chan_cap) {
                if (s->chan_dev) QS_HIP(s, hipFree(s->chan_dev));
                s->chan_dev = nullptr;
                s->chan_cap = 0;
                QS_HIP(s, hipMalloc(&s->chan_dev, sizeof(double) * total));
                s->chan_cap = total;
            }
            QS_HIP(s, hipMemcpyAsync(s->chan_dev, host.data(), sizeof(double) * total, hipMemcpyHostToDevice,
                                     s->st));
            QS_HIP(s, hipStreamSynchronize(s->st));  // `host` is pageable and ends with this call
            s->chan_tag = tag;
        }
        chan_buf = s->chan_dev;
        for (size_t c = 0; c < nch; ++c) {
            const auto &ci = m.channels[c];
            if (ci.mixture) continue;
            chan_excess[c] = chan_buf + at[c];
            chan_pbar[c] = chan_buf + at[c] + ci.excess_sorted.size() * 2;
        }
        return QS_OK;
    }

    // Clears the error flag before the call's first selection.
    qs_status open_selections() {
        if (selecting) return QS_OK;
        selecting = true;
        QS_HIP(s, hipMemsetAsync(dev_error, 0, sizeof(int), s->st));
        return QS_OK;
    }

    // Copy the error flag and the picks made on the device back.
    qs_status drain_choices() {
        if (!selecting) return QS_OK;
        QS_HIP(s, hipMemcpyAsync(host_choice, dev_error, sizeof(int) * (1 + choice_owner.size()),
                                 hipMemcpyDeviceToHost, s->st));
        QS_HIP(s, hipStreamSynchronize(s->st));
        const int nch = int(m.channels.size());
        if (res.kraus_choices)
            for (size_t i = 0; i < choice_owner.size(); ++i)
                res.kraus_choices[choice_owner[i].first * nch + choice_owner[i].second] =
                    int8_t(host_choice[1 + i]);
        choice_owner.clear();
        if (host_choice[0] != 0)
            return fail(QS_ERR_ZERO_NORM, "a channel needing inner products met a zero norm or weight");
        return QS_OK;
    }

    // Uploads `host` to the state's static buffer, which then holds the
    // matrices of the cached plan `tag` (0: of none).
    qs_status upload_static(const std::vector<float2> &host, uint64_t tag) {
        const size_t total = host.size();
        s->static_tag = 0;
        if (total > s->static_cap) {
            QS_HIP(s, hipStreamSynchronize(s->st));  // an earlier call's kernels may still read it
            if (s->static_buf) QS_HIP(s, hipFree(s->static_buf));
            s->static_buf = nullptr;
            s->static_cap = 0;
            QS_HIP(s, hipMalloc(&s->static_buf, sizeof(float2) * total));
            s->static_cap = total;
        }
        static_mats = s->static_buf;
        QS_HIP(s, hipMemcpyAsync(static_mats, host.data(), sizeof(float2) * total, hipMemcpyHostToDevice,
                                 s->st));
        QS_HIP(s, hipStreamSynchronize(s->st));  // `host` is pageable and ends with this call
        s->static_tag = tag;
        return QS_OK;
    }
    int64_t sample_fill = 0;        // samples buffered on the device
    int64_t sample_first_traj = 0;  // trajectory index (relative) of the first buffered sample
    int64_t z_fill = 0;             // Z-weight records buffered on the device
    int64_t z_first_traj = 0;
    std::vector<double> z_host;

    Runner(qs_state s_, const CircuitModel &m_, const qs_traj_params &p_, qs_traj_result &r_, uint64_t chash_,
           int64_t call_traj_, hipEvent_t ref = nullptr, std::vector<std::pair<double, double>> *intervals = nullptr)
        : s(s_), m(m_), p(p_), res(r_), max_fuse(p_.max_fuse > 0 ? p_.max_fuse : kDefaultFuse), chash(chash_),
          call_traj(call_traj_), plan(default_plan()), blocks(plan->blocks), op_block(plan->op_block), block_desc(plan->block_desc),
          sweeps(plan->sweeps), layouts(plan->layouts) {
        timer.ref = ref;
        timer.intervals = intervals;
    }

    int plan_tile_bits() const { return p.tile_bits == 0 ? qs::kDefaultTileBits : p.tile_bits; }

    // The call's default plan, from the cache or made now (delayed modes;
    // also fills default_mats).
    std::shared_ptr<const PlanEntry> default_plan() {
        if (p.mode == QS_KRAUS_NAIVE) return std::make_shared<PlanEntry>();
        const int n_ops = int(m.ops.size());
        default_mats.assign(n_ops, nullptr);
        for (int o = 0; o < n_ops; ++o) {
            if (m.kind[o] == QS_OP_GATE) {
                default_mats[o] = m.gate_mat[o];
            } else {
                const ChannelInfo &c = m.channels[m.channel_of_op[o]];
                default_mats[o] = fast_pick_matrix(c, c.default_pick);
            }
        }
        const int restarts = plan_restarts(m.n, call_traj);
        const PlanKey key{chash, m.n, p.mode, max_fuse, plan_tile_bits(), restarts};
        std::shared_ptr<const PlanEntry> cached;
        if (chash) plan_lookup(key, &cached);
        if (cached) return cached;
        auto e = std::make_shared<PlanEntry>();
        e->blocks = qs::fuse_greedy(m.n, m.ops, max_fuse, &e->op_block);
        e->block_desc.resize(e->blocks.size());
        for (size_t b = 0; b < e->blocks.size(); ++b) {
            BlockDesc &d = e->block_desc[b];
            build_block(m, e->blocks[b].ops, default_mats, tmp, d);
            for (int o : e->blocks[b].ops) {
                const int c = m.channel_of_op[o];
                d.log_bound += c < 0 ? m.gate_log_bound[o] : m.channels[c].log_pbar[m.channels[c].default_pick];
            }
            if (d.identity) continue;
            d.static_off = e->static_len;
            e->static_len += size_t(1) << (2 * d.g.k);
        }
        const int T = plan_tile_bits();
        if (T >= 10 && m.n >= qs::kTileMinQubits) {
            e->sweeps = qs::group_sweeps_best(m.n, e->blocks, std::min(T, m.n), qs::kTileLowBits, qs::kMaxTileGates,
                                              qs::tile_mat_budget(std::min(T, m.n)), tile_slots(),
                                              restarts, kGroupSeed);
        } else {
            for (size_t b = 0; b < e->blocks.size(); ++b) {
                qs::Sweep sw;
                sw.blocks.push_back(int(b));
                e->sweeps.push_back(std::move(sw));
            }
        }
        e->layouts.resize(e->sweeps.size());
        for (size_t u = 0; u < e->sweeps.size(); ++u) e->layouts[u] = TileLayout::of(m.n, e->sweeps[u], e->blocks);
        if (chash) plan_insert(key, e);
        return e;
    }

    // Device copies of the plan's matrices and the channels' tables.
    qs_status plan_delayed() {
        if (!tuning) QS_CHECK(upload_channels());
        // a plan from the cache is fixed by its key: the state keeps its
        // matrices from one call to the next (they do not depend on how the
        // blocks are grouped)
        const uint64_t tag = chash ? (chash << 16) | (uint64_t(p.mode & 3) << 12) |
                                         (uint64_t(max_fuse) << 8) | uint64_t(plan_tile_bits())
                                   : 0;
        if (plan->static_len == 0 || (tag != 0 && tag == s->static_tag && plan->static_len <= s->static_cap)) {
            static_mats = s->static_buf;
            return QS_OK;
        }
        std::vector<float2> host(plan->static_len);
        for (const BlockDesc &d : block_desc)
            if (!d.identity) std::memcpy(host.data() + d.static_off, d.g.m, sizeof(float2) << (2 * d.g.k));
        return upload_static(host, tag);
    }

    const float2 *mat_of(const BlockDesc &d) const { return d.dev ? d.dev : static_mats + d.static_off; }

    // The default plan once from |0...0> (every channel at its most likely
    // pick, no inner products): the autotuner's trial.
    qs_status run_default_plan() {
        QS_CHECK(restore_home(s));
        pending_reset = true;
        log_norm_bound = 0.0;
        std::vector<SegSweep> seg;
        segment_sweeps(0, int(m.ops.size()), true, run_layouts, seg);
        std::vector<Unit> units;
        for (const SegSweep &ss : seg) {
            Unit u{ss.L, {}};
            for (const auto &mem : ss.members)
                if (!block_desc[mem[0]].identity) u.items.push_back(&block_desc[mem[0]]);
            if (!u.items.empty()) units.push_back(std::move(u));
        }
        QS_CHECK(flush_units(units));
        return settle_reset();
    }

    // The sweeps of the segment [seg_start, seg_end): the call's plan when the
    // trajectory has no channel needing inner products; otherwise the blocks
    // restricted to the segment, regrouped into sweeps of their own (reusing
    // the whole-circuit sweeps would launch every sweep that straddles the
    // split twice: ~6 extra sweeps per split on a 24-qubit grid).
    void segment_sweeps(int seg_start, int seg_end, bool whole_plan, std::deque<TileLayout> &seg_layouts,
                        std::vector<SegSweep> &out) const {
        out.clear();
        if (whole_plan) {
            for (size_t u = 0; u < sweeps.size(); ++u) {
                SegSweep ss{&layouts[u], {}};
                for (int b : sweeps[u].blocks)
                    ss.members.push_back({b, 0, int(blocks[b].ops.size())});
                out.push_back(std::move(ss));
            }
            return;
        }
        std::vector<qs::Block> rb;
        std::vector<std::array<int, 3>> orig;
        for (size_t b = 0; b < blocks.size(); ++b) {
            const auto &ops = blocks[b].ops;
            const int lo = int(std::lower_bound(ops.begin(), ops.end(), seg_start) - ops.begin());
            const int hi = int(std::lower_bound(ops.begin() + lo, ops.end(), seg_end) - ops.begin());
            if (lo == hi) continue;
            qs::Block r;
            r.ops.assign(ops.begin() + lo, ops.begin() + hi);
            r.k = qs::union_qubits(r.ops, m.ops, r.q);
            rb.push_back(std::move(r));
            orig.push_back({int(b), lo, hi});
        }
        const int T = p.tile_bits == 0 ? qs::kDefaultTileBits : p.tile_bits;
        std::vector<qs::Sweep> sw;
        const SegKey skey{chash, p.mode, max_fuse, T, seg_start, seg_end};
        if (chash && segment_lookup(skey, &sw)) {
        } else if (T >= 10 && m.n >= qs::kTileMinQubits) {
            sw = qs::group_sweeps_best(m.n, rb, std::min(T, m.n), qs::kTileLowBits, qs::kMaxTileGates,
                                       qs::tile_mat_budget(std::min(T, m.n)), tile_slots(),
                                       segment_restarts(m.n, rb.size()), kGroupSeed);
            if (chash) segment_insert(skey, sw);
        } else {
            for (size_t b = 0; b < rb.size(); ++b) {
                qs::Sweep one;
                one.blocks.push_back(int(b));
                sw.push_back(std::move(one));
            }
        }
        // the last sweep before a one-qubit channel that needs inner products
        // holds that qubit, so that it can form the channel's reduced density
        // matrix on the way (a tile's qubits are its blocks' plus fill)
        const int rq = rdm_qubit(seg_end);
        for (size_t u = 0; u < sw.size(); ++u) {
            const qs::Sweep &w = sw[u];
            if (u + 1 == sw.size() && rq >= 0 && !w.bits.empty() &&  // a tile sweep
                std::find(w.bits.begin(), w.bits.end(), rq) == w.bits.end() &&
                int(w.bits.size()) < qs::kMaxTileBits) {
                qs::Sweep w2 = w;
                w2.bits.insert(std::upper_bound(w2.bits.begin(), w2.bits.end(), rq), rq);
                seg_layouts.push_back(TileLayout::of(m.n, w2, rb));
            } else {
                seg_layouts.push_back(TileLayout::of(m.n, w, rb));
            }
            SegSweep ss{&seg_layouts.back(), {}};
            for (int b : w.blocks) ss.members.push_back(orig[b]);
            out.push_back(std::move(ss));
        }
    }

    // The qubit of a one-qubit channel at op index `op` (a segment end), or -1.
    int rdm_qubit(int op) const {
        if (op >= int(m.ops.size()) || m.kind[op] != QS_OP_CHANNEL) return -1;
        const ChannelInfo &ci = m.channels[m.channel_of_op[op]];
        return ci.k == 1 ? ci.t[0] : -1;
    }

    // Launch the deferred reset, if any (before anything reads the state).
    qs_status settle_reset() {
        if (!pending_reset) return QS_OK;
        pending_reset = false;
        if (timing) QS_CHECK(timer.close(s));
        QS_HIP(s, qs::launch_set_basis(s->amp, s->n, 0, s->st));
        return QS_OK;
    }

    // Copy staged matrices, run a pending branch selection (it writes the
    // matrix one of the units reads), then launch the units in order.
    qs_status flush_units(std::vector<Unit> &units) {
        QS_CHECK(arena_commit(s));
        if (sel.active && sel.staged && !sel.launched) {
            QS_HIP(s, qs::launch_select(sel.args, s->st));
            sel.launched = true;
        }
        for (const Unit &x : units) QS_CHECK(launch_unit(x));
        if (timing) QS_CHECK(timer.close(s));
        units.clear();
        return QS_OK;
    }

    qs_status launch_unit(const Unit &u) {
        const TileLayout &L = *u.L;
        if (!L.tiled) {
            QS_CHECK(settle_reset());
            for (const BlockDesc *d : u.items) QS_CHECK(launch_block(*d));
            return QS_OK;
        }
        qs::TileArgs a;
        std::memset(&a, 0, sizeof(a));
        a.init_zero = pending_reset ? 1 : 0;
        if (pending_reset) res.zero_start_sweeps++;
        pending_reset = false;
        a.tb = L.tb;
        for (int i = 0; i < L.tb; ++i) a.pos[i] = L.pos[i];
        int lofs = 0;
        double lb = 0.0;
        for (const BlockDesc *d : u.items) {
            qs::TileGate &g = a.g[a.n_gates++];
            g.k = d->g.k;
            for (int b = 0; b < d->g.k; ++b) g.lt[b] = L.local[d->g.t[b]];
            g.lofs = lofs;
            g.mat = mat_of(*d);
            lofs += qs::tile_mat_slots(d->g.k);
            lb += d->log_bound;
            res.gate_k_launches[d->g.k]++;
        }
        a.mat_total = lofs;
        if (u.rdm_q >= 0) {
            a.rdm_lt = L.local[u.rdm_q];
            a.rdm_out = s->red_partials + kRdmRecordOffset;
            // a renormalisation this sweep would call for happens before it:
            // the channel's selection scales the next block by the norm of the
            // state the matrix is formed on
            if (!a.init_zero && log_norm_bound + lb < kRenormLogThreshold) {
                if (timing) QS_CHECK(timer.close(s));
                QS_CHECK(renormalize_now(s));
                res.sweeps += 2;
                log_norm_bound = 0.0;
            }
        }
        if (timing) QS_CHECK(timer.open(s));
        QS_HIP(s, qs::launch_apply_tile(s->amp, s->n, a, s->st, u.rdm_q >= 0 ? &rdm_records : nullptr));
        if (timing) timer.launched();
        res.sweeps++;
        res.gate_sweeps++;
        log_norm_bound += lb;
        if (log_norm_bound < kRenormLogThreshold) {
            if (timing) QS_CHECK(timer.close(s));
            QS_CHECK(renormalize_now(s));
            res.sweeps += 2;
            log_norm_bound = 0.0;
        }
        return QS_OK;
    }

    qs_status plan_naive() {
        // gates between consecutive channels, fused per segment
        std::vector<int> seg;
        std::vector<const cd *> mats(m.ops.size(), nullptr);
        for (size_t o = 0; o < m.ops.size(); ++o) mats[o] = m.gate_mat[o];
        auto close = [&]() {
            std::vector<BlockDesc> out;
            if (!seg.empty()) {
                std::vector<qs::PlanOp> sub(seg.size());
                std::vector<const cd *> submats(seg.size());
                for (size_t i = 0; i < seg.size(); ++i) {
                    sub[i] = m.ops[seg[i]];
                    submats[i] = mats[seg[i]];
                }
                const auto bl = qs::fuse_greedy(m.n, sub, max_fuse);
                for (const auto &b : bl) {
                    BlockDesc d;
                    int q[5];
                    const int k = qs::union_qubits(b.ops, sub, q);
                    tmp.resize(size_t(1) << (2 * k));
                    qs::fused_matrix(k, q, b.ops, sub, submats, tmp.data());
                    d.g.k = k;
                    for (int j = 0; j < 5; ++j) d.g.t[j] = j < k ? q[j] : 0;
                    const int D = 1 << k;
                    for (int i = 0; i < D * D; ++i)
                        d.g.m[i] = make_float2(float(tmp[i].real()), float(tmp[i].imag()));
                    cd c;
                    d.identity = qs::is_identity_multiple(D, tmp.data(), 1e-15, &c) && std::abs(c - cd(1.0)) < 1e-15;
                    for (int o : b.ops) d.log_bound += m.gate_log_bound[seg[o]];
                    out.push_back(d);
                }
            }
            naive_segments.push_back(std::move(out));
            seg.clear();
        };
        for (size_t o = 0; o < m.ops.size(); ++o) {
            if (m.kind[o] == QS_OP_GATE) seg.push_back(int(o));
            else close();
        }
        close();  // the tail after the last channel
        std::vector<float2> host;
        for (auto &segv : naive_segments)
            for (auto &d : segv) {
                if (d.identity) continue;
                d.static_off = host.size();
                host.insert(host.end(), d.g.m, d.g.m + (size_t(1) << (2 * d.g.k)));
            }
        return host.empty() ? QS_OK : upload_static(host, 0);
    }

    qs_status launch_block(const BlockDesc &d) {
        if (pending_scale != 1.0) {
            BlockDesc sc = d;
            const int D = 1 << d.g.k;
            const float f = float(pending_scale);
            for (int i = 0; i < D * D; ++i) sc.g.m[i] = make_float2(sc.g.m[i].x * f, sc.g.m[i].y * f);
            sc.identity = false;
            pending_scale = 1.0;
            QS_CHECK(stage_block(s, sc));
            QS_CHECK(arena_commit(s));
            return launch_block(sc);
        }
        if (d.identity) return QS_OK;
        if (timing) QS_CHECK(timer.open(s));
        QS_HIP(s, qs::launch_apply_gate(s->amp, s->n, d.g, mat_of(d), s->st));
        if (timing) {
            timer.launched();
            QS_CHECK(timer.close(s));
        }
        res.sweeps++;
        res.gate_sweeps++;
        res.gate_k_launches[d.g.k]++;
        log_norm_bound += d.log_bound;
        if (log_norm_bound < kRenormLogThreshold) {
            QS_CHECK(renormalize_now(s));
            res.sweeps += 2;
            log_norm_bound = 0.0;
        }
        return QS_OK;
    }

    qs_status flush_samples() {
        if (sample_fill == 0) return QS_OK;
        QS_HIP(s, hipStreamSynchronize(s->st));
        if (res.bitstrings)
            QS_HIP(s, hipMemcpy(res.bitstrings + sample_first_traj * p.n_samples, s->samp_out,
                                sizeof(uint64_t) * sample_fill, hipMemcpyDeviceToHost));
        sample_fill = 0;
        return QS_OK;
    }

    qs_status sample_trajectory(int64_t rel, uint32_t traj) {
        if (p.n_samples <= 0) return QS_OK;
        if (sample_fill + p.n_samples > int64_t(s->samp_cap)) QS_CHECK(flush_samples());
        if (sample_fill == 0) sample_first_traj = rel;
        QS_HIP(s, qs::launch_sample(s->amp, s->n, s->samp_sums, s->samp_incl, p.seed, traj,
                                    p.circuit_id, p.n_samples, ro, s->samp_out + sample_fill,
                                    s->samp_norm, s->st));
        res.sweeps += 1;
        sample_fill += p.n_samples;
        return QS_OK;
    }

    // <Z_q> of the trajectory's final state: one read pass into a device
    // record, copied back in batches (no synchronisation per trajectory)
    qs_status flush_z() {
        if (z_fill == 0) return QS_OK;
        z_host.resize(size_t(z_fill) * qs::kZRecord);
        QS_HIP(s, hipMemcpyAsync(z_host.data(), s->z_dev, sizeof(double) * z_host.size(),
                                 hipMemcpyDeviceToHost, s->st));
        QS_HIP(s, hipStreamSynchronize(s->st));
        for (int64_t i = 0; i < z_fill; ++i)
            QS_CHECK(z_from_record(s->n, z_host.data() + size_t(i) * qs::kZRecord,
                                   res.z_expect + (z_first_traj + i) * s->n));
        z_fill = 0;
        return QS_OK;
    }

    qs_status z_trajectory(int64_t rel) {
        if (!res.z_expect) return QS_OK;
        if (z_fill == int64_t(s->z_cap)) QS_CHECK(flush_z());
        if (z_fill == 0) z_first_traj = rel;
        QS_HIP(s, qs::launch_zweights(s->amp, s->n, s->red_partials,
                                      s->z_dev + size_t(z_fill) * qs::kZRecord, s->st));
        res.sweeps += 1;
        z_fill += 1;
        return QS_OK;
    }

    // Tile arguments of one unit of default-plan blocks, each matrix read
    // from the block's graph slot.
    void unit_args(const Unit &u, bool init_zero, qs::TileArgs &a) const {
        const TileLayout &L = *u.L;
        std::memset(&a, 0, sizeof(a));
        a.init_zero = init_zero ? 1 : 0;
        a.tb = L.tb;
        for (int i = 0; i < L.tb; ++i) a.pos[i] = L.pos[i];
        int lofs = 0;
        for (const BlockDesc *d : u.items) {
            qs::TileGate &g = a.g[a.n_gates++];
            g.k = d->g.k;
            for (int b = 0; b < d->g.k; ++b) g.lt[b] = L.local[d->g.t[b]];
            g.lofs = lofs;
            g.mat = gtab_dev + gtab_off[size_t(d - block_desc.data())];
            lofs += qs::tile_mat_slots(d->g.k);
        }
        a.mat_total = lofs;
    }

    // Capture the default plan's sweeps into a graph (once per call).  Any
    // failure leaves graph_failed set and the trajectories run directly.
    qs_status build_graph() {
        graph_failed = true;
        if (!s->st) return QS_OK;  // replays on the null stream are left out
        std::vector<SegSweep> seg;
        segment_sweeps(0, int(m.ops.size()), true, run_layouts, seg);
        std::vector<Unit> units;
        for (const SegSweep &ss : seg) {
            if (!ss.L->tiled) return QS_OK;  // only tile sweeps are captured
            Unit u{ss.L, {}};
            for (const auto &mem : ss.members)
                if (!block_desc[mem[0]].identity) u.items.push_back(&block_desc[mem[0]]);
            if (!u.items.empty()) units.push_back(std::move(u));
        }
        if (units.empty()) return QS_OK;
        gtab_off.assign(blocks.size(), kNoSlot);
        size_t total = 0;
        for (size_t b = 0; b < blocks.size(); ++b) {
            if (block_desc[b].identity) continue;
            gtab_off[b] = total;
            total += ((size_t(1) << (2 * block_desc[b].g.k)) + 31) & ~size_t(31);  // 256 B slots
        }
        gtab_host.assign(total, make_float2(0.f, 0.f));
        for (size_t b = 0; b < blocks.size(); ++b)
            if (gtab_off[b] != kNoSlot)
                std::memcpy(gtab_host.data() + gtab_off[b], block_desc[b].g.m,
                            sizeof(float2) << (2 * block_desc[b].g.k));
        QS_HIP(s, hipMalloc(&gtab_dev, sizeof(float2) * total));
        QS_HIP(s, hipMemcpyAsync(gtab_dev, gtab_host.data(), sizeof(float2) * total,
                                 hipMemcpyHostToDevice, s->st));
        QS_HIP(s, hipStreamSynchronize(s->st));
        for (int h = 0; h < kStages; ++h) {
            QS_HIP(s, hipHostMalloc(&gtab_stage[h], sizeof(float2) * total, hipHostMallocDefault));
            QS_HIP(s, hipEventCreateWithFlags(&gtab_ev[h], hipEventDisableTiming));
        }
        gdirty_prev.assign(blocks.size(), 0);
        std::vector<qs::TileArgs> args(units.size());
        for (size_t u = 0; u < units.size(); ++u) {
            unit_args(units[u], u == 0, args[u]);
            if (qs::prepare_apply_tile(s->n, args[u]) != hipSuccess) return QS_OK;
        }
        QS_CHECK(restore_home(s));
        // Captured on a private non-blocking stream, not the state's: capture
        // runs nothing, and a caller's stream may be a blocking one, whose
        // capture would make a synchronous copy on another thread (another
        // state of a concurrent call) fail for depending on it.  The graph is
        // replayed on the state's stream.
        if (hipStreamCreateWithFlags(&capture_st, hipStreamNonBlocking) != hipSuccess) {
            capture_st = nullptr;
            (void)hipGetLastError();
            return QS_OK;
        }
        if (hipStreamBeginCapture(capture_st, hipStreamCaptureModeThreadLocal) != hipSuccess) {
            (void)hipGetLastError();
            return QS_OK;
        }
        hipError_t e = hipSuccess;
        for (const auto &a : args)
            if ((e = qs::launch_apply_tile(s->amp, s->n, a, capture_st)) != hipSuccess) break;
        hipGraph_t g = nullptr;
        const hipError_t e_end = hipStreamEndCapture(capture_st, &g);
        if (e != hipSuccess || e_end != hipSuccess || !g) {
            if (g) (void)hipGraphDestroy(g);
            (void)hipGetLastError();
            return QS_OK;
        }
        graph = g;
        if (hipGraphInstantiate(&graph_exec, graph, nullptr, nullptr, 0) != hipSuccess) {
            graph_exec = nullptr;
            (void)hipGetLastError();
            return QS_OK;
        }
        graph_launches = int(units.size());
        for (const Unit &u : units)
            for (const BlockDesc *d : u.items) graph_k[d->g.k]++;
        graph_failed = false;
        return QS_OK;
    }

    // One trajectory by graph replay, when its channels were all picked from
    // the bounds (`mats`: its per-op matrices, `dirty`: blocks whose picks
    // differ from the default).  Returns false (nothing enqueued) when the
    // trajectory cannot use the graph: a patched block that the default plan
    // drops as the identity, or a norm bound that would need renormalising
    // on the way.
    qs_status try_graph(const std::vector<const cd *> &mats, const std::vector<char> &dirty,
                        const std::vector<int> &pick, bool *used) {
        *used = false;
        if (!graph_exec) {
            if (graph_failed) return QS_OK;
            QS_CHECK(build_graph());
            if (graph_failed) return QS_OK;
        }
        // the eager path renormalises when the running bound of the norm
        // (a sum of non-positive logs) falls below the threshold; the graph
        // carries no renormalisation, so such trajectories run directly
        double lb_total = 0.0;
        std::vector<std::pair<size_t, BlockDesc>> patched;
        for (size_t b = 0; b < blocks.size(); ++b) {
            if (!dirty[b]) {
                lb_total += block_desc[b].log_bound;
                continue;
            }
            if (gtab_off[b] == kNoSlot) return QS_OK;
            BlockDesc bd;
            build_block(m, blocks[b].ops, mats, tmp, bd);
            double lb = 0.0;
            for (int o : blocks[b].ops) {
                if (m.kind[o] == QS_OP_GATE) lb += m.gate_log_bound[o];
                else lb += m.channels[m.channel_of_op[o]].log_pbar[pick[m.channel_of_op[o]]];
            }
            lb_total += lb;
            if (bd.g.k != block_desc[b].g.k) return QS_OK;  // same qubits, so never
            patched.emplace_back(b, bd);
        }
        if (lb_total < kRenormLogThreshold) return QS_OK;
        // slots to rewrite: this trajectory's patches and the previous one's
        size_t lo = kNoSlot, hi = 0;
        auto touch = [&](size_t b) {
            const size_t len = size_t(1) << (2 * block_desc[b].g.k);
            lo = std::min(lo, gtab_off[b]);
            hi = std::max(hi, gtab_off[b] + len);
        };
        for (size_t b = 0; b < blocks.size(); ++b)
            if (gdirty_prev[b] && !dirty[b]) {
                std::memcpy(gtab_host.data() + gtab_off[b], block_desc[b].g.m,
                            sizeof(float2) << (2 * block_desc[b].g.k));
                touch(b);
            }
        for (const auto &pb : patched) {
            std::memcpy(gtab_host.data() + gtab_off[pb.first], pb.second.g.m,
                        sizeof(float2) << (2 * pb.second.g.k));
            touch(pb.first);
        }
        QS_CHECK(restore_home(s));
        QS_CHECK(settle_reset());
        if (lo != kNoSlot) {
            const int h = gtab_half;
            if (gtab_live[h]) QS_HIP(s, hipEventSynchronize(gtab_ev[h]));
            std::memcpy(gtab_stage[h] + lo, gtab_host.data() + lo, sizeof(float2) * (hi - lo));
            QS_HIP(s, hipMemcpyAsync(gtab_dev + lo, gtab_stage[h] + lo, sizeof(float2) * (hi - lo),
                                     hipMemcpyHostToDevice, s->st));
            QS_HIP(s, hipEventRecord(gtab_ev[h], s->st));
            gtab_live[h] = true;
            gtab_half = (gtab_half + 1) % kStages;
        }
        if (timing) QS_CHECK(timer.open(s));
        QS_HIP(s, hipGraphLaunch(graph_exec, s->st));
        if (timing) {
            timer.launched_n(graph_launches);
            QS_CHECK(timer.close(s));
        }
        res.sweeps += graph_launches;
        res.gate_sweeps += graph_launches;
        res.zero_start_sweeps += 1;
        for (int k = 1; k <= 5; ++k) res.gate_k_launches[k] += graph_k[k];
        gdirty_prev = dirty;
        pending_reset = false;
        log_norm_bound = 0.0;
        res.graph_replays++;
        *used = true;
        return QS_OK;
    }

    // Candidate i = (the block's later operations, fused once) x K_i on the
    // channel's qubits: the block begins with the channel, so each candidate
    // costs 2 Db^2 Dc multiply-adds instead of a fusion of its own.
    void fill_candidates(const ChannelInfo &ci, int kb, const int *q, const std::vector<int> &later,
                         const std::vector<const cd *> &mats, std::vector<cd> &work, double *out) const {
        const int Dc = 1 << ci.k, Db = 1 << kb;
        work.resize(size_t(Db) * Db);  // fused_matrix writes Db x Db entries
        qs::fused_matrix(kb, q, later, m.ops, mats, work.data());
        int cpos[2] = {0, 0};
        int cmask = 0;
        for (int j = 0; j < ci.k; ++j) {
            cpos[j] = int(std::find(q, q + kb, ci.t[j]) - q);
            cmask |= 1 << cpos[j];
        }
        auto spread = [&](int jx) {
            int x = 0;
            for (int j = 0; j < ci.k; ++j)
                if ((jx >> j) & 1) x |= 1 << cpos[j];
            return x;
        };
        for (int i = 0; i < ci.nk; ++i) {
            const cd *K = ci.kraus + size_t(i) * Dc * Dc;
            double *o = out + 2 * size_t(i) * Db * Db;
            for (int c = 0; c < Db; ++c) {
                int jc = 0;
                for (int j = 0; j < ci.k; ++j) jc |= ((c >> cpos[j]) & 1) << j;
                const int base = c & ~cmask;
                for (int r = 0; r < Db; ++r) {
                    cd acc = 0.0;
                    for (int jx = 0; jx < Dc; ++jx)
                        acc += work[size_t(r) * Db + (base | spread(jx))] * K[jx * Dc + jc];
                    o[2 * (size_t(r) * Db + c)] = acc.real();
                    o[2 * (size_t(r) * Db + c) + 1] = acc.imag();
                }
            }
        }
    }

    // ---- trajectories side by side

    bool resident() const { return m.n <= qs::kBatchLdsQubits; }

    // Whether the trajectories run side by side: on tiles of the default width,
    // in blocks that shared sweeps take.  (From 14 qubits on both ways round
    // alike, so each chunk of a concurrent call decides for itself.)
    bool side_by_side() const {
        if (tuning || one_by_one || plan_tile_bits() != qs::kDefaultTileBits) return false;
        const bool z = res.z_expect != nullptr;
        if (resident()) return side_call(m, p, z, call_traj) && resident_pays();
        return side_call(m, p, z, p.n_traj) && max_block() <= 4;
    }
    int max_block() const {
        int k = 0;
        for (const qs::Block &b : blocks) k = std::max(k, b.k);
        return k;
    }

    // Whether a call of resident states is faster side by side.  A few
    // trajectories are not where a workgroup is the slower place for their
    // blocks.  From three 5-qubit blocks on: they run on VALU there, but on
    // MFMA one by one from 11 qubits on (noiseless at max_fuse 5, in us a call
    // side by side and one by one: one of 11 / 12 / 13 qubits 343 / 355 / 396
    // and 104 / 125 / 176, three 350 / 365 / 404 and 241 / 307 / 440, four of
    // 11 354 and 309, thirty-two 401 / 416 / 458 and 2200 / 2894 / 4363), and
    // below 10 qubits on more than one workgroup (one of 6 / 9 qubits 193 / 238
    // and 145 / 184; of 10, on one either way, 256 and 280).  A 13-qubit state
    // without inner-product channels fills a workgroup's tile either way, and
    // small blocks cross it faster in sweeps (max_fuse 1 / 2 / 3 204 / 205 /
    // 138 and 189 / 189 / 126; with 4-qubit blocks 110 and 120).
    bool resident_pays() const {
        size_t k5 = 0, k4 = 0, all = 0;
        for (const BlockDesc &d : block_desc) {
            if (d.identity) continue;
            ++all;
            k5 += d.g.k == 5;
            k4 += d.g.k == 4;
        }
        if (k5 > 2 || 2 * k5 > all) return m.n == 10 || call_traj > (m.n < 10 ? 1 : m.n == 11 ? 4 : 3);
        if (m.n < qs::kBatchLdsQubits || call_traj > 1 || k4 + k5 > 0) return true;
        for (const ChannelInfo &c : m.channels)
            if (!c.mixture) return true;
        return false;
    }

    // Program of one trajectory (any host thread): as run_delayed, without
    // launching anything.  A trajectory whose norm bound would call for a
    // renormalisation in between is left to run_delayed.
    void plan_trajectory(int64_t rel, uint32_t traj, TrajPlan &P) const {
        P = TrajPlan();
        const int nch = int(m.channels.size());
        const int n_ops = int(m.ops.size());
        std::vector<int> pick(nch, -1), slow;  // slow: channel indices
        std::vector<double> resid(nch, 0.0);
        std::vector<const cd *> mats = default_mats;
        std::vector<char> dirty(blocks.size(), 0);
        for (int c = 0; c < nch; ++c) {
            const ChannelInfo &ci = m.channels[c];
            const double r = qs::philox_uniform(p.seed, channel_draw_index(uint32_t(c)), traj, p.circuit_id,
                                                qs::kStreamChannel);
            pick[c] = select_fast(ci, r, &resid[c]);
            if (pick[c] < 0) {
                slow.push_back(c);
            } else if (pick[c] != ci.default_pick) {
                mats[ci.op] = fast_pick_matrix(ci, pick[c]);
                dirty[op_block[ci.op]] = 1;
            }
        }
        int8_t *choices = res.kraus_choices ? res.kraus_choices + rel * nch : nullptr;
        int8_t *paths = res.kraus_paths ? res.kraus_paths + rel * nch : nullptr;
        for (int c = 0; c < nch; ++c) {
            if (choices) choices[c] = int8_t(pick[c]);
            if (paths) paths[c] = pick[c] < 0 ? 1 : 0;
        }
        if (res.n_slow) res.n_slow[rel] = int32_t(slow.size());

        std::vector<SegSweep> seg;
        std::deque<TileLayout> store;
        std::vector<int> sub, later;
        std::vector<cd> work;
        BlockDesc bd;
        double norm_bound = 0.0;
        int seg_start = 0, pending = -1;  // pending: the selection whose block is to come
        int unmade = -1;                  // the selection the next block follows
        auto push = [&](TrajPlan::Gate &g) {
            g.before = unmade;
            unmade = -1;
            P.gates.push_back(g);
        };
        auto reserve = [&](size_t f2) {
            const size_t at = P.mats.size();
            P.mats.resize(at + ((f2 + 3) & ~size_t(3)));
            return at;
        };
        for (size_t si = 0;; ++si) {
            const int seg_end = si < slow.size() ? m.channels[slow[si]].op : n_ops;
            // the one-by-one path's order of the blocks, also for a resident
            // state: from 10 qubits on the same trajectory then rounds alike
            // whichever way it runs, but for 5-qubit blocks of 11 to 13 qubits
            // (VALU in a workgroup, MFMA one by one); below 10 qubits the
            // kernels differ
            segment_sweeps(seg_start, seg_end, slow.empty(), store, seg);
            for (const SegSweep &ss : seg) {
                const size_t g0 = P.gates.size();
                double lb = 0.0;
                for (const auto &mem : ss.members) {
                    const int b = mem[0];
                    const auto &ops = blocks[b].ops;
                    const bool whole = mem[1] == 0 && mem[2] == int(ops.size());
                    TrajPlan::Gate g;
                    if (whole && !dirty[b]) {
                        if (block_desc[b].identity) continue;
                        g.k = block_desc[b].g.k;
                        for (int j = 0; j < 5; ++j) g.t[j] = block_desc[b].g.t[j];
                        g.dev = mat_of(block_desc[b]);
                        lb += block_desc[b].log_bound;
                        push(g);
                        continue;
                    }
                    sub.assign(ops.begin() + mem[1], ops.begin() + mem[2]);
                    if (pending >= 0 && m.channels[P.sels[pending].channel].op == sub[0]) {
                        TrajPlan::Select &S = P.sels[pending];
                        const ChannelInfo &ci = m.channels[S.channel];
                        int q[5] = {};
                        const int kb = qs::union_qubits(sub, m.ops, q);
                        if (kb > 4) return;
                        S.Db = 1 << kb;
                        later.assign(sub.begin() + 1, sub.end());
                        S.cand = reserve(size_t(ci.nk) * S.Db * S.Db * 2);
                        fill_candidates(ci, kb, q, later, mats, work, reinterpret_cast<double *>(&P.mats[S.cand]));
                        mats[ci.op] = ci.kraus + size_t(ci.nk - 1) * (size_t(1) << (2 * ci.k));
                        if (!resident()) S.dst = reserve(size_t(S.Db) * S.Db);
                        g.k = kb;
                        for (int j = 0; j < 5; ++j) g.t[j] = j < kb ? q[j] : 0;
                        g.sel = pending;
                        pending = -1;
                        push(g);
                        continue;
                    }
                    build_block(m, sub, mats, work, bd);
                    if (bd.identity) continue;
                    for (int o : sub) {
                        const int c = m.channel_of_op[o];
                        lb += c < 0 ? m.gate_log_bound[o] : (pick[c] >= 0 ? m.channels[c].log_pbar[pick[c]] : 0.0);
                    }
                    g.k = bd.g.k;
                    for (int j = 0; j < 5; ++j) g.t[j] = bd.g.t[j];
                    const size_t dd = size_t(1) << (2 * g.k);
                    g.off = reserve(dd);
                    std::memcpy(&P.mats[g.off], bd.g.m, sizeof(float2) * dd);
                    push(g);
                }
                norm_bound += lb;
                if (norm_bound < kRenormLogThreshold) return;
                if (P.gates.size() == g0) continue;
                ++P.sweeps;
                if (resident()) continue;
                TrajPlan::Cut c;
                c.g0 = int(g0);
                c.g1 = int(P.gates.size());
                set_tile(P, c, -1);
                P.cuts.push_back(c);
            }
            if (si == slow.size()) break;
            // the channel at seg_end: its qubit in the last sweep's tile, or in
            // a sweep without gates that only forms the density matrix
            TrajPlan::Select S;
            S.channel = slow[si];
            S.resid = resid[slow[si]];
            pending = unmade = int(P.sels.size());
            P.sels.push_back(S);
            if (!resident()) {
                const int q = m.channels[S.channel].t[0];
                if (P.cuts.empty() || P.cuts.back().sel >= 0 || !set_tile(P, P.cuts.back(), q)) {
                    TrajPlan::Cut c;
                    c.g0 = c.g1 = int(P.gates.size());
                    set_tile(P, c, q);
                    P.cuts.push_back(c);
                }
                P.cuts.back().sel = pending;
                P.cuts.back().rdm_q = q;
            }
            dirty[op_block[seg_end]] = 1;
            norm_bound = 0.0;  // renormalised by the folded 1/sqrt(p N)
            seg_start = seg_end;
        }
        if (!resident() && P.cuts.empty()) {  // no operation left: a sweep that writes |0...0>
            TrajPlan::Cut c;
            set_tile(P, c, -1);
            P.cuts.push_back(c);
        }
        P.ok = true;
    }

    // The tile of a side-by-side sweep: its gates' bits, then `extra` (>= 0),
    // then the lowest others.  Returns whether it holds `extra`.
    bool set_tile(const TrajPlan &P, TrajPlan::Cut &c, int extra) const {
        std::array<char, qs::kMaxQubits> in{};
        int cnt = 0;
        auto take = [&](int q) {
            if (cnt < qs::kBatchTileBits && !in[size_t(q)]) {
                in[size_t(q)] = 1;
                ++cnt;
            }
        };
        for (int q = 0; q < qs::kTileLowBits; ++q) take(q);
        for (int g = c.g0; g < c.g1; ++g)
            for (int j = 0; j < P.gates[size_t(g)].k; ++j) take(P.gates[size_t(g)].t[j]);
        if (extra >= 0) take(extra);
        for (int q = 0; q < m.n; ++q) take(q);
        int i = 0;
        for (int q = 0; q < m.n; ++q)
            if (in[size_t(q)]) c.pos[i++] = q;
        return extra < 0 || in[size_t(extra)];
    }

    // Workspace of the side-by-side sweeps: the states beside the caller's
    // and the workgroup records; false when there is no room for it.
    bool ensure_side(int slots, bool all_states) {
        const size_t dim = size_t(1) << m.n;
        const size_t states = (all_states ? size_t(slots) : size_t(slots) - 1) * dim * sizeof(float2);
        const size_t rec = resident() ? 0 : size_t(slots) * (size_t(1) << (m.n - qs::kBatchTileBits)) * 8 * sizeof(double);
        if (states + rec <= s->side_cap) return true;
        if (s->side_buf) {
            if (hipStreamSynchronize(s->st) != hipSuccess) return false;
            (void)hipFree(s->side_buf);
        }
        s->side_buf = nullptr;
        s->side_cap = 0;
        if (hipMalloc(&s->side_buf, states + rec) != hipSuccess) {
            (void)hipGetLastError();
            s->side_buf = nullptr;
            return false;
        }
        s->side_cap = states + rec;
        return true;
    }

    // What a finished trajectory leaves: samples and a Z record in their
    // places in the call's buffers.
    qs_status finish_side(int64_t rel, float2 *amp) {
        const uint32_t traj = uint32_t(p.traj_offset + rel);
        if (p.n_samples > 0) {
            QS_HIP(s, qs::launch_sample(amp, s->n, s->samp_sums, s->samp_incl, p.seed, traj, p.circuit_id,
                                        p.n_samples, ro, s->samp_out + rel * p.n_samples, s->samp_norm, s->st));
            res.sweeps += 1;
        }
        if (res.z_expect) {
            QS_HIP(s, qs::launch_zweights(amp, s->n, s->red_partials, s->z_dev + size_t(rel) * qs::kZRecord, s->st));
            res.sweeps += 1;
        }
        return QS_OK;
    }

    static size_t f2_of(size_t bytes) { return (bytes + 255) / 256 * 32; }

    size_t program_f2(const TrajPlan &P) const {
        return f2_of(P.mats.size() * sizeof(float2)) + f2_of(P.gates.size() * sizeof(qs::TrajGate)) +
               f2_of(P.cuts.size() * sizeof(qs::TrajSweep)) + f2_of(P.sels.size() * sizeof(qs::TrajSelect)) +
               f2_of(sizeof(qs::TrajJob)) + 64;
    }

    // Launches trajectories [first, first + plans.size()) of the call from
    // their programs, staged in the arena with one copy.
    qs_status launch_side(int64_t first, const TrajPlan *plans, const std::vector<int> &which, int slots) {
        const size_t n_traj = which.size();
        size_t mats = 0, n_gates = 0, n_cuts = 0, n_sels = 0;
        for (int w : which) {
            mats += plans[w].mats.size();
            n_gates += plans[w].gates.size();
            n_cuts += plans[w].cuts.size();
            n_sels += plans[w].sels.size();
        }
        if (choice_owner.size() + n_sels > size_t(kChoiceCap)) QS_CHECK(drain_choices());
        if (n_sels > 0) QS_CHECK(open_selections());
        const size_t f_gate = f2_of(n_gates * sizeof(qs::TrajGate)), f_sel = f2_of(n_sels * sizeof(qs::TrajSelect)),
                     f_cut = f2_of(n_cuts * sizeof(qs::TrajSweep)), f_job = f2_of(n_traj * sizeof(qs::TrajJob));
        float2 *h = nullptr;
        const float2 *d = nullptr;
        const size_t need = f2_of(mats * sizeof(float2)) + f_gate + f_sel + f_cut + f_job;
        QS_CHECK(arena_reserve(s, need <= kArenaSmallHalf / 2 ? kArenaSmallHalf : kArenaHalf));
        QS_CHECK(arena_stage(s, need, &h, &d));
        const size_t o_gate = f2_of(mats * sizeof(float2)), o_sel = o_gate + f_gate, o_cut = o_sel + f_sel,
                     o_job = o_cut + f_cut;
        auto *gates = reinterpret_cast<qs::TrajGate *>(h + o_gate);
        auto *sels = reinterpret_cast<qs::TrajSelect *>(h + o_sel);
        auto *cuts = reinterpret_cast<qs::TrajSweep *>(h + o_cut);
        auto *jobs = reinterpret_cast<qs::TrajJob *>(h + o_job);
        const bool keep = p.n_samples > 0 || res.z_expect;
        const size_t dim = size_t(1) << m.n;
        const int64_t last = p.n_traj - 1;
        // matrices, gates and selections trajectory by trajectory
        std::vector<size_t> mat0(n_traj), gate0(n_traj), sel0(n_traj);
        size_t mo = 0, go = 0, so = 0;
        for (size_t i = 0; i < n_traj; ++i) {
            const TrajPlan &P = plans[which[i]];
            res.sweeps += P.sweeps;
            res.gate_sweeps += P.sweeps;
            if (P.sweeps > 0) res.zero_start_sweeps++;
            mat0[i] = mo;
            gate0[i] = go;
            sel0[i] = so;
            if (!P.mats.empty()) std::memcpy(h + mo, P.mats.data(), sizeof(float2) * P.mats.size());
            mo += P.mats.size();
            so += P.sels.size();
            auto emit = [&](const TrajPlan::Gate &g, const int *pos, int &lofs) {
                int lt[qs::kMaxGateQubits];
                for (int j = 0; j < g.k; ++j)
                    lt[j] = pos ? int(std::find(pos, pos + qs::kBatchTileBits, g.t[j]) - pos) : g.t[j];
                qs::TrajGate &G = gates[go++];
                G.g = qs::batch_tile_gate(g.k, lt, lofs);
                lofs += qs::tile_mat_slots(g.k);
                if (g.sel >= 0) G.g.head |= qs::kSelectedGate;
                G.sel = g.before >= 0 ? int(sel0[i]) + g.before : -1;
                G.m = g.dev ? g.dev : d + mat0[i] + (g.sel >= 0 ? P.sels[size_t(g.sel)].dst : g.off);
                res.gate_k_launches[g.k]++;
            };
            if (resident()) {
                int lofs = 0;
                for (const auto &g : P.gates) emit(g, nullptr, lofs);
            } else {
                for (const auto &c : P.cuts) {
                    int lofs = 0;
                    for (int g = c.g0; g < c.g1; ++g) emit(P.gates[size_t(g)], c.pos, lofs);
                }
            }
        }
        auto fill_select = [&](qs::TrajSelect &D, size_t i, size_t si, const double *records) {
            const TrajPlan &P = plans[which[i]];
            const TrajPlan::Select &S = P.sels[si];
            const ChannelInfo &ci = m.channels[S.channel];
            D.excess = chan_excess[S.channel];
            D.pbar = chan_pbar[S.channel];
            D.cand = reinterpret_cast<const double *>(d + mat0[i] + S.cand);
            D.dst = const_cast<float2 *>(d + mat0[i] + S.dst);
            D.records = records;
            D.choice = dev_choice + choice_owner.size();
            D.err = dev_error;
            D.resid = S.resid;
            D.nk = ci.nk;
            D.k = ci.k;
            D.Db = S.Db;
            D.n_records = 0;  // set with the step's workgroup count
            for (int j = 0; j < 2; ++j) D.t[j] = j < ci.k ? ci.ts[j] : 0;
            choice_owner.emplace_back(first + which[i], S.channel);
        };
        float2 *side = s->side_buf;
        if (resident()) {
            for (size_t i = 0; i < n_traj; ++i) {
                const TrajPlan &P = plans[which[i]];
                const bool is_last = first + which[i] == last;
                jobs[i].g0 = int(gate0[i]);
                jobs[i].n_gates = int(P.gates.size());
                jobs[i].out = is_last ? s->amp : (keep ? side + size_t(i) * dim : nullptr);
                for (size_t si = 0; si < P.sels.size(); ++si) fill_select(sels[sel0[i] + si], i, si, nullptr);
            }
            QS_CHECK(arena_commit(s));
            qs::TrajResidentArgs A;
            A.jobs = reinterpret_cast<const qs::TrajJob *>(d + o_job);
            A.gates = reinterpret_cast<const qs::TrajGate *>(d + o_gate);
            A.sels = reinterpret_cast<const qs::TrajSelect *>(d + o_sel);
            A.n = m.n;
            QS_HIP(s, qs::launch_traj_resident(A, int(n_traj), s->st));
            if (keep)
                for (size_t i = 0; i < n_traj; ++i)
                    QS_CHECK(finish_side(first + which[i], first + which[i] == last ? s->amp : side + i * dim));
            return QS_OK;
        }
        // each state runs a queue of trajectories; the call's last one ends
        // the queue of the caller's state (state 0)
        std::vector<std::vector<size_t>> queue(static_cast<size_t>(slots));
        {
            std::vector<size_t> load(size_t(slots), 0);
            size_t n_free = n_traj;
            const bool has_last = first + which[n_traj - 1] == last;
            if (has_last) {
                --n_free;
                load[0] = plans[which[n_free]].cuts.size();
            }
            for (size_t i = 0; i < n_free; ++i) {
                const size_t q = size_t(std::min_element(load.begin(), load.end()) - load.begin());
                load[q] += plans[which[i]].cuts.size();
                queue[q].push_back(i);
            }
            if (has_last) queue[0].push_back(n_free);
        }
        const size_t rec_len = (size_t(1) << (m.n - qs::kBatchTileBits)) * 8;
        double *records = reinterpret_cast<double *>(side + size_t(slots - 1) * dim);
        struct Step {
            size_t c0, c1, s0, s1;
            std::vector<std::pair<size_t, size_t>> ends;  // (trajectory, state)
        };
        std::vector<Step> steps;
        std::vector<size_t> qi(size_t(slots), 0), ci(size_t(slots), 0);
        size_t co = 0;
        so = 0;
        for (;;) {
            Step st{co, co, so, so, {}};
            for (size_t q = 0; q < size_t(slots); ++q) {
                if (qi[q] >= queue[q].size()) continue;
                const size_t i = queue[q][qi[q]];
                const TrajPlan &P = plans[which[i]];
                const TrajPlan::Cut &c = P.cuts[ci[q]];
                qs::TrajSweep &D = cuts[co++];
                D.amp = q == 0 ? s->amp : side + (q - 1) * dim;
                D.rdm_out = c.sel >= 0 ? records + q * rec_len : nullptr;
                for (int b = 0; b < qs::kMaxTileBits; ++b) D.pos[b] = c.pos[b];
                D.g0 = int(gate0[i]) + c.g0;
                D.n_gates = c.g1 - c.g0;
                D.init_zero = ci[q] == 0 ? 1 : 0;
                D.rdm_lt = c.sel >= 0 ? int(std::find(c.pos, c.pos + qs::kBatchTileBits, c.rdm_q) - c.pos) : 0;
                if (c.sel >= 0) fill_select(sels[so++], i, size_t(c.sel), records + q * rec_len);
                if (++ci[q] == P.cuts.size()) {
                    st.ends.emplace_back(i, q);
                    ci[q] = 0;
                    ++qi[q];
                }
            }
            if (co == st.c0) break;
            st.c1 = co;
            st.s1 = so;
            for (size_t i = st.s0; i < st.s1; ++i)
                sels[i].n_records = qs::traj_sweep_groups(m.n, int(st.c1 - st.c0));
            steps.push_back(std::move(st));
        }
        QS_CHECK(arena_commit(s));
        const auto *dcuts = reinterpret_cast<const qs::TrajSweep *>(d + o_cut);
        const auto *dgates = reinterpret_cast<const qs::TrajGate *>(d + o_gate);
        const auto *dsels = reinterpret_cast<const qs::TrajSelect *>(d + o_sel);
        for (const Step &st : steps) {
            QS_HIP(s, qs::launch_traj_sweep(dcuts + st.c0, dgates, m.n, int(st.c1 - st.c0), s->st));
            if (st.s1 > st.s0) QS_HIP(s, qs::launch_traj_select(dsels + st.s0, int(st.s1 - st.s0), s->st));
            for (const auto &e : st.ends) {
                QS_CHECK(finish_side(first + which[e.first], e.second == 0 ? s->amp : side + (e.second - 1) * dim));
            }
        }
        return QS_OK;
    }

    // The call's trajectories side by side; *done stays false when there is
    // no room for the workspace.
    qs_status run_side_by_side(bool *done) {
        const bool keep = p.n_samples > 0 || res.z_expect;
        const int slots =
            resident() ? 256
                       : int(std::min<int64_t>(std::max(kSideTiles >> (m.n - qs::kBatchTileBits), 2),
                                               std::min<int64_t>(p.n_traj, 64)));
        // (the call's last trajectory ends in the caller's state)
        if (resident() ? keep && !ensure_side(int(std::min<int64_t>(slots, p.n_traj - 1)), true)
                       : !ensure_side(slots, false))
            return QS_OK;
        *done = true;
        QS_CHECK(restore_home(s));
        const int64_t chunk = resident() ? 256 : std::max<int64_t>(4 * slots, 32);
        std::vector<TrajPlan> plans;
        std::vector<int> which;
        for (int64_t first = 0; first < p.n_traj; first += chunk) {
            const int64_t count = std::min<int64_t>(chunk, p.n_traj - first);
            plans.resize(size_t(count));
            // a thread for about 40 us of planning (1000 operations; a channel that
            // needs inner products weighs as 500): less is done before a helper
            // is awake
            const double load = double(count) * (double(m.ops.size()) + 500.0 * expected_slow_paths(m));
            const unsigned threads = unsigned(std::min(16.0, 1.0 + load / 1000.0));
            qs::HostPool::get().run(size_t(count), 1, threads, [&](size_t lo, size_t hi) {
                for (size_t i = lo; i < hi; ++i)
                    plan_trajectory(first + int64_t(i), uint32_t(p.traj_offset + first + int64_t(i)), plans[i]);
            });
            // the ones left to the one-by-one path, in the caller's state; the
            // call's last trajectory stays last there
            auto alone = [&](int64_t i) -> qs_status {
                QS_CHECK(arena_reserve(s, kArenaHalf));
                QS_CHECK(run_delayed(first + i, uint32_t(p.traj_offset + first + i)));
                QS_CHECK(settle_reset());
                return finish_side(first + i, s->amp);
            };
            auto fits = [&](int64_t i) { return plans[size_t(i)].ok && program_f2(plans[size_t(i)]) <= kArenaHalf / 2; };
            for (int64_t i = 0; i < count; ++i)
                if (!fits(i) && first + i != p.n_traj - 1) QS_CHECK(alone(i));
            which.clear();
            size_t f2 = 0;
            for (int64_t i = 0; i < count; ++i) {
                if (!fits(i)) continue;
                const size_t need = program_f2(plans[size_t(i)]);
                if (!which.empty() && f2 + need > kArenaHalf) {
                    QS_CHECK(launch_side(first, plans.data(), which, slots));
                    which.clear();
                    f2 = 0;
                }
                which.push_back(int(i));
                f2 += need;
            }
            if (!which.empty()) QS_CHECK(launch_side(first, plans.data(), which, slots));
            if (first + count == p.n_traj && !fits(count - 1)) QS_CHECK(alone(count - 1));
        }
        pending_reset = false;
        if (p.n_samples > 0) {
            sample_first_traj = 0;
            sample_fill = p.n_traj * p.n_samples;
        }
        if (res.z_expect) {
            z_first_traj = 0;
            z_fill = p.n_traj;
        }
        return QS_OK;
    }

    qs_status run_delayed(int64_t rel, uint32_t traj) {
        const int nch = int(m.channels.size());
        // steps 1-11 of Algorithm 2 for every channel: state-independent
        std::vector<int> pick(nch, -1);
        std::vector<double> resid(nch, 0.0);
        std::vector<int> slow_ops;
        std::vector<std::pair<int, const cd *>> overrides;  // (op, matrix)
        std::vector<double> override_log;
        for (int c = 0; c < nch; ++c) {
            const ChannelInfo &ci = m.channels[c];
            const double r = qs::philox_uniform(p.seed, channel_draw_index(uint32_t(c)), traj,
                                                p.circuit_id, qs::kStreamChannel);
            pick[c] = select_fast(ci, r, &resid[c]);
            if (pick[c] < 0) {
                slow_ops.push_back(ci.op);
            } else if (pick[c] != ci.default_pick) {
                overrides.emplace_back(ci.op, fast_pick_matrix(ci, pick[c]));
            }
        }
        int8_t *choices = res.kraus_choices ? res.kraus_choices + rel * nch : nullptr;
        int8_t *paths = res.kraus_paths ? res.kraus_paths + rel * nch : nullptr;
        for (int c = 0; c < nch; ++c) {
            if (choices) choices[c] = int8_t(pick[c]);
            if (paths) paths[c] = pick[c] < 0 ? 1 : 0;
        }
        if (res.n_slow) res.n_slow[rel] = int32_t(slow_ops.size());

        QS_CHECK(restore_home(s));
        pending_reset = true;  // the first tile sweep writes |0...0> itself
        log_norm_bound = 0.0;

        std::vector<const cd *> mats = default_mats;
        std::vector<char> dirty(blocks.size(), 0);
        for (auto &ov : overrides) {
            mats[ov.first] = ov.second;
            dirty[op_block[ov.first]] = 1;
        }
        if (graph_wanted && slow_ops.empty()) {
            bool used = false;
            QS_CHECK(try_graph(mats, dirty, pick, &used));
            if (used) return QS_OK;
        }
        slow_mats.clear();
        const int n_ops = int(m.ops.size());
        int seg_start = 0;
        int slow_idx = 0;
        std::vector<int> sub;
        std::deque<BlockDesc> dyn;
        std::vector<Unit> units;
        std::vector<SegSweep> seg;
        run_layouts.clear();
        for (;;) {
            const int seg_end = slow_idx < int(slow_ops.size()) ? slow_ops[slow_idx] : n_ops;
            dyn.clear();
            units.clear();
            segment_sweeps(seg_start, seg_end, slow_ops.empty(), run_layouts, seg);
            for (const SegSweep &ss : seg) {
                Unit unit{ss.L, {}};
                for (const auto &mem : ss.members) {
                    const int b = mem[0];
                    const auto &ops = blocks[b].ops;
                    auto lo = ops.begin() + mem[1];
                    auto hi = ops.begin() + mem[2];
                    if (lo == hi) continue;
                    const bool whole = (lo == ops.begin() && hi == ops.end());
                    if (whole && !dirty[b]) {
                        if (!block_desc[b].identity) unit.items.push_back(&block_desc[b]);
                        continue;
                    }
                    sub.assign(lo, hi);
                    dyn.emplace_back();
                    BlockDesc &bd = dyn.back();
                    const bool holds_slow = sel.active && !sel.staged && *lo == sel.op;
                    if (holds_slow) {
                        // one candidate matrix per Kraus operator; the select kernel
                        // scales the chosen one into this block's slot
                        const ChannelInfo &ci = m.channels[sel.channel];
                        const int Dc = 1 << ci.k;
                        int q[5];
                        const int kb = qs::union_qubits(sub, m.ops, q);
                        const int Db = 1 << kb;
                        const size_t cand_f2 = size_t(ci.nk) * Db * Db * 2;  // complex128 as float2 pairs
                        const size_t need = cand_f2 + size_t(Db) * Db + 64;
                        if (!arena_fits(s, need)) QS_CHECK(flush_units(units));
                        float2 *hc = nullptr;
                        const float2 *dc = nullptr;
                        QS_CHECK(arena_stage(s, cand_f2, &hc, &dc));
                        double *hcd = reinterpret_cast<double *>(hc);
                        rest_ops.assign(sub.begin() + 1, sub.end());
                        fill_candidates(ci, kb, q, rest_ops, mats, tmp, hcd);
                        mats[sel.op] = ci.kraus + size_t(ci.nk - 1) * Dc * Dc;
                        bd.g.k = kb;
                        for (int b2 = 0; b2 < 5; ++b2) bd.g.t[b2] = b2 < kb ? q[b2] : 0;
                        bd.identity = false;
                        bd.log_bound = 0.0;
                        float2 *hd = nullptr;
                        QS_CHECK(arena_stage(s, size_t(Db) * Db, &hd, &bd.dev));
                        std::memset(hd, 0, sizeof(float2) * Db * Db);
                        if (int(choice_owner.size()) >= kChoiceCap) {
                            QS_CHECK(flush_units(units));
                            QS_CHECK(drain_choices());
                        }
                        qs::SelectArgs &A = sel.args;
                        A.rdm = sel_rdm;
                        A.excess = chan_excess[sel.channel];
                        A.pbar = chan_pbar[sel.channel];
                        A.cand = reinterpret_cast<const double *>(dc);
                        A.dst = const_cast<float2 *>(bd.dev);
                        A.choice = dev_choice + choice_owner.size();
                        A.err = dev_error;
                        QS_CHECK(open_selections());
                        A.resid = sel.resid;
                        A.nk = ci.nk;
                        A.D = Dc;
                        A.Db = Db;
                        choice_owner.emplace_back(rel, sel.channel);
                        sel.staged = true;
                        unit.items.push_back(&bd);
                        continue;
                    }
                    build_block(m, sub, mats, tmp, bd);
                    if (bd.identity) continue;
                    double lb = 0.0;
                    for (int o : sub) {
                        if (m.kind[o] == QS_OP_GATE) lb += m.gate_log_bound[o];
                        else {
                            const ChannelInfo &ci = m.channels[m.channel_of_op[o]];
                            const int pk = pick[m.channel_of_op[o]];
                            lb += pk >= 0 ? ci.log_pbar[pk] : 0.0;
                        }
                    }
                    bd.log_bound = lb;
                    if (!arena_fits(s, size_t(1) << (2 * bd.g.k))) QS_CHECK(flush_units(units));
                    QS_CHECK(stage_block(s, bd));
                    unit.items.push_back(&bd);
                }
                if (!unit.items.empty()) units.push_back(std::move(unit));
            }
            // the segment's last sweep forms the next channel's reduced density
            // matrix when its tile holds the channel's qubit (and it has no
            // 5-qubit block); otherwise a read pass does, below
            bool rdm_fused = false;
            const int rq = seg_end < n_ops ? rdm_qubit(seg_end) : -1;
            if (rq >= 0 && !units.empty()) {
                Unit &lu = units.back();
                bool k5 = false;
                double lb = 0.0;
                for (const BlockDesc *d : lu.items) {
                    k5 |= d->g.k == 5;
                    lb += d->log_bound;
                }
                if (lu.L->tiled && lu.L->tb >= 10 && lu.L->local[rq] >= 0 && !k5 &&
                    lb >= kRenormLogThreshold) {
                    QS_CHECK(ensure_reduce(s));
                    lu.rdm_q = rq;
                    rdm_fused = true;
                }
            }
            QS_CHECK(flush_units(units));
            sel = PendingSelect();
            if (seg_end == n_ops) break;
            // steps 12-20 for the channel at seg_end, without a host round trip:
            // one read pass forms R on the device; the select kernel launched
            // with the next segment picks the branch and scales its block
            const int c = m.channel_of_op[seg_end];
            const ChannelInfo &ci = m.channels[c];
            if (rdm_fused) {
                QS_HIP(s, qs::launch_reduce_records(s->red_partials + kRdmRecordOffset, rdm_records, 8,
                                                    sel_rdm, s->st));
            } else {
                QS_CHECK(settle_reset());
                QS_CHECK(ensure_reduce(s));
                QS_HIP(s, qs::launch_rdm(s->amp, s->n, ci.k, ci.ts, s->red_partials, sel_rdm, s->st));
                res.sweeps++;
            }
            sel.active = true;
            sel.op = seg_end;
            sel.channel = c;
            sel.resid = resid[c];
            dirty[op_block[seg_end]] = 1;
            log_norm_bound = 0.0;  // renormalised by the folded 1/sqrt(p N)
            seg_start = seg_end;
            ++slow_idx;
        }
        return QS_OK;
    }

    qs_status run_naive(int64_t rel, uint32_t traj) {
        const int nch = int(m.channels.size());
        int8_t *choices = res.kraus_choices ? res.kraus_choices + rel * nch : nullptr;
        int8_t *paths = res.kraus_paths ? res.kraus_paths + rel * nch : nullptr;
        QS_CHECK(restore_home(s));
        QS_HIP(s, qs::launch_set_basis(s->amp, s->n, 0, s->st));
        log_norm_bound = 0.0;
        pending_scale = 1.0;
        for (int c = 0; c <= nch; ++c) {
            for (const auto &d : naive_segments[c]) QS_CHECK(launch_block(d));
            if (c == nch) break;
            const ChannelInfo &ci = m.channels[c];
            const double r = qs::philox_uniform(p.seed, channel_draw_index(uint32_t(c)), traj,
                                                p.circuit_id, qs::kStreamChannel);
            int pk = -1;
            double accepted = 0.0;
            QS_CHECK(naive_channel(s, ci, r, &pk, &accepted));
            res.sweeps += pk + 1;
            if (!(accepted > 0.0)) return fail(QS_ERR_ZERO_NORM, "chosen Kraus operator has zero weight");
            if (choices) choices[c] = int8_t(pk);
            if (paths) paths[c] = 1;
            // |psi> <- K_i |psi> / sqrt(p_i): the stored vector is now K_i psi_stored with
            // norm^2 `accepted`, so 1/sqrt(accepted) (replacing any scale still
            // pending for the old vector) normalises it; fold it into the next block
            pending_scale = 1.0 / std::sqrt(accepted);
            if (pending_scale > 1e15 || pending_scale < 1e-15) {
                QS_HIP(s, qs::launch_scale(s->amp, s->n, float(pending_scale), s->st));
                res.sweeps++;
                pending_scale = 1.0;
            }
        }
        if (res.n_slow) res.n_slow[rel] = nch;
        return QS_OK;
    }

    qs_status run() {
        QS_CHECK(fill_readout(m.n, p.p0to1, p.p1to0, ro));
        if (p.n_samples > 0) {
            const int64_t total = p.n_traj * int64_t(p.n_samples);
            const int64_t cap = std::max<int64_t>(p.n_samples, std::min<int64_t>(total, kSampleRecords));
            QS_CHECK(ensure_sampling(s, size_t(cap)));
        }
        QS_CHECK(ensure_reduce(s));
        if (res.z_expect && p.n_traj > 0)
            QS_CHECK(ensure_zrecords(s, size_t(std::min<int64_t>(p.n_traj, kZRecords))));
        timing = (p.flags & QS_TRAJ_TIME_KERNELS) != 0;
        if (timing) QS_CHECK(timer.init(s, 256));
        // the in-place conventional mode runs on the delayed machinery (its
        // channels carry zero bounds, so every one takes the inner-product path)
        const bool delayed = p.mode != QS_KRAUS_NAIVE;
        if (delayed) QS_CHECK(plan_delayed());
        else QS_CHECK(plan_naive());
        graph_wanted = !tuning && graph_call(m, p, p.n_traj);
        bool side = false;
        if (delayed && side_by_side()) QS_CHECK(run_side_by_side(&side));
        if (!side && s->arena_dev) QS_CHECK(arena_reserve(s, kArenaHalf));
        for (int64_t rel = side ? p.n_traj : 0; rel < p.n_traj; ++rel) {
            const uint32_t traj = uint32_t(p.traj_offset + rel);
            if (delayed) QS_CHECK(run_delayed(rel, traj));
            else QS_CHECK(run_naive(rel, traj));
            QS_CHECK(settle_reset());
            QS_CHECK(sample_trajectory(rel, traj));
            QS_CHECK(z_trajectory(rel));
        }
        QS_CHECK(flush_samples());
        QS_CHECK(flush_z());
        if (delayed) QS_CHECK(drain_choices());
        if (timing) {
            QS_CHECK(timer.finish(s));
            res.gate_kernel_ms = timer.total_ms;
            res.gate_kernel_launches = timer.count;
        }
        if ((p.flags & QS_TRAJ_RETURN_STATE) && res.final_state && p.n_traj > 0) {
            QS_HIP(s, hipStreamSynchronize(s->st));
            QS_HIP(s, hipMemcpy(res.final_state, s->amp, sizeof(float2) << s->n, hipMemcpyDeviceToHost));
        }
        QS_CHECK(restore_home(s));
        QS_HIP(s, hipStreamSynchronize(s->st));
        return QS_OK;
    }
};

}  // namespace

namespace {

// ---- autotuning of the fusion width and the tile width
// Section 3.2: the best largest fused-gate size depends on the circuit and
// the machine (larger on GPUs and for large circuits), and the choice is left
// to trying values.  Here the driver tries them, on the path that the call
// takes: for every candidate pair of widths it plans the circuit's default
// plan (each channel at its most likely pick) and times one pass of it from
// |0...0> on the state's own stream, keeping the fastest.  Where the channels'
// bounds predict two or more inner-product channels per trajectory, and where
// the call can run side by side, it times some of the call's trajectories
// instead, host planning included.  The choice is cached per (circuit, size,
// mode, kind of call) for the life of the process, so later calls, and the
// chunks of a concurrent call, run the same plan.
// Kinds of call: passes of one state; one trajectory of at most 13 qubits; 2 to
// 7, 8 to 31, and more trajectories side by side (the launches of a few are
// bound by their chain of blocks, those of many by planning and by the work:
// 8 qubits without noise, 3 trajectories 83 us at max_fuse 2 and 138 at 4, 100
// trajectories 408 and 270).
enum TuneKind { kTuneOneByOne, kTuneResident, kTuneFew, kTuneSome, kTuneMany };
struct TuneKey {
    uint64_t hash;
    int n, mode, f_req, tb_req, kind;
    bool operator<(const TuneKey &o) const {
        return std::tie(hash, n, mode, f_req, tb_req, kind) <
               std::tie(o.hash, o.n, o.mode, o.f_req, o.tb_req, o.kind);
    }
};

constexpr double kTuneMargin = 0.03;  // a candidate must beat the default widths by 3 %
// From this many expected inner-product channels per trajectory on, the
// trials are whole trajectories timed on the host clock (the host's
// per-split planning then weighs as much as the sweeps), with a wider margin
// for their noisier timings.
constexpr double kTuneSlowPaths = 2.0;
constexpr double kTuneTrajMargin = 0.05;
constexpr int64_t kTuneTrajectories = 4;
// Trials of calls that can run side by side: up to this many trajectories.
constexpr int64_t kTuneSideTrajectories = 32;

std::mutex g_tune_mu;  // one tuning at a time: concurrent trials would disturb each other's timings
std::map<TuneKey, std::pair<int, int>> g_tune_cache;

// The widths a call runs with (tiles: 1 = none).  Tunes when max_fuse is 0
// in the delayed mode; otherwise max_fuse (0: 4) and tile_bits (0: 13).
qs_status resolve_widths(qs_state s, const CircuitModel &m, uint64_t chash, const qs_traj_params &p,
                         bool z_records, int *f_out, int *tb_out, double *tune_ms) {
    *tune_ms = 0.0;
    *f_out = p.max_fuse > 0 ? p.max_fuse : kDefaultFuse;
    *tb_out = p.tile_bits == 0 ? qs::kDefaultTileBits : p.tile_bits;
    const bool tb_ok = p.tile_bits == 0 || p.tile_bits == 1 ||
                       (p.tile_bits >= 10 && p.tile_bits <= qs::kMaxTileBits);
    if (p.max_fuse != 0 || p.mode != QS_KRAUS_DELAYED || p.n_traj <= 0 || !tb_ok || m.n != s->n)
        return QS_OK;
    const bool side = (p.tile_bits == 0 || p.tile_bits == qs::kDefaultTileBits) &&
                      side_call(m, p, z_records, p.n_traj);
    const TuneKind kind = !side ? kTuneOneByOne
                          : p.n_traj < 2 ? kTuneResident
                          : p.n_traj < 8 ? kTuneFew
                          : p.n_traj < kTuneSideTrajectories ? kTuneSome : kTuneMany;
    const bool several = kind >= kTuneFew;
    std::vector<int> fs = m.n < 16 ? std::vector<int>{2, 3, 4, 5} : std::vector<int>{3, 4, 5};
    if (several && m.n > qs::kBatchLdsQubits) fs.pop_back();
    // several trajectories run side by side on 13-bit tiles only, three to five
    // times as fast as one by one on any (200 trajectories of the grid at depth
    // 20, 12-bit tiles one by one against 13-bit side by side: 13 qubits 11.2k
    // against 53k trajectories/s, 14 qubits 9.6k against 49k, 16 qubits 7.4k
    // against 35k, 18 qubits 6.3k against 24k, 20 qubits 4.2k against 10k);
    // smaller states fit one tile of any width
    std::vector<int> tbs;
    if (p.tile_bits != 0) tbs = {p.tile_bits};
    else if (!several && m.n > 12) tbs = {12, 13, 14};
    else tbs = {qs::kDefaultTileBits};
    const TuneKey key{chash, m.n, p.mode, p.max_fuse, p.tile_bits, kind};
    std::lock_guard<std::mutex> lock(g_tune_mu);
    auto it = g_tune_cache.find(key);
    if (it != g_tune_cache.end()) {
        *f_out = it->second.first;
        *tb_out = it->second.second;
        return QS_OK;
    }
    const auto t0 = std::chrono::steady_clock::now();
    hipEvent_t ev[2] = {nullptr, nullptr};
    for (auto &e : ev) QS_HIP(s, hipEventCreateWithFlags(&e, hipEventDisableSystemFence));
    struct EvGuard {
        hipEvent_t *e;
        ~EvGuard() {
            for (int i = 0; i < 2; ++i)
                if (e[i]) (void)hipEventDestroy(e[i]);
        }
    } guard{ev};
    const int reps = m.n >= 29 ? 1 : 2;  // the first of two also warms caches
    // circuits whose trajectories often need inner products, and calls that can
    // run side by side, are timed over the call's first few trajectories (the
    // same draws for every candidate) after a run of others that loads each
    // candidate's plan and kernels; side by side a call takes as little as
    // 50 us, so the fastest of five counts (fewer where the candidate is out)
    const bool by_traj = side || expected_slow_paths(m) >= kTuneSlowPaths;
    const int64_t nt = std::min<int64_t>(side ? kTuneSideTrajectories : kTuneTrajectories, p.n_traj);
    const int64_t warm_nt = side ? nt : 1;
    double best = 1e300, t_default = -1.0;
    for (int f : fs) {
        for (int tb : tbs) {
            qs_traj_params q = p;
            q.max_fuse = f;
            q.tile_bits = tb;
            q.flags = 0;
            q.n_samples = 0;
            q.p0to1 = q.p1to0 = nullptr;
            qs_traj_result dummy;
            std::memset(&dummy, 0, sizeof(dummy));
            double t = 1e300;
            if (by_traj) {
                q.n_traj = warm_nt;
                q.traj_offset = p.traj_offset + nt + warm_nt <= (int64_t(1) << 32) ? p.traj_offset + nt : p.traj_offset;
                Runner warm(s, m, q, dummy, chash, p.n_traj);
                warm.one_by_one = !side;
                QS_CHECK(warm.run());
                q.n_traj = nt;
                q.traj_offset = p.traj_offset;
                for (int r = 0; r < (side ? 5 : 1) && (r == 0 || t < 1.5 * best); ++r) {
                    const auto ta = std::chrono::steady_clock::now();
                    Runner trial(s, m, q, dummy, chash, p.n_traj);
                    trial.one_by_one = !side;
                    QS_CHECK(trial.run());  // ends with a stream synchronisation
                    t = std::min(t, 1e3 * std::chrono::duration<double>(std::chrono::steady_clock::now() - ta).count());
                }
            } else {
                Runner trial(s, m, q, dummy, chash, p.n_traj);
                trial.tuning = true;
                QS_CHECK(trial.plan_delayed());
                for (int r = 0; r < reps; ++r) {
                    QS_HIP(s, hipEventRecord(ev[0], s->st));
                    QS_CHECK(trial.run_default_plan());
                    QS_HIP(s, hipEventRecord(ev[1], s->st));
                    QS_HIP(s, hipEventSynchronize(ev[1]));
                    float ms = 0.f;
                    QS_HIP(s, hipEventElapsedTime(&ms, ev[0], ev[1]));
                    t = std::min(t, double(ms));
                }
            }
            if (f == kDefaultFuse && tb == (p.tile_bits == 0 ? qs::kDefaultTileBits : p.tile_bits))
                t_default = t;
            if (t < best) {
                best = t;
                *f_out = f;
                *tb_out = tb;
            }
        }
    }
    // the default widths stay unless another pair is clearly faster: trial
    // times of one pass differ by a percent or two from run to run
    const double margin = by_traj ? kTuneTrajMargin : kTuneMargin;
    if (t_default > 0.0 && best > (1.0 - margin) * t_default) {
        *f_out = kDefaultFuse;
        *tb_out = p.tile_bits == 0 ? qs::kDefaultTileBits : p.tile_bits;
    }
    g_tune_cache[key] = {*f_out, *tb_out};
    *tune_ms = 1e3 * std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return QS_OK;
}

// Tile width reported for a run: 1 when the plan uses no tiles.
int tile_bits_reported(int n, int tb) {
    return (tb >= 10 && n >= qs::kTileMinQubits) ? std::min(tb, n) : 1;
}

// qs_run_trajectories, optionally reporting every timed bracket of sweeps as
// an interval after the completed event `ref`; `call_traj`: trajectories of
// the concurrent call that these are a chunk of.
qs_status run_trajectories_impl(qs_state s, const qs_circuit *c, const qs_traj_params *p,
                                qs_traj_result *r, int64_t call_traj, hipEvent_t ref,
                                std::vector<std::pair<double, double>> *intervals) {
    const auto t0 = std::chrono::steady_clock::now();
    QS_CHECK(check_handle(s));
    if (!c || !p || !r) return fail(QS_ERR_INVALID_ARGUMENT, "null argument");
    if (c->n_qubits != s->n) return fail(QS_ERR_INVALID_ARGUMENT, "circuit and state qubit counts differ");
    if (p->n_traj < 0 || p->traj_offset < 0 || p->traj_offset + p->n_traj > (int64_t(1) << 32))
        return fail(QS_ERR_INVALID_ARGUMENT, "trajectory range outside 32-bit counters");
    if (p->mode != QS_KRAUS_DELAYED && p->mode != QS_KRAUS_NAIVE &&
        p->mode != QS_KRAUS_CONVENTIONAL_INPLACE)
        return fail(QS_ERR_INVALID_ARGUMENT, "bad mode");
    if (p->max_fuse < 0 || p->max_fuse > qs::kMaxGateQubits)
        return fail(QS_ERR_INVALID_ARGUMENT, "max_fuse outside 0..5");
    if (!(p->tile_bits == 0 || p->tile_bits == 1 ||
          (p->tile_bits >= 10 && p->tile_bits <= qs::kMaxTileBits)))
        return fail(QS_ERR_INVALID_ARGUMENT, "tile_bits must be 0, 1 or 10..14");
    if (p->n_samples < 0) return fail(QS_ERR_INVALID_ARGUMENT, "negative sample count");
    if (int64_t(p->n_samples) * int64_t(s->n) > (int64_t(1) << 32))
        return fail(QS_ERR_INVALID_ARGUMENT, "readout counter would overflow");
    std::shared_ptr<const ModelEntry> me;
    QS_CHECK(circuit_model(c, &me));
    const CircuitModel *mp = &me->model;
    CircuitModel conv;
    if (p->mode == QS_KRAUS_CONVENTIONAL_INPLACE) {
        conv = me->model;
        for (auto &ci : conv.channels) to_conventional(ci);
        mp = &conv;
    }
    const CircuitModel &m = *mp;
    QS_CHECK(flush_pending(s));
    r->sweeps = 0;
    r->gate_sweeps = 0;
    r->gate_kernel_ms = 0.0;
    r->gate_kernel_launches = 0;
    for (int i = 0; i < 6; ++i) r->gate_k_launches[i] = 0;
    r->zero_start_sweeps = 0;
    r->graph_replays = 0;
    const uint64_t chash = me->id;
    qs_traj_params q = *p;
    double tms = 0.0;
    QS_CHECK(resolve_widths(s, m, chash, *p, r->z_expect != nullptr, &q.max_fuse, &q.tile_bits, &tms));
    r->max_fuse_used = q.max_fuse;
    r->tile_bits_used = tile_bits_reported(m.n, q.tile_bits);
    r->tune_ms = tms;
    Runner run(s, m, q, *r, chash, call_traj, ref, intervals);
    const qs_status st = run.run();
    r->host_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return st;
}

// Total length of the union of intervals.
double union_length(std::vector<std::pair<double, double>> iv) {
    std::sort(iv.begin(), iv.end());
    double total = 0.0, a = 0.0, b = 0.0;
    bool open = false;
    for (const auto &x : iv) {
        if (!open || x.first > b) {
            if (open) total += b - a;
            a = x.first;
            b = x.second;
            open = true;
        } else if (x.second > b) {
            b = x.second;
        }
    }
    if (open) total += b - a;
    return total;
}

}  // namespace

qs_status qs_run_trajectories(qs_state s, const qs_circuit *c, const qs_traj_params *p,
                              qs_traj_result *r) {
    return run_trajectories_impl(s, c, p, r, p ? p->n_traj : 0, nullptr, nullptr);
}

qs_status qs_run_trajectories_concurrent(qs_state *states, int n_states, const qs_circuit *c,
                                         const qs_traj_params *p, qs_traj_result *r) {
    const auto t0 = std::chrono::steady_clock::now();
    if (!states || !c || !p || !r) return fail(QS_ERR_INVALID_ARGUMENT, "null argument");
    if (n_states < 1 || n_states > 16) return fail(QS_ERR_INVALID_ARGUMENT, "n_states outside 1..16");
    for (int j = 0; j < n_states; ++j) {
        QS_CHECK(check_handle(states[j]));
        for (int i = 0; i < j; ++i)
            if (states[i] == states[j]) return fail(QS_ERR_INVALID_ARGUMENT, "a state appears twice");
    }
    if (p->n_traj < 0) return fail(QS_ERR_INVALID_ARGUMENT, "negative trajectory count");
    const int nch = [&] {
        int k = 0;
        if (c->ops)
            for (int o = 0; o < c->n_ops; ++o) k += c->ops[o].kind == QS_OP_CHANNEL ? 1 : 0;
        return k;
    }();
    const int n = c->n_qubits;
    // the widths are chosen once (tuning on the first state if asked), so
    // every chunk runs the same plan as one state would
    qs_traj_params pr = *p;
    double tms = 0.0;
    {
        std::shared_ptr<const ModelEntry> me;
        QS_CHECK(circuit_model(c, &me));
        CircuitModel conv;
        if (p->mode == QS_KRAUS_CONVENTIONAL_INPLACE) {
            conv = me->model;
            for (auto &ci : conv.channels) to_conventional(ci);
        }
        const CircuitModel &m = p->mode == QS_KRAUS_CONVENTIONAL_INPLACE ? conv : me->model;
        QS_CHECK(flush_pending(states[0]));
        QS_CHECK(resolve_widths(states[0], m, me->id, *p, r->z_expect != nullptr, &pr.max_fuse, &pr.tile_bits, &tms));
    }
    // contiguous chunks, the first (n_traj mod n_states) one trajectory longer
    std::vector<qs_traj_params> sp(n_states, pr);
    std::vector<qs_traj_result> sr(n_states);
    int64_t start = 0;
    for (int j = 0; j < n_states; ++j) {
        const int64_t cnt = p->n_traj / n_states + (j < p->n_traj % n_states ? 1 : 0);
        sp[j].traj_offset = p->traj_offset + start;
        sp[j].n_traj = cnt;
        qs_traj_result &x = sr[j];
        std::memset(&x, 0, sizeof(x));
        x.bitstrings = r->bitstrings ? r->bitstrings + start * p->n_samples : nullptr;
        x.kraus_choices = r->kraus_choices ? r->kraus_choices + start * nch : nullptr;
        x.kraus_paths = r->kraus_paths ? r->kraus_paths + start * nch : nullptr;
        x.n_slow = r->n_slow ? r->n_slow + start : nullptr;
        x.z_expect = r->z_expect ? r->z_expect + start * n : nullptr;
        // the final state is the last trajectory's: the last non-empty chunk returns it
        const bool last = start + cnt == p->n_traj && cnt > 0;
        x.final_state = last ? r->final_state : nullptr;
        if (!last) sp[j].flags &= ~uint32_t(QS_TRAJ_RETURN_STATE);
        start += cnt;
    }
    std::vector<qs_status> status(n_states, QS_OK);
    std::vector<std::string> message(n_states);
    // with kernel timing, every stream's sweep brackets are placed on one
    // time axis (a reference event, completed before any of them starts)
    const bool timing = (p->flags & QS_TRAJ_TIME_KERNELS) != 0;
    hipEvent_t ref = nullptr;
    std::vector<std::vector<std::pair<double, double>>> iv(n_states);
    if (timing) {
        QS_HIP(states[0], hipEventCreate(&ref));
        QS_HIP(states[0], hipEventRecord(ref, states[0]->st));
        QS_HIP(states[0], hipEventSynchronize(ref));
    }
    auto work = [&](int j) {
        // a new host thread starts on device 0: work on the state's device
        if (hipSetDevice(states[j]->device) != hipSuccess) {
            status[j] = QS_ERR_DEVICE;
            message[j] = "cannot select the state's device";
            return;
        }
        status[j] = run_trajectories_impl(states[j], c, &sp[j], &sr[j], p->n_traj, ref, timing ? &iv[j] : nullptr);
        if (status[j] != QS_OK) message[j] = g_last_error;
    };
    std::vector<std::thread> pool;
    for (int j = 1; j < n_states; ++j) pool.emplace_back(work, j);
    {
        // chunk 0 runs on the calling thread, whose current device is restored
        int prev = 0;
        const bool had = hipGetDevice(&prev) == hipSuccess;
        work(0);
        if (had) (void)hipSetDevice(prev);
    }
    for (auto &t : pool) t.join();
    r->sweeps = r->gate_sweeps = r->gate_kernel_launches = r->zero_start_sweeps = 0;
    r->graph_replays = 0;
    r->gate_kernel_ms = 0.0;
    r->max_fuse_used = sr[0].max_fuse_used;
    r->tile_bits_used = sr[0].tile_bits_used;
    r->tune_ms = tms;
    for (int i = 0; i < 6; ++i) r->gate_k_launches[i] = 0;
    for (int j = 0; j < n_states; ++j) {
        r->sweeps += sr[j].sweeps;
        r->gate_sweeps += sr[j].gate_sweeps;
        r->gate_kernel_ms += sr[j].gate_kernel_ms;
        r->gate_kernel_launches += sr[j].gate_kernel_launches;
        r->zero_start_sweeps += sr[j].zero_start_sweeps;
        r->graph_replays += sr[j].graph_replays;
        for (int i = 0; i < 6; ++i) r->gate_k_launches[i] += sr[j].gate_k_launches[i];
    }
    if (timing) {
        // time during which at least one of the call's sweeps was running
        std::vector<std::pair<double, double>> all;
        for (const auto &v : iv) all.insert(all.end(), v.begin(), v.end());
        r->gate_kernel_ms = union_length(std::move(all));
        (void)hipEventDestroy(ref);
    }
    r->host_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    for (int j = 0; j < n_states; ++j)
        if (status[j] != QS_OK) return fail(status[j], message[j].c_str());
    return QS_OK;
}

qs_status qs_fusion_plan(const qs_circuit *c, int max_fuse, int32_t *n_blocks_out,
                         int32_t *block_k, int32_t *block_targets, double *block_mats,
                         int32_t *op_block) {
    if (!c || !n_blocks_out || !block_k || !block_targets || !block_mats || !op_block)
        return fail(QS_ERR_INVALID_ARGUMENT, "null argument");
    if (max_fuse < 1 || max_fuse > qs::kMaxGateQubits)
        return fail(QS_ERR_INVALID_ARGUMENT, "max_fuse outside 1..5");
    if (c->n_qubits < 1 || c->n_qubits > qs::kMaxQubits)
        return fail(QS_ERR_INVALID_ARGUMENT, "n out of range");
    CircuitModel m;
    QS_CHECK(build_model(c, m));
    if (!m.channels.empty()) return fail(QS_ERR_INVALID_ARGUMENT, "fusion plan takes gates only");
    std::vector<int> ob;
    const auto blocks = qs::fuse_greedy(m.n, m.ops, max_fuse, &ob);
    std::vector<cd> tmp(1024);
    for (size_t b = 0; b < blocks.size(); ++b) {
        block_k[b] = blocks[b].k;
        for (int j = 0; j < 5; ++j) block_targets[5 * b + j] = j < blocks[b].k ? blocks[b].q[j] : 0;
        qs::fused_matrix(blocks[b].k, blocks[b].q, blocks[b].ops, m.ops, m.gate_mat, tmp.data());
        const int D = 1 << blocks[b].k;
        double *dst = block_mats + b * 2048;
        for (int i = 0; i < 2048; ++i) dst[i] = 0.0;
        for (int i = 0; i < D * D; ++i) {
            dst[2 * i] = tmp[i].real();
            dst[2 * i + 1] = tmp[i].imag();
        }
    }
    for (size_t o = 0; o < ob.size(); ++o) op_block[o] = ob[o];
    *n_blocks_out = int32_t(blocks.size());
    return QS_OK;
}

qs_status qs_sweep_plan(const qs_circuit *c, int max_fuse, int tile_bits, int32_t *n_sweeps_out,
                        int32_t *order_out, int32_t *sweep_of_order, uint64_t *sweep_bits) {
    if (!c || !n_sweeps_out || !order_out || !sweep_of_order || !sweep_bits)
        return fail(QS_ERR_INVALID_ARGUMENT, "null argument");
    if (max_fuse < 1 || max_fuse > qs::kMaxGateQubits)
        return fail(QS_ERR_INVALID_ARGUMENT, "max_fuse outside 1..5");
    if (!(tile_bits == 0 || tile_bits == 1 || (tile_bits >= 10 && tile_bits <= qs::kMaxTileBits)))
        return fail(QS_ERR_INVALID_ARGUMENT, "tile_bits must be 0, 1 or 10..14");
    if (c->n_qubits < 1 || c->n_qubits > qs::kMaxQubits)
        return fail(QS_ERR_INVALID_ARGUMENT, "n out of range");
    CircuitModel m;
    QS_CHECK(build_model(c, m));
    const auto blocks = qs::fuse_greedy(m.n, m.ops, max_fuse);
    const int T = tile_bits == 0 ? qs::kDefaultTileBits : tile_bits;
    std::vector<qs::Sweep> sw;
    if (T >= 10 && m.n >= qs::kTileMinQubits) {
        sw = qs::group_sweeps_best(m.n, blocks, std::min(T, m.n), qs::kTileLowBits, qs::kMaxTileGates,
                                   qs::tile_mat_budget(std::min(T, m.n)), tile_slots(),
                                   plan_restarts(m.n, 1 << 20), kGroupSeed);
    } else {
        for (size_t b = 0; b < blocks.size(); ++b) {
            qs::Sweep one;
            one.blocks.push_back(int(b));
            for (int j = 0; j < blocks[b].k; ++j) one.bits.push_back(blocks[b].q[j]);
            sw.push_back(std::move(one));
        }
    }
    int i = 0;
    for (size_t u = 0; u < sw.size(); ++u) {
        uint64_t mask = 0;
        for (int q : sw[u].bits) mask |= uint64_t(1) << q;
        sweep_bits[u] = mask;
        for (int b : sw[u].blocks) {
            order_out[i] = b;
            sweep_of_order[i] = int32_t(u);
            ++i;
        }
    }
    *n_sweeps_out = int32_t(sw.size());
    return QS_OK;
}

}  // extern "C"

// --------------------------------------------------------------------------
// Batched launches: host planning.
// --------------------------------------------------------------------------

namespace {

constexpr int kBatchDefaultFuse = 3;

// Per-circuit fusion and sweep grouping of the batched launch, cached by
// circuit, fusion width and grouping restarts (a batch of the same circuits is planned
// once; only the per-trajectory draws and patched blocks are redone).
struct BatchPlanKey {
    uint64_t hash;  // model id
    int f;
    int restarts;   // of the sweep grouping (0: resident, not grouped)
    bool operator<(const BatchPlanKey &o) const {
        return std::tie(hash, f, restarts) < std::tie(o.hash, o.f, o.restarts);
    }
};
struct BatchPlanEntry {
    std::vector<qs::BatchSweep> sweeps;     // gate ranges local to the circuit
    std::vector<qs::BatchGate> gates;       // mat: offset into pool; m0, m1: into members
    std::vector<qs::BatchTileGate> tile_gates;  // the blocks with their LDS address tables
    std::vector<float2> pool;               // the default matrices of the blocks
    std::vector<qs::BatchChannel> chans;    // pbar: into pbar; unit: into fmats
    std::vector<double> pbar;
    std::vector<qs::BatchMember> members;   // src >= 0: into fmats
    std::vector<double2> fmats;             // FP64 gate and channel matrices of the members
    bool k5 = false;                        // a sweep holds a 5-qubit block
};
constexpr size_t kBatchPlanEntries = 2048;
std::mutex g_bplan_mu;
std::map<BatchPlanKey, std::shared_ptr<const BatchPlanEntry>> g_bplan_cache;
std::deque<BatchPlanKey> g_bplan_fifo;

void batch_plan_lookup(const BatchPlanKey &k, std::shared_ptr<const BatchPlanEntry> *out) {
    std::lock_guard<std::mutex> lock(g_bplan_mu);
    auto it = g_bplan_cache.find(k);
    *out = it == g_bplan_cache.end() ? nullptr : it->second;
}

void batch_plan_insert(const BatchPlanKey &k, std::shared_ptr<const BatchPlanEntry> e) {
    std::lock_guard<std::mutex> lock(g_bplan_mu);
    if (g_bplan_cache.count(k)) return;
    if (g_bplan_fifo.size() >= kBatchPlanEntries) {
        g_bplan_cache.erase(g_bplan_fifo.front());
        g_bplan_fifo.pop_front();
    }
    g_bplan_cache[k] = std::move(e);
    g_bplan_fifo.push_back(k);
}

struct BatchPlanCircuit {
    std::shared_ptr<const ModelEntry> me;
    const CircuitModel *m = nullptr;  // me->model
    std::shared_ptr<const BatchPlanEntry> plan;
    bool resident = false;
};

// Grow-only device buffers for the batched launch, one set per device; a
// call holds the lock for its duration.
struct BatchBuffers {
    std::mutex lock;
    char *prog = nullptr;
    size_t prog_cap = 0;
    float2 *slots = nullptr;
    size_t slots_cap = 0;    // bytes
    float2 *patched = nullptr;
    size_t patched_cap = 0;  // bytes
    char *host = nullptr;    // pinned staging for the program
    size_t host_cap = 0;
    // the plans' tables on the device, one after another; a plan in the map
    // finds its own in place.  Full, the area starts over (kBatchTableBytes
    // at most, unless one batch needs more).
    char *tables = nullptr;
    size_t tables_cap = 0, tables_used = 0;
    std::map<std::shared_ptr<const BatchPlanEntry>, size_t> tables_at;
};
constexpr size_t kBatchTableBytes = size_t(64) << 20;

// Where a plan's tables lie within its piece of the device area.
struct BatchTableLayout {
    size_t sweeps, gates, tile_gates, mats, chans, pbar, members, fmats, bytes;
    explicit BatchTableLayout(const BatchPlanEntry &E) {
        size_t at = 0;
        auto take = [&at](size_t len) {
            const size_t here = at;
            at += (len + 255) & ~size_t(255);
            return here;
        };
        sweeps = take(sizeof(qs::BatchSweep) * E.sweeps.size());
        gates = take(sizeof(qs::BatchGate) * E.gates.size());
        tile_gates = take(sizeof(qs::BatchTileGate) * E.tile_gates.size());
        mats = take(sizeof(float2) * E.pool.size());
        chans = take(sizeof(qs::BatchChannel) * E.chans.size());
        pbar = take(sizeof(double) * E.pbar.size());
        members = take(sizeof(qs::BatchMember) * E.members.size());
        fmats = take(sizeof(double2) * E.fmats.size());
        bytes = at + 256;  // descriptors are read two blocks ahead
    }
    void write(const BatchPlanEntry &E, char *to) const {
        auto put = [to](size_t at, const auto &v) {
            if (!v.empty()) std::memcpy(to + at, v.data(), sizeof(v[0]) * v.size());
        };
        put(sweeps, E.sweeps);
        put(gates, E.gates);
        put(tile_gates, E.tile_gates);
        put(mats, E.pool);
        put(chans, E.chans);
        put(pbar, E.pbar);
        put(members, E.members);
        put(fmats, E.fmats);
    }
};

BatchBuffers &batch_buffers() {
    static std::mutex map_lock;
    static std::map<int, BatchBuffers *> per_device;
    int dev = 0;
    (void)hipGetDevice(&dev);
    std::lock_guard<std::mutex> g(map_lock);
    BatchBuffers *&b = per_device[dev];
    if (!b) b = new BatchBuffers();
    return *b;
}

void to_float2(int D, const cd *m, float2 *out) {
    for (int i = 0; i < D * D; ++i) out[i] = make_float2(float(m[i].real()), float(m[i].imag()));
}

// The blocks in the order of `order`, cut into runs whose qubits fit a tile
// and whose staged matrices fit its budget.
std::vector<qs::Sweep> cut_sweeps(const std::vector<qs::Sweep> &order, const std::vector<qs::Block> &blocks) {
    std::vector<qs::Sweep> out;
    const uint64_t low = (uint64_t(1) << qs::kTileLowBits) - 1;
    uint64_t bits = low;
    int slots = 0;
    if (order.empty()) {  // a circuit without operations still writes |0...0>
        out.emplace_back();
        for (int q = 0; q < qs::kTileLowBits; ++q) out.back().bits.push_back(q);
    }
    for (const auto &w : order)
        for (int b : w.blocks) {
            uint64_t need = low;
            for (int j = 0; j < blocks[size_t(b)].k; ++j) need |= uint64_t(1) << blocks[size_t(b)].q[j];
            const int cost = qs::tile_mat_slots(blocks[size_t(b)].k);
            if (out.empty() || __builtin_popcountll(bits | need) > qs::kBatchTileBits ||
                slots + cost > qs::tile_mat_budget(qs::kBatchTileBits)) {
                out.emplace_back();
                bits = 0;
                slots = 0;
            }
            bits |= need;
            slots += cost;
            out.back().blocks.push_back(b);
            out.back().bits.clear();
            for (int q = 0; q < 64; ++q)
                if ((bits >> q) & 1) out.back().bits.push_back(q);
        }
    return out;
}

// Fusion, sweep grouping and default block matrices of one circuit for the
// batched launch (every channel at its most likely pick), with what the
// device needs to redo a block for other picks: the channel table and, for
// each block holding a channel, its operations with FP64 matrices.
qs_status plan_batched_circuit(const CircuitModel &m, const std::vector<const cd *> &default_mats,
                               int f, bool resident, int restarts, BatchPlanEntry &e) {
    const int n = m.n;
    std::vector<int> op_block;
    const std::vector<qs::Block> blocks = qs::fuse_greedy(n, m.ops, f, &op_block);
    if (blocks.size() > size_t(qs::kBatchMaxBlocks))
        return fail(QS_ERR_NOT_SUPPORTED, "batched circuits fuse into at most 16384 blocks");
    std::vector<qs::Sweep> sw;
    if (resident) {
        qs::Sweep one;
        for (size_t b = 0; b < blocks.size(); ++b) one.blocks.push_back(int(b));
        sw.push_back(std::move(one));
    } else {
        static const int no_budget[6] = {0, 0, 0, 0, 0, 0};
        const auto order = qs::group_sweeps_best(n, blocks, qs::kBatchOrderBits, qs::kBatchOrderLowBits, 1 << 30,
                                                 1 << 30, no_budget, restarts, kGroupSeed);
        sw = cut_sweeps(order, blocks);
    }
    std::vector<char> has_channel(blocks.size(), 0);
    for (const ChannelInfo &c : m.channels) has_channel[size_t(op_block[size_t(c.op)])] = 1;
    std::vector<int> gate_of_block(blocks.size(), -1);
    std::vector<cd> tmp(1024);
    for (const auto &w : sw) {
        qs::BatchSweep S;
        std::memset(&S, 0, sizeof(S));
        int local[64];
        for (int q = 0; q < 64; ++q) local[q] = q;
        if (!resident) {
            std::vector<char> in(n, 0);
            for (int q : w.bits) in[q] = 1;
            int cnt = int(w.bits.size());
            for (int q = 0; q < n && cnt < qs::kBatchTileBits; ++q)
                if (!in[q]) {
                    in[q] = 1;
                    ++cnt;
                }
            int i = 0;
            for (int q = 0; q < n; ++q)
                if (in[q]) {
                    S.pos[i] = q;
                    local[q] = i;
                    ++i;
                }
        }
        int lofs = 0;
        S.g0 = int(e.gates.size());
        for (int b : w.blocks) {
            const qs::Block &B = blocks[b];
            qs::BatchGate G;
            std::memset(&G, 0, sizeof(G));
            G.k = B.k;

            int lt[qs::kMaxGateQubits];
            for (int j = 0; j < B.k; ++j) lt[j] = local[B.q[j]];
            e.tile_gates.push_back(qs::batch_tile_gate(B.k, lt, lofs));
            lofs += qs::tile_mat_slots(B.k);
            e.k5 |= !resident && B.k == 5;
            qs::fused_matrix(B.k, B.q, B.ops, m.ops, default_mats, tmp.data());
            const int D = 1 << B.k;
            G.mat = int(e.pool.size());
            e.pool.resize(e.pool.size() + size_t(D) * D + (D * D) % 2);
            to_float2(D, tmp.data(), e.pool.data() + G.mat);
            G.m0 = G.m1 = int(e.members.size());
            if (has_channel[size_t(b)]) {
                for (int o : B.ops) {
                    const qs::PlanOp &op = m.ops[size_t(o)];
                    qs::BatchMember M;
                    std::memset(&M, 0, sizeof(M));
                    M.k = op.k;
                    for (int j = 0; j < op.k; ++j) M.lp[j] = int(std::find(B.q, B.q + B.k, op.q[j]) - B.q);
                    if (m.kind[size_t(o)] == QS_OP_GATE) {
                        const cd *U = m.gate_mat[size_t(o)];
                        if (!U) continue;  // left out of the product, as in the default fusion
                        M.src = int(e.fmats.size());
                        const int d = 1 << op.k;
                        for (int x = 0; x < d * d; ++x) e.fmats.push_back(make_double2(U[x].real(), U[x].imag()));
                    } else {
                        M.src = -m.channel_of_op[size_t(o)] - 1;
                    }
                    e.members.push_back(M);
                }
                G.m1 = int(e.members.size());
            }
            gate_of_block[size_t(b)] = int(e.gates.size());
            e.gates.push_back(G);
        }
        S.g1 = int(e.gates.size());
        e.sweeps.push_back(S);
    }
    for (const ChannelInfo &c : m.channels) {
        if (c.nk > 32) return fail(QS_ERR_NOT_SUPPORTED, "batched channels have at most 32 Kraus operators");
        const int D = 1 << c.k;
        qs::BatchChannel ch;
        ch.nk = c.nk;
        ch.default_pick = c.default_pick;
        ch.pbar = int32_t(e.pbar.size());
        ch.gate = gate_of_block[size_t(op_block[size_t(c.op)])];
        ch.unit = int32_t(e.fmats.size());
        ch.identity = 0;
        for (int i = 0; i < c.nk; ++i) {
            if (c.identity[size_t(i)]) ch.identity |= 1u << i;
            for (int x = 0; x < D * D; ++x) {
                const cd u = c.unit[size_t(i) * D * D + x];
                e.fmats.push_back(make_double2(u.real(), u.imag()));
            }
        }
        e.pbar.insert(e.pbar.end(), c.pbar.begin(), c.pbar.end());
        e.chans.push_back(ch);
    }
    if (e.pool.size() > size_t(1) << 28 || e.fmats.size() > size_t(1) << 28)
        return fail(QS_ERR_NOT_SUPPORTED, "batched circuit too large");
    return QS_OK;
}

}  // namespace

namespace {

// Items with at least this many samples take them straight into the caller's
// buffer when it is pinned host memory (smaller ones are not worth a
// transfer of their own).
constexpr int64_t kDirectSamples = int64_t(1) << 14;

// Whether a host pointer lies in pinned (page-locked, device-visible) host
// memory.  Pageable memory makes the query fail; its error is cleared.
bool pinned_host(const void *p) {
    if (!p) return false;
    hipPointerAttribute_t a;
    std::memset(&a, 0, sizeof(a));
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return a.type == hipMemoryTypeHost;
}

// Jobs [first, first + count) of the larger circuits run their sweeps
// together; sweep s is one launch over the first active[s] of the wave's
// parts (its jobs are sorted by sweep count).
struct BatchWave {
    int first = 0, count = 0;
    size_t part0 = 0;
    std::vector<int> active;
};

// States of a wave (1 GiB at most): every launch ends with a partly filled
// round of workgroups, so few large waves beat cache-sized ones (64 circuits
// of 12..18 qubits x 16 trajectories: 6.87 ms a batch with 128 MiB waves, 6.01
// with 256 MiB, 5.72 with all 570 MiB in one).
constexpr size_t kWaveAmps = size_t(1) << 27;
constexpr size_t kWavePatched = size_t(1) << 25;  // float2 of rebuilt matrices

void plan_waves(std::vector<qs::BatchJob> &jobs, const std::vector<qs::BatchCircuit> &circs,
                const std::vector<BatchPlanCircuit> &plans, int64_t resident_jobs, size_t patched0,
                std::vector<BatchWave> &waves, std::vector<qs::BatchPart> &parts, size_t &slot_amps,
                size_t &wide_patched, size_t &n_mptr) {
    size_t j = size_t(resident_jobs);
    while (j < jobs.size()) {
        BatchWave w;
        w.first = int(j);
        w.part0 = parts.size();
        size_t amps = 0, patched = 0, mp = 0;
        for (; j < jobs.size(); ++j) {
            qs::BatchJob &J = jobs[j];
            const qs::BatchCircuit &C = circs[size_t(J.circuit)];
            const size_t need = size_t(1) << C.n;
            const size_t pat =
                C.nch > 0 ? (plans[size_t(J.circuit)].plan->pool.size() + 63) & ~size_t(63) : 0;
            if (w.count > 0 && (amps + need > kWaveAmps || patched + pat > kWavePatched)) break;
            J.slot = int64_t(amps);
            J.mine = int64_t(patched0 + patched);
            J.mptr = int64_t(mp);
            amps += need;
            patched += pat;
            mp += size_t(C.n_gates);
            ++w.count;
        }
        // two tiles per workgroup share the staging of the sweep's matrices
        // once that leaves four rounds of workgroups (two per CU); more than
        // two make the launch's last round longer than they save (at 1 / 2 / 4
        // / 8 tiles the same batch takes 5.91, 5.66, 5.85, 6.52 ms, 512
        // trajectories of 18 qubits 7.69, 7.23, 7.29, 7.18, 1024 of 14 0.94,
        // 0.87, 0.87, 0.87; 16 of 16 qubits, 128 tiles, 0.26, 0.35, 0.54, 0.92)
        const size_t tiles = amps >> qs::kBatchTileBits;
        const int per = tiles >= 4096 ? 2 : 1;
        for (int i = 0; i < w.count; ++i) {
            const qs::BatchJob &J = jobs[size_t(w.first + i)];
            const int nt = 1 << (circs[size_t(J.circuit)].n - qs::kBatchTileBits);
            for (int t = 0; t < nt; t += per)
                parts.push_back(qs::BatchPart{w.first + i, t, std::min(per, nt - t)});
            const size_t steps = plans[size_t(J.circuit)].plan->sweeps.size();
            w.active.resize(std::max(w.active.size(), steps), 0);
            for (size_t s = 0; s < steps; ++s) w.active[s] = int(parts.size() - w.part0);
        }
        slot_amps = std::max(slot_amps, amps);
        wide_patched = std::max(wide_patched, patched);
        n_mptr = std::max(n_mptr, mp);
        waves.push_back(std::move(w));
    }
}

// `sized`: the items whose trajectory counts the plans are searched for (an
// autotuner trial runs fewer trajectories on the plans of the whole batch).
qs_status run_batched_impl(const qs_batch_item *items, const qs_batch_item *sized, int n_items,
                           const qs_batch_params *bp, int f, qs_batch_result *r) {
    const auto t0 = std::chrono::steady_clock::now();
    hipStream_t st = static_cast<hipStream_t>(bp->hip_stream);
    std::memset(r, 0, sizeof(*r));
    r->max_fuse_used = f;

    // ---- per-circuit plans (threads over circuits, cached per circuit and
    // width), then concatenated
    std::vector<BatchPlanCircuit> plans(n_items);
    std::vector<qs::BatchCircuit> circs(n_items);
    struct CircPieces {
        std::vector<double> readout;
        qs_status status = QS_OK;
        std::string error;
    };
    std::vector<CircPieces> pieces(n_items);
    for (int it = 0; it < n_items; ++it) {
        const qs_batch_item &I = items[it];
        if (!I.circuit) return fail(QS_ERR_INVALID_ARGUMENT, "null circuit");
        if (I.circuit->n_qubits < 1) return fail(QS_ERR_INVALID_ARGUMENT, "n out of range");
        if (I.circuit->n_qubits > qs::kBatchMaxQubits)
            return fail(QS_ERR_NOT_SUPPORTED, "batched circuits have at most 18 qubits");
        if (I.n_traj < 0 || I.traj_offset < 0 || I.traj_offset + I.n_traj > (int64_t(1) << 32))
            return fail(QS_ERR_INVALID_ARGUMENT, "trajectory range outside 32-bit counters");
        if (I.n_samples < 0 || I.n_samples > qs::kBatchMaxSamples)
            return fail(QS_ERR_INVALID_ARGUMENT, "n_samples outside 0..4096");
        if (I.n_samples > 0 && I.n_traj > 0 && !I.bitstrings)
            return fail(QS_ERR_INVALID_ARGUMENT, "null bitstrings");
    }
    auto plan_one = [&](int it) {
        const qs_batch_item &I = items[it];
        BatchPlanCircuit &P = plans[it];
        CircPieces &X = pieces[it];
        qs_status stt = circuit_model(I.circuit, &P.me);
        if (stt != QS_OK) {
            X.status = stt;
            X.error = g_last_error;
            return;
        }
        P.m = &P.me->model;
        for (const auto &c : P.m->channels)
            if (!c.mixture) {
                X.status = QS_ERR_NOT_SUPPORTED;
                X.error = "batched launch takes channels whose Kraus operators are all proportional to unitaries";
                return;
            }
        qs::ReadoutDesc ro;
        stt = fill_readout(P.m->n, I.p0to1, I.p1to0, ro);
        if (stt != QS_OK) {
            X.status = stt;
            X.error = g_last_error;
            return;
        }
        const int n = P.m->n;
        P.resident = n <= qs::kBatchLdsQubits;
        qs::BatchCircuit &C = circs[it];
        std::memset(&C, 0, sizeof(C));
        C.n = n;
        C.n_samples = I.n_samples;
        C.readout = -1;
        if (ro.enabled) {
            C.readout = 0;  // local; shifted when concatenated
            for (int q = 0; q < n; ++q) X.readout.push_back(ro.e0[q]);
            for (int q = 0; q < n; ++q) X.readout.push_back(ro.e1[q]);
        }
        const int restarts = P.resident ? 0 : plan_restarts(n, sized[it].n_traj);
        const BatchPlanKey bkey{P.me->id, f, restarts};
        batch_plan_lookup(bkey, &P.plan);
        if (!P.plan) {
            const int n_ops = int(P.m->ops.size());
            std::vector<const cd *> default_mats(size_t(n_ops), nullptr);
            for (int o = 0; o < n_ops; ++o) {
                if (P.m->kind[size_t(o)] == QS_OP_GATE) default_mats[size_t(o)] = P.m->gate_mat[size_t(o)];
                else {
                    const ChannelInfo &c = P.m->channels[size_t(P.m->channel_of_op[size_t(o)])];
                    default_mats[size_t(o)] = fast_pick_matrix(c, c.default_pick);
                }
            }
            auto e = std::make_shared<BatchPlanEntry>();
            const qs_status ps = plan_batched_circuit(*P.m, default_mats, f, P.resident, restarts, *e);
            if (ps != QS_OK) {
                X.status = ps;
                X.error = g_last_error;
                return;
            }
            batch_plan_insert(bkey, e);
            P.plan = std::move(e);
        }
    };
    qs::HostPool::get().run(size_t(n_items), 1, 16u, [&](size_t lo, size_t hi) {
        for (size_t it = lo; it < hi; ++it) plan_one(int(it));
    });
    for (int it = 0; it < n_items; ++it)
        if (pieces[it].status != QS_OK) return fail(pieces[it].status, pieces[it].error);

    // ---- what the call's circuits add up to
    size_t n_ro = 0;
    bool wide_k5 = false;
    int64_t max_pool = 0, total_jobs = 0, total_samples = 0, total_choices = 0;
    for (int it = 0; it < n_items; ++it) {
        const BatchPlanEntry &E = *plans[it].plan;
        qs::BatchCircuit &C = circs[it];
        C.n_gates = int(E.gates.size());
        C.nch = int(E.chans.size());
        if (C.readout >= 0) C.readout = int(n_ro);
        n_ro += pieces[it].readout.size();
        wide_k5 |= E.k5;
        if (plans[it].resident && !E.chans.empty()) max_pool = std::max<int64_t>(max_pool, int64_t(E.pool.size()));
        total_jobs += items[it].n_traj;
        total_samples += items[it].n_traj * int64_t(items[it].n_samples);
        if (items[it].kraus_choices) total_choices += items[it].n_traj * int64_t(E.chans.size());
    }

    // ---- jobs: the resident ones first, largest first (the persistent workgroups
    // finish together), then the larger ones by sweep count
    std::vector<qs::BatchJob> jobs;
    jobs.reserve(size_t(total_jobs));
    std::vector<double> cost;
    cost.reserve(size_t(total_jobs));
    int64_t blocks_applied = 0, resident_jobs = 0;
    {
        int64_t out = 0, ch = 0;
        for (int it = 0; it < n_items; ++it) {
            const qs_batch_item &I = items[it];
            const BatchPlanEntry &E = *plans[it].plan;
            const bool rec = I.kraus_choices != nullptr;
            for (int64_t t = 0; t < I.n_traj; ++t) {
                qs::BatchJob J;
                std::memset(&J, 0, sizeof(J));
                J.circuit = it;
                J.traj = uint32_t(I.traj_offset + t);
                J.circ_id = I.circuit_id;
                J.seed = I.seed;
                J.out = out + t * I.n_samples;
                J.choices = rec ? ch + t * int64_t(E.chans.size()) : -1;
                jobs.push_back(J);
                cost.push_back(double(int64_t(1) << circs[it].n) * double(E.gates.size()));
            }
            out += I.n_traj * int64_t(I.n_samples);
            if (rec) ch += I.n_traj * int64_t(E.chans.size());
            blocks_applied += I.n_traj * int64_t(E.gates.size());
            if (plans[it].resident) resident_jobs += I.n_traj;
        }
    }
    {
        std::vector<size_t> order(jobs.size());
        for (size_t j = 0; j < order.size(); ++j) order[j] = j;
        auto wide_sweeps = [&](size_t j) {
            const size_t it = size_t(jobs[j].circuit);
            return plans[it].resident ? size_t(0) : plans[it].plan->sweeps.size();
        };
        std::stable_sort(order.begin(), order.end(), [&](size_t a, size_t b) {
            const size_t sa = wide_sweeps(a), sb = wide_sweeps(b);
            if ((sa == 0) != (sb == 0)) return sa == 0;
            return sa != sb ? sa > sb : cost[a] > cost[b];
        });
        std::vector<qs::BatchJob> sorted(jobs.size());
        for (size_t j = 0; j < order.size(); ++j) sorted[j] = jobs[order[j]];
        jobs.swap(sorted);
    }
    std::vector<BatchWave> waves;
    std::vector<qs::BatchPart> parts;
    const size_t patched_stride = (size_t(max_pool) + 63) & ~size_t(63);
    const int grid = qs::batched_grid();
    const size_t resident_patched =
        resident_jobs > 0 ? std::max<size_t>(patched_stride, 64) * size_t(grid) : 0;
    size_t slot_amps = 0, wide_patched = 0, n_mptr = 0;
    plan_waves(jobs, circs, plans, resident_jobs, resident_patched, waves, parts, slot_amps, wide_patched, n_mptr);
    r->jobs = int64_t(jobs.size());
    r->resident_jobs = resident_jobs;
    r->gate_blocks = blocks_applied;
    if (jobs.empty()) {
        r->plan_seconds = r->host_seconds =
            std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        return QS_OK;
    }

    // ---- device buffers (one program allocation, one upload)
    auto align = [](size_t x) { return (x + 255) & ~size_t(255); };
    const size_t b_circ = align(sizeof(qs::BatchCircuit) * circs.size());
    const size_t b_job = align(sizeof(qs::BatchJob) * jobs.size());
    const size_t b_ro = align(sizeof(double) * std::max<size_t>(n_ro, 1));
    const size_t b_out = align(sizeof(uint64_t) * size_t(std::max<int64_t>(total_samples, 1)));
    const size_t b_choice = align(size_t(std::max<int64_t>(total_choices, 1)));
    const size_t b_part = align(sizeof(qs::BatchPart) * parts.size());
    // the call's own part, then its outputs; the circuits' tables apart
    const size_t prog_bytes = b_circ + b_job + b_ro + b_part;
    const size_t total = prog_bytes + b_out + b_choice;
    const size_t b_slots = sizeof(float2) * slot_amps;
    const size_t b_mptr = sizeof(float2 *) * n_mptr;
    const size_t b_pmat = align(sizeof(float2) * (resident_patched + wide_patched));
    const size_t b_patched = b_pmat + b_mptr;
    BatchBuffers &BB = batch_buffers();
    std::lock_guard<std::mutex> hold(BB.lock);
    hipError_t e = hipSuccess;
    auto grow_dev = [&](void **ptr, size_t *cap, size_t need, const char *what) -> qs_status {
        if (need <= *cap) return QS_OK;
        if (*ptr) (void)hipFree(*ptr);
        *ptr = nullptr;
        *cap = 0;
        size_t free_b = 0, total_b = 0;
        if ((e = hipMemGetInfo(&free_b, &total_b)) != hipSuccess)
            return fail(QS_ERR_DEVICE, std::string("hipMemGetInfo: ") + hipGetErrorString(e));
        if (free_b < need) return fail(QS_ERR_OUT_OF_MEMORY, std::string("batched ") + what + " do not fit");
        if (hipMalloc(ptr, need) != hipSuccess) {
            (void)hipGetLastError();
            return fail(QS_ERR_OUT_OF_MEMORY, std::string("allocating batched ") + what + " failed");
        }
        *cap = need;
        return QS_OK;
    };
    QS_CHECK(grow_dev(reinterpret_cast<void **>(&BB.prog), &BB.prog_cap, b_out + b_choice, "output buffers"));
    QS_CHECK(grow_dev(reinterpret_cast<void **>(&BB.slots), &BB.slots_cap, b_slots, "state slots"));
    QS_CHECK(grow_dev(reinterpret_cast<void **>(&BB.patched), &BB.patched_cap, b_patched, "patched matrices"));
    // the plans whose tables are not on the device yet
    std::vector<std::pair<const BatchPlanEntry *, size_t>> fresh;  // and where they go
    size_t fresh_bytes = 0, fresh_at = 0;
    auto miss = [&](bool all) {
        fresh.clear();
        fresh_bytes = 0;
        fresh_at = BB.tables_used;
        std::map<std::shared_ptr<const BatchPlanEntry>, size_t> add;
        for (int it = 0; it < n_items; ++it) {
            const auto &P = plans[it].plan;
            if ((!all && BB.tables_at.count(P)) || add.count(P)) continue;
            add[P] = fresh_at + fresh_bytes;
            fresh.emplace_back(P.get(), fresh_bytes);
            fresh_bytes += BatchTableLayout(*P).bytes;
        }
        return add;
    };
    auto added = miss(false);
    // (the call's own part is staged behind them, in the same copy)
    if (fresh_at + fresh_bytes + prog_bytes > BB.tables_cap) {
        // start over, in a larger area while it may grow (no launch reads the
        // old one: every call ends with its stream idle)
        BB.tables_at.clear();
        BB.tables_used = 0;
        added = miss(true);
        const size_t need = fresh_bytes + prog_bytes;
        if (need > BB.tables_cap || BB.tables_cap < kBatchTableBytes)
            QS_CHECK(grow_dev(reinterpret_cast<void **>(&BB.tables), &BB.tables_cap,
                              std::max(need, std::min(kBatchTableBytes, std::max(2 * BB.tables_cap, 4 * need))),
                              "circuit tables"));
    }
    for (int it = 0; it < n_items; ++it) {
        const auto &P = plans[it].plan;
        const auto in = added.find(P);
        const char *base = BB.tables + (in != added.end() ? in->second : BB.tables_at[P]);
        const BatchTableLayout L(*P);
        qs::BatchCircuit &C = circs[it];
        C.sweeps = reinterpret_cast<const qs::BatchSweep *>(base + L.sweeps);
        C.gates = reinterpret_cast<const qs::BatchGate *>(base + L.gates);
        C.tile_gates = reinterpret_cast<const qs::BatchTileGate *>(base + L.tile_gates);
        C.mats = reinterpret_cast<const float2 *>(base + L.mats);
        C.chans = reinterpret_cast<const qs::BatchChannel *>(base + L.chans);
        C.pbar = reinterpret_cast<const double *>(base + L.pbar);
        C.members = reinterpret_cast<const qs::BatchMember *>(base + L.members);
        C.fmats = reinterpret_cast<const double2 *>(base + L.fmats);
    }
    const size_t host_bytes = total + fresh_bytes;
    if (host_bytes > BB.host_cap) {
        if (BB.host) (void)hipHostFree(BB.host);
        BB.host = nullptr;
        BB.host_cap = 0;
        if (hipHostMalloc(reinterpret_cast<void **>(&BB.host), host_bytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            return fail(QS_ERR_OUT_OF_MEMORY, "allocating pinned staging failed");
        }
        BB.host_cap = host_bytes;
    }
    char *fresh_host = BB.host;
    char *hostp = BB.host + fresh_bytes;
    char *dbuf = BB.tables + fresh_at + fresh_bytes;
    char *dout = BB.prog, *hout = hostp + prog_bytes;
    // the program, written straight into the pinned staging
    const size_t o_circ = 0, o_job = o_circ + b_circ, o_ro = o_job + b_job, o_part = o_ro + b_ro,
                 o_out = 0, o_choice = o_out + b_out;
    std::memcpy(hostp + o_circ, circs.data(), sizeof(qs::BatchCircuit) * circs.size());
    std::memcpy(hostp + o_job, jobs.data(), sizeof(qs::BatchJob) * jobs.size());
    if (!parts.empty()) std::memcpy(hostp + o_part, parts.data(), sizeof(qs::BatchPart) * parts.size());
    for (int it = 0; it < n_items; ++it)
        if (circs[it].readout >= 0)
            std::memcpy(reinterpret_cast<double *>(hostp + o_ro) + circs[it].readout, pieces[it].readout.data(),
                        sizeof(double) * pieces[it].readout.size());
    qs::HostPool::get().run(fresh.size(), 4, 16u, [&](size_t lo, size_t hi) {
        for (size_t i = lo; i < hi; ++i)
            BatchTableLayout(*fresh[i].first).write(*fresh[i].first, fresh_host + fresh[i].second);
    });
    const auto t_plan = std::chrono::steady_clock::now();
    r->plan_seconds = std::chrono::duration<double>(t_plan - t0).count();
    std::vector<char> direct(size_t(n_items), 0);
    for (int it = 0; it < n_items; ++it)
        direct[size_t(it)] = items[it].n_traj * int64_t(items[it].n_samples) >= kDirectSamples &&
                             pinned_host(items[it].bitstrings);
    qs_status status = QS_OK;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    do {
        if ((e = hipMemcpyAsync(BB.tables + fresh_at, fresh_host, fresh_bytes + prog_bytes, hipMemcpyHostToDevice,
                                st)) != hipSuccess)
            break;
        qs::BatchArgs A;
        A.circs = reinterpret_cast<const qs::BatchCircuit *>(dbuf + o_circ);
        A.jobs = reinterpret_cast<const qs::BatchJob *>(dbuf + o_job);
        A.readout = reinterpret_cast<const double *>(dbuf + o_ro);
        A.patched = BB.patched;
        A.patched_stride = int64_t(patched_stride);
        A.choices = reinterpret_cast<int8_t *>(dout + o_choice);
        A.slots = b_slots ? BB.slots : nullptr;
        A.mptr = reinterpret_cast<const float2 **>(reinterpret_cast<char *>(BB.patched) + b_pmat);
        A.out = reinterpret_cast<uint64_t *>(dout + o_out);
        A.n_jobs = int(resident_jobs);
        const auto *dparts = reinterpret_cast<const qs::BatchPart *>(dbuf + o_part);
        const bool timing = (bp->flags & QS_TRAJ_TIME_KERNELS) != 0;
        if (timing) {
            if ((e = hipEventCreate(&ev0)) != hipSuccess) break;
            if ((e = hipEventCreate(&ev1)) != hipSuccess) break;
            if ((e = hipEventRecord(ev0, st)) != hipSuccess) break;
        }
        for (const BatchWave &w : waves) {
            if ((e = qs::launch_batch_prepare(A, w.first, w.count, st)) != hipSuccess) break;
            for (size_t s = 0; s < w.active.size() && e == hipSuccess; ++s)
                e = qs::launch_batch_sweep(A, dparts + w.part0, w.active[s], int(s), wide_k5, st);
            if (e != hipSuccess) break;
            if ((e = qs::launch_batch_sample(A, w.first, w.count, st)) != hipSuccess) break;
        }
        if (e != hipSuccess) break;
        if (resident_jobs > 0 &&
            (e = qs::launch_batched(A, int(std::min<int64_t>(grid, resident_jobs)), st)) != hipSuccess)
            break;
        if (timing && (e = hipEventRecord(ev1, st)) != hipSuccess) break;
        // samples come straight into a caller's buffer that is pinned host
        // memory (one transfer, no staging copy) when the item has many;
        // the rest, and the picks, into the pinned staging (its program part
        // has been sent)
        bool staged = false;
        {
            int64_t ob = 0;
            for (int it = 0; it < n_items && e == hipSuccess; ++it) {
                const int64_t cnt = items[it].n_traj * int64_t(items[it].n_samples);
                if (cnt > 0 && direct[size_t(it)])
                    e = hipMemcpyAsync(items[it].bitstrings, dout + o_out + sizeof(uint64_t) * size_t(ob),
                                       sizeof(uint64_t) * size_t(cnt), hipMemcpyDeviceToHost, st);
                else if (cnt > 0)
                    staged = true;
                ob += cnt;
            }
            if (e != hipSuccess) break;
        }
        if (staged &&
            (e = hipMemcpyAsync(hout + o_out, dout + o_out, sizeof(uint64_t) * size_t(total_samples),
                                hipMemcpyDeviceToHost, st)) != hipSuccess)
            break;
        if (total_choices > 0 &&
            (e = hipMemcpyAsync(hout + o_choice, dout + o_choice, size_t(total_choices), hipMemcpyDeviceToHost,
                                st)) != hipSuccess)
            break;
        if ((e = hipStreamSynchronize(st)) != hipSuccess) break;
        BB.tables_at.insert(added.begin(), added.end());
        BB.tables_used += fresh_bytes;
        if (timing) {
            float ms = 0.f;
            if ((e = hipEventElapsedTime(&ms, ev0, ev1)) != hipSuccess) break;
            r->kernel_ms = ms;
        }
    } while (false);
    if (e != hipSuccess)
        status = fail(QS_ERR_DEVICE, std::string("batched launch: ") + hipGetErrorString(e));
    (void)hipStreamSynchronize(st);
    if (ev0) (void)hipEventDestroy(ev0);
    if (ev1) (void)hipEventDestroy(ev1);
    if (status != QS_OK) return status;
    {
        const uint64_t *out = reinterpret_cast<const uint64_t *>(hout + o_out);
        const int8_t *chs = reinterpret_cast<const int8_t *>(hout + o_choice);
        int64_t ob = 0, cb = 0;
        for (int it = 0; it < n_items; ++it) {
            const int64_t cnt = items[it].n_traj * int64_t(items[it].n_samples);
            if (cnt > 0 && !direct[size_t(it)])
                std::memcpy(items[it].bitstrings, out + ob, sizeof(uint64_t) * size_t(cnt));
            ob += cnt;
            if (items[it].kraus_choices) {
                const int64_t nc = items[it].n_traj * int64_t(plans[it].plan->chans.size());
                if (nc > 0) std::memcpy(items[it].kraus_choices, chs + cb, size_t(nc));
                cb += nc;
            }
        }
    }
    r->host_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return QS_OK;
}

// Batched autotuning (Section 3.2's fusion-width choice, measured): every
// candidate width runs the batch cut to at most two trajectories per circuit,
// timed whole (host planning of the patched blocks, upload and the launch:
// a wider fusion shortens the kernel but lengthens the planning), and the
// fastest is kept, cached per batch of circuits for the life of the process.
std::mutex g_btune_mu;
std::map<std::pair<uint64_t, int>, int> g_btune_cache;

}  // namespace

extern "C" qs_status qs_run_batched(const qs_batch_item *items, int n_items,
                                    const qs_batch_params *bp, qs_batch_result *r) {
    if (!items || n_items < 0 || !bp || !r) return fail(QS_ERR_INVALID_ARGUMENT, "null argument");
    if (bp->max_fuse < 0 || bp->max_fuse > qs::kMaxGateQubits)
        return fail(QS_ERR_INVALID_ARGUMENT, "max_fuse outside 0..5");
    if (bp->max_fuse > 0) return run_batched_impl(items, items, n_items, bp, bp->max_fuse, r);
    for (int it = 0; it < n_items; ++it)
        if (!items[it].circuit || !items[it].circuit->ops || !items[it].circuit->mat_pool ||
            items[it].circuit->n_ops < 0 || items[it].circuit->pool_len < 0)
            return fail(QS_ERR_INVALID_ARGUMENT, "null circuit");
    uint64_t h = 1469598103934665603ull;
    for (int it = 0; it < n_items; ++it) h = (h ^ circuit_hash(items[it].circuit)) * 1099511628211ull;
    const auto key = std::make_pair(h, n_items);
    const auto t0 = std::chrono::steady_clock::now();
    int f = kBatchDefaultFuse;
    double tune_ms = 0.0;
    {
        std::lock_guard<std::mutex> lock(g_btune_mu);
        auto found = g_btune_cache.find(key);
        if (found != g_btune_cache.end()) {
            f = found->second;
        } else {
            std::vector<qs_batch_item> trial(items, items + n_items);
            size_t outs = 0;
            for (auto &I : trial) {
                I.n_traj = std::min<int64_t>(I.n_traj, 2);
                outs += size_t(I.n_traj) * size_t(std::max(I.n_samples, 0));
                I.kraus_choices = nullptr;
            }
            std::vector<uint64_t> scratch_bits(std::max<size_t>(outs, 1));
            size_t pos = 0;
            for (auto &I : trial) {
                I.bitstrings = scratch_bits.data() + pos;
                pos += size_t(I.n_traj) * size_t(std::max(I.n_samples, 0));
            }
            qs_batch_params tp = *bp;
            tp.flags &= ~uint32_t(QS_TRAJ_TIME_KERNELS);
            double best = 1e300, t_default = -1.0;
            for (int cand : {2, 3, 4, 5}) {
                qs_batch_result tr;
                QS_CHECK(run_batched_impl(trial.data(), items, n_items, &tp, cand, &tr));
                if (cand == kBatchDefaultFuse) t_default = tr.host_seconds;
                if (tr.host_seconds < best) {
                    best = tr.host_seconds;
                    f = cand;
                }
            }
            if (t_default > 0.0 && best > (1.0 - kTuneMargin) * t_default) f = kBatchDefaultFuse;
            g_btune_cache[key] = f;
            tune_ms = 1e3 * std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
        }
    }
    const qs_status st = run_batched_impl(items, items, n_items, bp, f, r);
    r->tune_ms = tune_ms;
    return st;
}
