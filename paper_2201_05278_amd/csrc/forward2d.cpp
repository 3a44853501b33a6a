// 2D constant-density time loop in launches of several steps.
//
// The caller's scratch holds two more wavefields (a launch reads one pair of
// levels and writes the other), two sets of the levels between them (the
// receivers of a launch's levels are recorded by the next launch) and the
// injected values of every step.  The steps divide into an even number of
// launches of two steps at least, so that the last launch writes the caller's
// own pair; up to three steps before them run singly where the count does not
// divide so.
#include <algorithm>
#include <limits>
#include <type_traits>
#include <vector>

#include "device64.h"
#include "forward2d.h"
#include "runtime.h"

namespace sw {

namespace {

constexpr int kMaxInjected = 512;       // unique source nodes whose values a tile keeps in LDS
constexpr int64_t kAlign = 256;

int64_t align_up(int64_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

int value_bytes(const sw_plan *p) { return p->prob.dtype == SW_F64 ? 8 : 4; }

// Byte offsets in the scratch: buffer k (0, 1: the second pair; from 2 on the
// levels between, `between` of them per set), then the injected values.
struct ScratchMap {
    int between;
    int64_t field, inj, total;
    ScratchMap(const sw_plan *p, int steps, int nsteps, bool levels)
    {
        between = levels || p->rec.count ? std::max(0, steps - 2) : 0;
        field = align_up(p->field_elems * value_bytes(p));
        inj = field * (2 + 2 * between);
        total = inj + align_up(int64_t(nsteps) * int64_t(p->src.unode.size()) * value_bytes(p));
    }
};

template <typename T>
bool wants_levels(const Run2D<T> &io)
{
    return (io.snaps && io.saving_stride > 0) || io.ckpt;
}

// Launches for n steps of at most T each, an even number of launches of two
// steps at least; 0 where there is none.
int launches_for(int n, int T)
{
    const int L = 2 * ((n + 2 * T - 1) / (2 * T));
    return L > 0 && n >= 2 * L ? L : 0;
}

template <typename T>
struct Points {
    const int32_t *ptr, *uptr, *uent, *pid;
    const int64_t *node, *unode;
    const T *coef_a, *wscaled;
};

template <typename T>
Points<T> points_of(const WorkspaceMap::Pts &o, void *ws)
{
    return {at<int32_t>(ws, o.ptr),   at<int32_t>(ws, o.uptr),  at<int32_t>(ws, o.uent), at<int32_t>(ws, o.pid),
            at<int64_t>(ws, o.node),  at<int64_t>(ws, o.unode), at<T>(ws, o.coef_a),     at<T>(ws, o.wscaled)};
}

int pow2_group(int n)
{
    int g = 1;
    while (g < n && g < 64) g *= 2;
    return g;
}

}  // namespace

Multi2DChoice multi2d_choice(const sw_plan *p)
{
    if (p->ndim != 2 || p->prob.scheme != SW_CONST || !library_picks(p, MODE_FWD) || p->src.unode.size() > size_t(kMaxInjected) ||
        p->field_elems > std::numeric_limits<int32_t>::max())   // 32-bit element offsets
        return {};
    if (p->pin[0].tile >= 0) return {p->pin[0].extent, p->pin[0].tile};
    uint64_t v = p->choice[0].load(std::memory_order_relaxed);
    if (!v) {
        const Multi2DChoice c = choose_multi2d(p->r, value_bytes(p), p->dims[0], p->dims[2], compute_units(p));
        v = Choice::pack(c.steps, c.tile);
        p->choice[0].store(v, std::memory_order_relaxed);
    }
    return {Choice::first(v), Choice::second(v)};
}

int64_t multi2d_scratch_bytes(const sw_plan *p, int nsteps, bool levels)
{
    const Multi2DChoice c = multi2d_choice(p);
    return c.steps ? ScratchMap(p, c.steps, nsteps, levels).total : 0;
}

// Steps that run singly before the others divide into launches (-1: none do).
static int singles_of(int nsteps, int steps)
{
    for (int r = 0; r <= 3; ++r)
        if (launches_for(nsteps - r, steps)) return r;
    return -1;
}

// Checkpoints of a plan with mirror sides hold the ghosts that the single-step
// kernels leave in the halo.
static bool checkpoints_need_singles(const sw_plan *p) { return p->mirror; }

bool multi2d_divides(const sw_plan *p, int nsteps, bool ckpt)
{
    const Multi2DChoice c = multi2d_choice(p);
    return c.steps && !(ckpt && checkpoints_need_singles(p)) && singles_of(nsteps, c.steps) >= 0;
}

template <typename T>
int multi2d_singles(const sw_plan *p, const Run2D<T> &io, const void *scratch, int64_t bytes)
{
    const Multi2DChoice c = multi2d_choice(p);
    if (!c.steps || !scratch || bytes < ScratchMap(p, c.steps, io.nsteps_run, wants_levels(io)).total) return -1;
    if (io.ckpt && checkpoints_need_singles(p)) return -1;
    // the kernels read and write whole 16-byte vectors
    for (const void *q : {static_cast<const void *>(io.field[0]), static_cast<const void *>(io.field[1]), scratch})
        if (reinterpret_cast<uintptr_t>(q) % 16) return -1;
    return singles_of(io.nsteps_run, c.steps);
}

template <typename T>
sw_status enqueue_multi2d(const sw_plan *p, const Run2D<T> &io, int singles, void *scratch, hipStream_t s)
{
    constexpr bool f64 = std::is_same_v<T, double>;
    const Multi2DChoice choice = multi2d_choice(p);
    const Multi2DTile tile = multi2d_tile(choice.tile, int(sizeof(T)));
    const ScratchMap map(p, choice.steps, io.nsteps_run, wants_levels(io));
    char *base = static_cast<char *>(scratch);
    auto buffer = [&](int k) { return reinterpret_cast<T *>(base + map.field * k); };
    T *inj = reinterpret_cast<T *>(base + map.inj);
    void *ws = io.workspace;
    const int total = io.nsteps_run - singles, L = launches_for(total, choice.steps);
    const int n0 = io.step0 + singles;
    const Points<T> src = points_of<T>(p->ws.src, ws), rec = points_of<T>(p->ws.rec, ws);
    const int nuniq = int(p->src.unode.size()), nrec = p->rec.count;

    Multi2DParams<T> P{};
    P.g = make_geom(p);
    P.K = at<T>(ws, p->ws.model_k);
    P.damp = at<typename Pair<T>::type>(ws, p->ws.damp);
    const double h2z = p->hh[0] * p->hh[0], h2y = p->hh[2] * p->hh[2];
    P.c0 = T(p->v2[0] / h2z + p->v2[0] / h2y);
    for (int j = 1; j <= p->r; ++j) {
        P.cz[j] = T(p->v2[j] / h2z);
        P.cy[j] = T(p->v2[j] / h2y);
    }
    for (int k = 0; k < 2; ++k) {
        P.bcz[k] = p->bcm[0][k];
        P.bcy[k] = p->bcm[2][k];
    }
    P.unode = src.unode;
    P.nuniq = nuniq;
    P.box[0] = P.box[2] = 1 << 30;
    P.box[1] = P.box[3] = -1;
    for (const int64_t e : p->src.unode) {
        const int z = int((e - p->origin) / p->pad[2]), y = int((e - p->origin) % p->pad[2]);
        P.box[0] = std::min(P.box[0], z);
        P.box[1] = std::max(P.box[1], z);
        P.box[2] = std::min(P.box[2], y);
        P.box[3] = std::max(P.box[3], y);
    }
    P.ptr = rec.ptr;
    P.node = rec.node;
    P.wscaled = rec.wscaled;
    P.count = nrec;
    P.group = pow2_group(p->rec.max_per_point);
    if (nuniq) {
        const InjectTable<T> t{src.uptr, src.uent, src.pid, src.coef_a, nuniq, p->src.count, p->src.max_per_node};
        SW_HIP(launch_inject_all<T>(t, io.wavelet + size_t(n0) * p->src.count, total, inj, s));
    }
    const bool snaps = io.snaps && io.saving_stride > 0, ckpts = io.ckpt != nullptr;
    // whole buffers are copied into checkpoints, and their halo stays zero
    if (ckpts)
        for (int k = 0; k < 2 + 2 * map.between; ++k) {
            if constexpr (f64) SW_HIP(launch_fill64(buffer(k), p->field_elems, s));
            else SW_HIP(launch_fill(buffer(k), p->field_elems, 0.0f, s));
        }

    const T *cur = io.field[singles % 2], *prv = io.field[(singles + 1) % 2];
    int n = n0, recorded = n0;                  // first step of the launch; of the levels not recorded yet
    for (int j = 0; j < L; ++j) {
        const int nt = total / L + (j < total % L ? 1 : 0);
        const int last = n + nt - io.step0;     // steps done after the launch
        P.cur = cur;
        P.prv = prv;
        P.nt = nt;
        for (int k = 0; k < kMulti2DMax; ++k) P.out[k] = nullptr;
        // odd launches write the caller's pair, even ones the scratch's
        P.out[nt - 1] = j % 2 ? io.field[last % 2] : buffer(0);
        P.out[nt - 2] = j % 2 ? io.field[(last + 1) % 2] : buffer(1);
        if (nrec || snaps || ckpts)
            for (int k = 0; k < nt - 2; ++k) P.out[k] = buffer(2 + (j % 2) * map.between + k);
        P.inj = inj + size_t(n - n0) * nuniq;
        P.tz = tile.ez - 2 * p->r * nt;
        P.ty = tile.ey - 2 * multi2d_pad_y(p->r * nt, int(sizeof(T)));
        P.ntz = (p->dims[0] + P.tz - 1) / P.tz;
        P.nty = (p->dims[2] + P.ty - 1) / P.ty;
        P.rout = io.traces + size_t(recorded) * nrec;
        SW_HIP(launch_multi2d<T>(p->r, choice.tile, P, s));
        // this launch's levels: recorded by the next one, or after the loop
        P.rnt = nrec ? nt : 0;
        for (int k = 0; k < nt; ++k) P.rlev[k] = P.out[k];
        recorded = n;
        for (int k = 0; k < nt; ++k) {
            const int done = n + k + 1;         // out[k] = p^{done}
            if (snaps && done % io.saving_stride == 0) {
                T *slot = io.snaps + size_t(done / io.saving_stride - 1) * p->grid_nodes;
                if constexpr (f64) SW_HIP(launch_snapshot64(P.g, P.out[k], slot, s));
                else SW_HIP(launch_snapshot(P.g, P.out[k], slot, s));
            }
            if constexpr (!f64)
                if (ckpts && (n + k) % io.ckpt_every == 0) {
                    T *slot = io.ckpt + size_t((n + k) / io.ckpt_every) * 2 * p->field_elems;
                    SW_HIP(launch_copy(slot, k ? P.out[k - 1] : cur, p->field_elems, s));
                    SW_HIP(launch_copy(slot + p->field_elems, k == 0 ? prv : k == 1 ? cur : P.out[k - 2], p->field_elems, s));
                }
        }
        prv = P.out[nt - 2];
        cur = P.out[nt - 1];
        n += nt;
    }
    if (nrec) {
        P.ntz = 0;                              // no tiles: the recording blocks alone
        P.rout = io.traces + size_t(recorded) * nrec;
        SW_HIP(launch_multi2d<T>(p->r, choice.tile, P, s));
    }
    return SW_OK;
}

template int multi2d_singles<float>(const sw_plan *, const Run2D<float> &, const void *, int64_t);
template int multi2d_singles<double>(const sw_plan *, const Run2D<double> &, const void *, int64_t);
template sw_status enqueue_multi2d<float>(const sw_plan *, const Run2D<float> &, int, void *, hipStream_t);
template sw_status enqueue_multi2d<double>(const sw_plan *, const Run2D<double> &, int, void *, hipStream_t);

}  // namespace sw
