// Minimum-cost paths on the product of a transition system and a runtime
// monitor (Sec. 3.2): product vertices are (v, q), and a transition e = (u,
// v) of cost C(e) joins (u, q) to (v, q') when the monitor moves from q to q'
// on the label of e.  A monitor with no move for a label has met a bad
// prefix, so that product edge is absent.
//
// Bellman-Ford on the device: a sweep relaxes the (edge, state) pairs of every
// edge whose source vertex came nearer in the sweep before, with a 64-bit
// atomic minimum of (distance << 32 | product edge id), until a sweep brings
// no vertex nearer.  Values only decrease and each is the cost of a real
// path, and every edge is relaxed with its source's final distance, so the
// fixpoint holds the shortest distances, and in the low word the smallest
// product edge id among the edges on a shortest path into the vertex.  Costs
// are at least 1, so predecessors always have a smaller distance and the
// predecessor graph is a tree.  A graph with n product vertices needs at most
// n sweeps (each kernel ends; the host loop is bounded).
//
// A sweep reads 13 bytes of every edge and its source's mark and distances;
// only the few edges that leave a changed vertex read more.  What a call costs
// beyond that is launches and waits, so the host does not wait between sweeps: it keeps
// kAhead of them enqueued and reads in pinned memory, where each sweep reports
// on the one before, whether that one changed anything.  The sweep after the
// first that did not writes the outputs, the ones after it do nothing.
//
// 568,958 transitions, 2 states: 135 us per call in 5 sweeps of up to 16 looks
// (k_plan_sweep), 140 with 8, 154 with 4 and 175 with one, in 16 sweeps; 256
// when every sweep relaxed every reached edge and the host waited for each
// group of four.  Bound by the chain of the path's hops: source distance,
// target distance, atomic minimum, about 1 us each.  An atomic for every
// candidate instead of the check against the target's distance, which may be
// old: 360-460 us, as the sinks' atomics go one by one.  Changed vertices as
// bits set by atomics took up to 37 us in one sweep.  Random graphs: kLargeEdges.
#include <algorithm>
#include <type_traits>

#include "lbl_internal.h"

namespace lbl {
namespace {

constexpr uint32_t kInf = 0xFFFFFFFFu;
constexpr uint64_t kNone = ~0ull;
constexpr uint32_t kAhead = 4;    // sweeps enqueued beyond the last one reported on
constexpr uint32_t kReports = 64; // report slots, used in turn (more than kAhead)
constexpr uint32_t kMaxDelta = 8u << 8;
// Edges from which k_plan_sweep's LARGE form runs.  Ms per call of random graphs
// without and with it (and when every sweep relaxed every reached edge):
// vertices x edges x states, unsorted 1e5 x 1e6 x 2 1.72, 1.64 (1.83); 1e6 x 4e6 x
// 2 6.28, 4.49 (5.88); 2e6 x 6e6 x 1 8.45, 5.29 (6.52); by source 1e5 x 1e6 x 2
// 1.41, 1.21 (1.35); 1e6 x 2e6 x 1 4.58, 3.61 (3.92); 1e6 x 4e6 x 2 4.54, 3.27
// (3.79).  Below: 4e4 edges of 2e4 vertices 0.26, 0.29; roadmaps of 122,358 and
// 151,916 transitions, 8 states, 0.154, 0.160 and 0.183, 0.189.
constexpr uint64_t kLargeEdges = 3u << 18;

struct Delta {
    uint8_t move[kMaxDelta];
};

// What the kernels of one call share.
struct PlanArgs {
    const uint32_t *src, *dst, *cost;
    uint64_t n_vertices, n_edges, start;
    uint32_t n_props, n_states;
    uint64_t *best;       // [n_vertices * n_states]
    // byte per vertex (set by plain stores: bits would need atomics on the few
    // words that a frontier shares), in dwords: sweep k reads [k % 3], sets
    // [(k + 1) % 3], clears [(k + 2) % 3]
    uint32_t *near[3];
    uint32_t near_words;
    uint8_t *delta;       // the monitor's moves
    uint8_t *sigma;       // [n_edges] labels as bit sets
    uint32_t *changed;    // [4] whether sweep k brought a vertex nearer: [k % 4]
    uint64_t *report;     // pinned: [kReports] of sweep k: 2 (k + 1) + changed; [kReports]: an edge is invalid
    uint32_t *dist, *pred;
};

__device__ __forceinline__ void to_host(uint64_t *p, uint64_t v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

__device__ __forceinline__ bool edge_ok(const PlanArgs &p, uint32_t u, uint32_t v, uint32_t c)
{
    return u < p.n_vertices && v < p.n_vertices && c != 0;
}

__global__ void __launch_bounds__(256) k_plan_init(PlanArgs p, Delta delta, uint32_t n_delta,
                                                   const uint8_t *__restrict__ L, uint32_t l_stride)
{
    const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (uint64_t)gridDim.x * blockDim.x;
    const uint64_t n = p.n_vertices * p.n_states;
    const uint32_t v0 = (uint32_t)(p.start / p.n_states);
    for (uint64_t i = i0; i < n; i += step) p.best[i] = i == p.start ? (uint64_t)kInf : kNone;  // start: distance 0, no predecessor
    for (uint64_t i = i0; i < p.near_words; i += step) {
        p.near[0][i] = i == v0 / 4 ? 1u << (8 * (v0 % 4)) : 0u;
        p.near[1][i] = 0;
        p.near[2][i] = 0;
    }
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i < n_delta; i += blockDim.x) p.delta[i] = delta.move[i];
        if (threadIdx.x < 4) p.changed[threadIdx.x] = 0;
    }
    bool bad = false;
    for (uint64_t e = i0; e < p.n_edges; e += step) {
        bad = bad || !edge_ok(p, p.src[e], p.dst[e], p.cost[e]);
        uint32_t sigma = 0;  // the label as a proposition bit set
        for (uint32_t q = 0; q < p.n_props; ++q) sigma |= (L[e * l_stride + q] != 0 ? 1u : 0u) << q;
        p.sigma[e] = (uint8_t)sigma;
    }
    if (bad) to_host(p.report + kReports, 1);
}

// best[to] = min(best[to], cand).  Where many lanes have the same target (the
// sink vertices of a roadmap end thousands of edges, and atomics on one
// address go one by one), their minimum is formed in the wavefront first.
__device__ __forceinline__ void best_min(uint64_t *best, uint64_t to, uint64_t cand)
{
    const uint64_t here = __ballot(true);
    const int lead = __builtin_ctzll(here);
    const uint64_t t0 = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)to) |
                        ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(to >> 32)) << 32);
    const uint64_t same = __ballot(to == t0);
    if (__popcll(same) >= 8) {
        if (to == t0) {
            for (uint64_t left = same & (same - 1ull); left; left &= left - 1ull) {
                const int l = __builtin_ctzll(left);
                const uint64_t c = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)cand, l) |
                                   ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(cand >> 32), l) << 32);
                cand = c < cand ? c : cand;
            }
            if ((int)(threadIdx.x & 63) != lead) return;
        }
    }
    atomicMin(reinterpret_cast<unsigned long long *>(best + to), (unsigned long long)cand);
}

// Sweep k, for monitors of at most S states.  A sweep is a chain of loads that
// wait for each other, so as many as can go together do: the edge's four
// fields; then its source's flag and distances; then the distances its
// candidates would replace.  Whether a candidate brings its vertex nearer is
// judged by the value read, which may be older and larger than the current
// one (the vertex is then relaxed once more, to no effect), so nothing waits
// for the atomic minimum.
//
// A vertex that comes nearer is relaxed onward in the next sweep, or in this
// one: a lane looks at its edge's source up to most_looks times and relaxes the
// edge again when another workgroup has brought the source nearer meanwhile.
// What it misses the next sweep does (the source is marked for it), so looks
// change the number of sweeps, not the result, and none waits for anything.
// Looks cost about 1 us each where the sources of a wavefront's edges share a
// few cache lines (edges stored by source vertex) and far more where they
// don't: such wavefronts look once.
//
// LARGE (more than kLargeEdges): the edges take several turns on the chip and
// a sweep is bound by its accesses, not by the chain.  Wavefronts whose sources lie
// far apart read the rest only for edges of marked sources, a vertex that was
// marked earlier in this sweep counts as marked (its edges are relaxed now and,
// to no effect, in the next), and there are fewer looks.
template <int S, bool LARGE>
__global__ void __launch_bounds__(256) k_plan_sweep(PlanArgs p, uint64_t k, uint32_t most_looks)
{
    __shared__ uint8_t moves[S << 8];
    const uint64_t i0 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (uint64_t)gridDim.x * blockDim.x;
    const bool ended = k > 0 && p.changed[(k + 3) % 4] == 0;  // the sweep before changed nothing
    if (i0 == 0) {
        if (k > 0) to_host(p.report + (k - 1) % kReports, 2 * k + (ended ? 0 : 1));
        p.changed[(k + 1) % 4] = 0;
    }
    if (ended) {
        // the first sweep after the fixpoint writes the outputs
        if (k == 1 || p.changed[(k + 2) % 4] != 0)
            for (uint64_t i = i0; i < p.n_vertices * p.n_states; i += step) {
                const uint64_t b = p.best[i];
                p.dist[i] = (uint32_t)(b >> 32);
                p.pred[i] = (uint32_t)b;
            }
        return;
    }
    const uint8_t *now = reinterpret_cast<const uint8_t *>(p.near[k % 3]);
    uint8_t *next = reinterpret_cast<uint8_t *>(p.near[(k + 1) % 3]);
    uint32_t *clear = p.near[(k + 2) % 3];
    for (uint32_t i = threadIdx.x; i < p.n_states << p.n_props; i += blockDim.x) moves[i] = p.delta[i];
    for (uint64_t i = i0; i < p.near_words; i += step) clear[i] = 0;
    __syncthreads();
    bool changed = false;
    for (uint64_t e = i0; e < p.n_edges; e += step) {
        const uint32_t u = p.src[e];
        auto marked = [&] { return (LARGE ? now[u] | next[u] : now[u]) != 0; };
        // whether the sources of the wavefront's edges lie far apart
        auto far = [&] { return __ballot((uint64_t)(u - (uint32_t)__builtin_amdgcn_readfirstlane((int)u)) * p.n_states >= 128u) != 0; };
        if (LARGE && far() && (u >= p.n_vertices || !marked())) continue;
        const uint32_t v = p.dst[e], c = p.cost[e], sigma = p.sigma[e];
        if (!edge_ok(p, u, v, c)) continue;
        bool go = marked();
        uint32_t du[S];
#pragma unroll
        for (int q = 0; q < S; ++q) du[q] = (uint32_t)(p.best[(uint64_t)u * p.n_states + min((uint32_t)q, p.n_states - 1)] >> 32);
        const uint32_t looks = far() ? 1u : most_looks;
        for (uint32_t r = 1;; ++r) {
            if (go) {
                uint64_t cand[S], to[S], old[S];
#pragma unroll
                for (int q = 0; q < S; ++q) {
                    const uint32_t q2 = (uint32_t)q < p.n_states ? moves[((uint32_t)q << p.n_props) | sigma] : p.n_states;
                    const uint64_t nd = (uint64_t)du[q] + c;
                    to[q] = (uint64_t)v * p.n_states + min(q2, p.n_states - 1);
                    // no product edge: the source is not reached, the monitor
                    // rejects, the cost cannot be represented, or it ends at the
                    // start, which keeps distance 0 and no predecessor
                    const bool edge = du[q] != kInf && q2 < p.n_states && nd < kInf && to[q] != p.start;
                    cand[q] = edge ? (nd << 32) | (e * p.n_states + q) : kNone;
                    old[q] = p.best[to[q]];
                }
                bool nearer = false;
#pragma unroll
                for (int q = 0; q < S; ++q)
                    if (cand[q] < old[q]) {  // values only decrease: otherwise it cannot win
                        best_min(p.best, to[q], cand[q]);
                        // a smaller edge id at the same distance changes no neighbour
                        nearer = nearer || cand[q] >> 32 < old[q] >> 32;
                    }
                if (nearer) {
                    changed = true;
                    next[v] = 1;
                }
            }
            if (r >= looks) break;
            // the source again, as the other workgroups have left it by now
            go = false;
#pragma unroll
            for (int q = 0; q < S; ++q) {
                const uint32_t *d = reinterpret_cast<const uint32_t *>(p.best + (uint64_t)u * p.n_states + min((uint32_t)q, p.n_states - 1)) + 1;
                const uint32_t n = __hip_atomic_load(d, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                go = go || n < du[q];
                du[q] = min(du[q], n);
            }
        }
    }
    const uint64_t any = __ballot(changed);  // one atomic per wavefront that saw a change
    if (any && (threadIdx.x & 63) == (uint32_t)__builtin_ctzll(any)) atomicOr(p.changed + k % 4, 1u);
}

unsigned blocks_for(uint64_t n) { return (unsigned)std::min<uint64_t>(std::max<uint64_t>((n + 255) / 256, 1), 8192); }

}  // namespace

// A sweep's threads take edges, and the one that writes the outputs (and every
// sweep, in clearing its marks) product vertices, of which a roadmap has fewer
// than edges; a graph of few edges still gets a thread for every 16.  Us per call
// by edges alone and so: 100,000 vertices and 1,000 edges 53, 40; 1,000,000 and
// 1,000 240, 47; 10,000,000 and 1,000 2,576, 83; 10,000,000 and 100,000 103, 93.
unsigned plan_sweep_blocks(uint64_t n_product, uint64_t n_edges) { return blocks_for(std::max(n_edges, n_product / 16)); }

}  // namespace lbl

using namespace lbl;

extern "C" lbl_status lbl_product_shortest_paths(uint64_t n_vertices, uint64_t n_edges, const uint32_t *src,
                                                 const uint32_t *dst, const uint32_t *cost, const uint8_t *L,
                                                 uint32_t l_stride, uint32_t n_props, uint32_t n_states,
                                                 const uint8_t *delta,
                                                 uint32_t v0, uint32_t q0, uint32_t *dist, uint32_t *pred,
                                                 uint32_t *n_sweeps, void *hip_stream)
{
    clear_error();
    LBL_REQUIRE(n_vertices > 0, "n_vertices must be positive");
    LBL_REQUIRE(n_edges == 0 || (src && dst && cost && L), "src, dst, cost or L is null");
    LBL_REQUIRE(delta && dist && pred, "delta, dist or pred is null");
    LBL_REQUIRE(n_props >= 1 && n_props <= 8, "n_props must be in [1, 8]");
    LBL_REQUIRE(l_stride >= n_props, "l_stride must be at least n_props");
    LBL_REQUIRE(n_states >= 1 && n_states <= 8, "n_states must be in [1, 8]");
    LBL_REQUIRE(v0 < n_vertices && q0 < n_states, "start vertex or state out of range");
    LBL_REQUIRE(n_vertices * n_states < 0xFFFFFFFFull, "too many product vertices (n_vertices * n_states >= 2^32 - 1)");
    LBL_REQUIRE(n_edges * n_states < 0xFFFFFFFFull, "too many product edges (n_edges * n_states >= 2^32 - 1)");
    const size_t n_delta = (size_t)n_states << n_props;
    for (size_t i = 0; i < n_delta; ++i)
        LBL_REQUIRE(delta[i] < n_states || delta[i] == LBL_MONITOR_REJECT,
                    "delta holds a state >= n_states (use LBL_MONITOR_REJECT for no move)");
    hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
    int cur = 0;
    LBL_HIP_TRY(hipGetDevice(&cur));

    const uint64_t n = n_vertices * n_states;
    const uint64_t near_words = (n_vertices + 3) / 4;
    auto up = [](size_t x) { return (x + 255) & ~size_t(255); };
    void *ws = nullptr, *pin = nullptr;
    lbl_status st = workspace(s, up(n * sizeof(uint64_t)) + 3 * up(near_words * 4) + up(n_delta) + up(n_edges) + 256, &ws);
    if (st != LBL_OK) return st;
    st = pinned_flags(s, &pin);
    if (st != LBL_OK) return st;
    static_assert((kReports + 1) * sizeof(uint64_t) <= kPinnedBytes, "reports must fit the pinned memory");
    volatile uint64_t *report = static_cast<volatile uint64_t *>(pin);
    for (uint32_t i = 0; i <= kReports; ++i) report[i] = 0;
    uint8_t *at = static_cast<uint8_t *>(ws);
    auto take = [&](size_t bytes) {
        uint8_t *r = at;
        at += up(bytes);
        return r;
    };
    PlanArgs p{};
    p.src = src;
    p.dst = dst;
    p.cost = cost;
    p.n_vertices = n_vertices;
    p.n_edges = n_edges;
    p.start = (uint64_t)v0 * n_states + q0;
    p.n_props = n_props;
    p.n_states = n_states;
    p.best = reinterpret_cast<uint64_t *>(take(n * sizeof(uint64_t)));
    for (uint32_t *&w : p.near) w = reinterpret_cast<uint32_t *>(take(near_words * 4));
    p.near_words = (uint32_t)near_words;
    p.delta = take(n_delta);
    p.sigma = take(n_edges);
    p.changed = reinterpret_cast<uint32_t *>(take(16));
    void *dev_report = nullptr;
    LBL_HIP_TRY(hipHostGetDevicePointer(&dev_report, pin, 0));
    p.report = static_cast<uint64_t *>(dev_report);
    p.dist = dist;
    p.pred = pred;
    Delta d{};
    std::copy(delta, delta + n_delta, d.move);
    hipLaunchKernelGGL(k_plan_init, dim3(blocks_for(std::max(n, n_edges))), dim3(256), 0, s, p, d, (uint32_t)n_delta, L,
                       l_stride);
    LBL_HIP_TRY(hipGetLastError());
    // Bellman-Ford needs at most n sweeps before one that changes nothing
    // (sweep n at the latest), and sweep n + 1 to report on it
    uint64_t launched = 0, known = 0;  // sweeps enqueued; reported on
    bool done = false;
    uint32_t idle = 0;
    const dim3 grid(plan_sweep_blocks(n, n_edges));
    // a look reads n_states distances per edge
    const bool large = n_edges > kLargeEdges;
    const uint32_t looks = large ? 4u : std::min(16u, std::max(4u, 32u / n_states));
    auto of = [large](auto s) { return large ? &k_plan_sweep<s.value, true> : &k_plan_sweep<s.value, false>; };
    const auto sweep = n_states <= 1   ? of(std::integral_constant<int, 1>())
                       : n_states <= 2 ? of(std::integral_constant<int, 2>())
                       : n_states <= 4 ? of(std::integral_constant<int, 4>())
                                       : of(std::integral_constant<int, 8>());
    while (!done && known <= n) {
        if (launched < known + 1 + kAhead && launched < n + 2) {
            hipLaunchKernelGGL(sweep, grid, dim3(256), 0, s, p, launched, looks);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) {
                (void)hipStreamSynchronize(s);  // the pinned memory and the caller's arrays are still in use
                LBL_HIP_TRY(e);
            }
            ++launched;
        } else if (++idle % 4096 == 0) {
            // nothing for a while: a kernel that failed will never report
            hipError_t e = hipStreamQuery(s);
            if (e != hipErrorNotReady) {
                LBL_HIP_TRY(e);
                const uint64_t r = report[known % kReports];
                LBL_REQUIRE(r >> 1 == known + 1, "the sweeps ended without a report");
            }
        }
        for (;;) {
            const uint64_t r = report[known % kReports];
            if (r >> 1 != known + 1) break;
            ++known;
            idle = 0;
            if (!(r & 1)) {
                done = true;
                break;
            }
        }
    }
    LBL_HIP_TRY(hipStreamSynchronize(s));
    LBL_REQUIRE(report[kReports] == 0, "an edge names a vertex >= n_vertices or has cost 0");
    LBL_REQUIRE(done, "no fixpoint within the Bellman-Ford bound (cannot happen with costs >= 1)");
    const uint64_t sweeps = known;
    if (n_sweeps) *n_sweeps = (uint32_t)std::min<uint64_t>(sweeps, 0xFFFFFFFFull);
    return LBL_OK;
}
