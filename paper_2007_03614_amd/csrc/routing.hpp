// Routes on travel times (the fixed routes of Sec. II-C, re-computed on the
// GPU from current per-edge costs, e.g. the mean traversal times of the step
// statistics).  Binary32 costs; for a destination d
//   dist(d) = 0,  dist(v) = min over out-edges e = (v -> u) of fl(cost_e + dist(u)),
// and a route leaves every node by the out-edge of smallest
// (fl(cost_e + dist(head e)), edge id).  Any order of relaxation reaches the
// same least fixed point as Dijkstra from d when every cost is positive, so
// the result does not depend on the schedule of the sweeps.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace manta {

constexpr int kRouteNT = 1024;
constexpr int kRouteMaxNodes = 16000;   // one binary32 label per node, within 64 KiB of LDS

// Networks with a node of more than kRouteTreeDeg out-edges: one workgroup
// per destination, labels in LDS, Bellman-Ford sweeps in place until one
// changes nothing (at most V sweeps).  Out-edges of node v are
// out_edge[out_off[v] .. out_off[v + 1]).
__global__ void __launch_bounds__(kRouteNT) k_route_dist(int V, const int* out_off, const int* out_edge,
                                                        const int* edge_to, const float* cost, const int* dests,
                                                        int nd, float* dist_out) {
    __shared__ float dist[kRouteMaxNodes];
    __shared__ int changed;
    for (int q = blockIdx.x; q < nd; q += gridDim.x) {
        const int d = dests[q];
        for (int v = threadIdx.x; v < V; v += kRouteNT) dist[v] = v == d ? 0.0f : INFINITY;
        __syncthreads();
        for (int it = 0; it < V; ++it) {
            if (threadIdx.x == 0) changed = 0;
            __syncthreads();
            bool ch = false;
            for (int v = threadIdx.x; v < V; v += kRouteNT) {
                float best = dist[v];
                for (int k = out_off[v]; k < out_off[v + 1]; ++k) {
                    const int e = out_edge[k];
                    const float c = cost[e] + dist[edge_to[e]];
                    if (c < best) best = c;
                }
                if (best < dist[v]) {
                    dist[v] = best;
                    ch = true;
                }
            }
            if (ch) changed = 1;
            __syncthreads();
            const bool more = changed != 0;
            __syncthreads();   // every thread has read the flag before it is reset
            if (!more) break;
        }
        for (int v = threadIdx.x; v < V; v += kRouteNT) dist_out[(size_t)q * V + v] = dist[v];
        __syncthreads();
    }
}

// ---- label trees in LDS ----------------------------------------------------
// Networks of at most kRouteTreeNodes nodes and out-degree kRouteTreeDeg: one
// workgroup per destination holds every label in LDS and relaxes from a
// frontier, the nodes whose label dropped, over their in-edges.  Sweeps over
// all nodes touch every label some 150 times on a 10,000-node city.  A plain
// frontier expands each node 5 times there and 14 times on a 40,000-node
// lattice, since labels drop again as longer chains of cheaper edges arrive;
// expanding only labels below a threshold, raised by a few mean edge costs
// when none is left below it, brings that to 1.2 in both at a fifth more
// rounds.
//
// A label word is the bit pattern of its non-negative float shifted left by
// one, with bit 0 set while the node is NOT waiting to be expanded, so one
// atomicMin lowers the label, marks the node waiting and returns what it was.
// (Shifted patterns order like the floats.)  Waiting nodes below the threshold
// are listed in what is left of the workgroup's LDS; those above it, and a
// round that lists more than fits, are found again by their bit.
//
// What bounds it: the chain of rounds, one dependent load of adjacency from L2
// and five LDS operations each, so four lanes share a node's in-edges and as
// many workgroups as the LDS holds share a CU.  9,900 destinations of the
// city: 2.8 ms, against 10.4 ms for sweeps with the adjacency in registers;
// 400 destinations of the lattice: 1.1 ms, against 23 ms for labels in device
// memory.
constexpr int kRouteTreeNodes = 40400;  // 4 bytes each, and at least 512 entries in each of two lists, in 160 KiB
constexpr int kRouteTreeDeg = 8;        // bounds the in-edge records by the network's own arrays
constexpr size_t kRouteTreeLds = 163840 - 64;   // dynamic LDS of one workgroup at most
// Threshold step, in mean edge costs (route_tree_step): small steps rescan the labels for the
// nodes below the next threshold more often, large ones expand more nodes
// twice.  200,000 routes on a 10,040-node city end to end: 8.9 ms at 3, 7.6 at
// 8, 7.47 at 16, 7.42 at 24; a 40,000-node lattice 3.14, 3.10, 3.5 at 8, 16, 24.
constexpr double kRouteTreeStep = 16.0;
// Edges of more than kRouteTreeDear times the mean are not in it (closed roads, priced far above any time: with 1 %
// of the edges at 1e6 s in the mean no threshold binds, and the city takes 14.7 ms, the lattice 10.7; without them 7.8
// and 3.3, and 7.6 and 3.1 with no road closed.
constexpr double kRouteTreeDear = 16.0;
constexpr int kRouteTreeList = 1024;    // entries of a frontier list at most
constexpr unsigned kLabelInf = (0x7f800000u << 1) | 1u;

// The threshold step of n positive costs: kRouteTreeStep times the mean of those that are not dear against it.
inline float route_tree_step(const float* cost, int n) {
    constexpr int kU = 8;
    double mean = 0.0;
    float cut = INFINITY;
    for (int pass = 0; pass < 4; ++pass) {
        double part[kU] = {}, sum = 0.0;         // sums side by side, so that the additions overlap
        float top[kU] = {}, most = 0.0f;
        int in[kU] = {}, many = 0;
        const auto take = [&](const float* from, int j) {
            const float c = from[j] <= cut ? from[j] : 0.0f;
            part[j] += c;
            in[j] += c > 0.0f;
            top[j] = c > top[j] ? c : top[j];
        };
        int e = 0;
        for (; e + kU <= n; e += kU)
            for (int j = 0; j < kU; ++j) take(cost + e, j);
        for (int j = 0; e + j < n; ++j) take(cost + e, j);
        for (int j = 0; j < kU; ++j) {
            sum += part[j];
            many += in[j];
            most = top[j] > most ? top[j] : most;
        }
        mean = sum / many;
        if (!((double)most > kRouteTreeDear * mean)) break;
        cut = (float)(kRouteTreeDear * mean);
    }
    return (float)(kRouteTreeStep * mean);
}

// The in-edges of a node, four at a time: tails (-1 unused) and costs.  A node
// with more links on: tail[3] = -2 - index of the next record.
struct __align__(16) RouteIn {
    int tail[4];
    float cost[4];
};

struct RouteOut {   // an out-edge, in the order of the CSR: head and cost
    int head;
    float cost;
};

// lane J of the caller's quad of lanes (a DPP move; the four are active together)
template <int J>
__device__ inline int quad_lane(int x) {
    return __builtin_amdgcn_mov_dpp(x, J * 0x55, 0xf, 0xf, false);
}

// tab[q * V + v]: CSR index of the out-edge by which the route to dests[q]
// leaves v (-1: the destination itself, or no route).  len[i]: route edges of
// query i (-1: origin == destination, unreachable, or longer than V edges);
// the queries of destination q are qord[qoff[q] .. qoff[q + 1]).
__global__ void __launch_bounds__(kRouteNT) k_route_tree(int V, const RouteIn* __restrict__ in,
                                                        const int* __restrict__ out_off,
                                                        const RouteOut* __restrict__ out,
                                                        const int* __restrict__ dests, int list, float step,
                                                        int* __restrict__ tab, const int* __restrict__ qoff,
                                                        const int* __restrict__ qord, const int* __restrict__ origin,
                                                        int* __restrict__ len) {
    extern __shared__ unsigned lab[];
    __shared__ int cnt[3];                  // listed by round r: cnt[(r + 1) % 3]
    __shared__ unsigned lowest;             // smallest waiting label above the threshold
    uint16_t* const q0 = (uint16_t*)(lab + (V + 3) / 4 * 4);
    const int NT = (int)blockDim.x, tid = (int)threadIdx.x;
    const int q = blockIdx.x, d = dests[q];
    for (int v = tid; v < (V + 3) / 4 * 4; v += NT) lab[v] = v == d ? 0u : kLabelInf;
    if (tid < 3) cnt[tid] = 0;
    if (tid == 0) q0[0] = (uint16_t)d;
    __syncthreads();
    int ncur = 1;
    unsigned bar = __float_as_uint(step) << 1;   // labels below it are expanded
    for (int r = 0;; ++r) {
        uint16_t* const cur = q0 + (r & 1) * list;
        uint16_t* const nxt = q0 + ((r & 1) ^ 1) * list;
        int* const pushed = &cnt[(r + 1) % 3];
        auto push = [&](int v) {
            const int k = atomicAdd(pushed, 1);
            if (k < list) nxt[k] = (uint16_t)v;
        };
        // the four lanes of a quad take one node's in-edges, lane j the j-th of a record
        auto expand = [&](int u, int j) {
            const RouteIn* p = &in[u];
            int t = p->tail[j];
            float c = p->cost[j];
            unsigned w = 1u;
            if (j == 0) w = atomicOr(&lab[u], 1u);
            w = (unsigned)quad_lane<0>((int)w);
            if (w & 1u) return;              // expanded in a round without a list
            const float du = __uint_as_float(w >> 1);
            for (;;) {
                if (t >= 0) {
                    const unsigned key = __float_as_uint(c + du) << 1;
                    if (key < (lab[t] & ~1u)) {
                        const unsigned old = atomicMin(&lab[t], key);
                        // listed already: waiting with a label below the threshold
                        if (old > key && key < bar && ((old & 1u) || old >= bar)) push(t);
                    }
                }
                const int link = quad_lane<3>(t);
                if (link >= -1) break;
                p = &in[-2 - link];
                t = p->tail[j];
                c = p->cost[j];
            }
        };
        if (tid == 0) cnt[(r + 2) % 3] = 0;
        if (ncur <= list) {
            for (int i = tid >> 2; i < ncur; i += NT >> 2) expand(cur[i], tid & 3);
        } else {
            for (int v = tid >> 2; v < V; v += NT >> 2) {
                const unsigned w = lab[v];
                if (!(w & 1u) && w < bar) expand(v, tid & 3);
            }
        }
        __syncthreads();
        ncur = *pushed;
        if (ncur > 0) continue;
        // None left below the threshold: raise it by a step and list the
        // nodes that are now below it; where there is none, start from the
        // smallest label that waits (and past it, so that every pass lists one).
        if (tid == 0) lowest = ~0u;
        bar = __float_as_uint(__uint_as_float(bar >> 1) + step) << 1;
        __syncthreads();
        unsigned low = ~0u;
        for (int v = 4 * tid; v < V; v += 4 * NT) {
            const uint4 w4 = *(const uint4*)(lab + v);       // the words past V do not wait
            const unsigned w[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (!(w[j] & 1u)) {
                    low = min(low, w[j]);
                    if (w[j] < bar) push(v + j);
                }
        }
        if (low != ~0u) atomicMin(&lowest, low);
        __syncthreads();
        ncur = *pushed;
        if (ncur > 0) continue;
        if (lowest == ~0u) break;
        __syncthreads();                     // every thread has read the count before it is pushed to again
        bar = max(__float_as_uint(__uint_as_float(lowest >> 1) + step) << 1, lowest + 2u);
        for (int v = tid; v < V; v += NT) {
            const unsigned w = lab[v];
            if (!(w & 1u) && w < bar) push(v);
        }
        __syncthreads();
        ncur = *pushed;
    }
    // the edge by which each node's route leaves it: smallest cost + label,
    // lowest edge id; four nodes a thread at once, so that their loads overlap
    constexpr int kU = 4;
    int* const row = tab + (size_t)q * V;
    for (int v0 = tid; v0 < V; v0 += kU * NT) {
        int k0[kU], k1[kU], be[kU];
        float bc[kU];
#pragma unroll
        for (int j = 0; j < kU; ++j) {
            const int v = min(v0 + j * NT, V - 1);
            k0[j] = out_off[v];
            k1[j] = v == d || lab[v] == kLabelInf ? 0 : out_off[v + 1];
            be[j] = -1;
            bc[j] = INFINITY;
        }
        for (bool more = true; more;) {
            more = false;
#pragma unroll
            for (int j = 0; j < kU; ++j) {
                if (k0[j] >= k1[j]) continue;
                const RouteOut o = out[k0[j]];
                const float c = o.cost + __uint_as_float(lab[o.head] >> 1);
                if (be[j] < 0 || c < bc[j]) {
                    be[j] = k0[j];
                    bc[j] = c;
                }
                more |= ++k0[j] < k1[j];
            }
        }
#pragma unroll
        for (int j = 0; j < kU; ++j)
            if (v0 + j * NT < V) row[v0 + j * NT] = be[j];
    }
    __syncthreads();
#pragma unroll 4
    for (int v = tid; v < V; v += NT) {      // the labels make room for the next nodes
        const int k = row[v];                // written by this thread
        lab[v] = k >= 0 ? (unsigned)out[k].head : ~0u;
    }
    __syncthreads();
    for (int i = qoff[q] + tid; i < qoff[q + 1]; i += NT) {
        const int qi = qord[i], o = origin[qi];
        int n = 0;
        unsigned v = (unsigned)o;
        bool ok = o != d;
        while (ok && v != (unsigned)d) {
            v = lab[v];
            ok = v != ~0u && n < V;
            ++n;
        }
        len[qi] = ok ? n : -1;
    }
}

// The routes of one destination's queries from its row of tab: the next nodes
// in LDS (16 bits each), one wavefront per query.  Every lane walks the same
// chain; lane n % 64 keeps node n, and every 64 nodes the wavefront looks up
// and writes their edges together, so the chain waits for LDS only.
__global__ void __launch_bounds__(256) k_route_write(int V, const int* __restrict__ tab,
                                                    const RouteOut* __restrict__ out,
                                                    const int* __restrict__ out_edge, const int* __restrict__ dests,
                                                    const int* __restrict__ qoff, const int* __restrict__ qord,
                                                    const int* __restrict__ origin, const int64_t* __restrict__ off,
                                                    int* __restrict__ route_edges) {
    extern __shared__ unsigned lab[];
    uint16_t* const nx = (uint16_t*)lab;
    const int q = blockIdx.x, d = dests[q];
    const int* const row = tab + (size_t)q * V;
    for (int v = threadIdx.x; v < V; v += 256) {
        const int k = row[v];
        nx[v] = k >= 0 ? (uint16_t)out[k].head : (uint16_t)0;
    }
    __syncthreads();
    const int lane = threadIdx.x & 63;
    for (int i = qoff[q] + (int)(threadIdx.x >> 6); i < qoff[q + 1]; i += 4) {
        const int qi = qord[i];
        const int64_t o0 = off[qi];
        const int n = (int)(off[qi + 1] - o0);
        int v = origin[qi];
        for (int b = 0; b < n; b += 64) {
            const int m = min(64, n - b);
            int mine = 0;
            for (int j = 0; j < m; ++j) {
                mine = lane == j ? v : mine;
                v = nx[v];
            }
            if (lane < m) route_edges[o0 + b + lane] = out_edge[row[mine]];
        }
    }
}

// Networks above kRouteTreeNodes: one workgroup per destination with its
// labels in global memory (row q of dist_out), relaxed from a frontier -- the
// nodes whose label dropped in the last round push the drop to the tails of
// their in-edges (a label-correcting search; with positive costs it ends at
// the same binary32 fixed point as any other relaxation order, see above).
// A node enters the next frontier once per round (mark holds the round of
// its last push).  Labels are positive floats, so their bit patterns order
// like the values and atomicMin on the integer view takes the minimum.
// Labels, marks and frontier entries are read and written only by atomics
// at device scope (performed in L2, never served stale from a CU's L1), and
// every thread waits for its memory operations before each barrier.
// Per workgroup: frontier space 2 * V and marks V (fq, mk at blockIdx * V).
__device__ inline int ld_l2(const int* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void st_l2(int* p, int v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline void settle_and_sync() {
    __builtin_amdgcn_s_waitcnt(0);   // this thread's loads, stores and atomics are done
    __syncthreads();
}

__global__ void __launch_bounds__(kRouteNT) k_route_dist_global(int V, const int* in_off, const int* in_edge,
                                                               const int* edge_from, const float* cost,
                                                               const int* dests, int nd, float* dist_out, int* fq,
                                                               int* mk) {
    __shared__ int n_next;
    int* fa = fq + (size_t)blockIdx.x * 2 * V;
    int* fb = fa + V;
    int* mark = mk + (size_t)blockIdx.x * V;
    for (int q = blockIdx.x; q < nd; q += gridDim.x) {
        const int d = dests[q];
        int* idist = (int*)(dist_out + (size_t)q * V);
        for (int v = threadIdx.x; v < V; v += kRouteNT) {
            st_l2(&idist[v], __float_as_int(v == d ? 0.0f : INFINITY));
            st_l2(&mark[v], -1);
        }
        if (threadIdx.x == 0) {
            st_l2(&fa[0], d);
            n_next = 0;
        }
        settle_and_sync();
        int n_cur = 1;
        int* cur = fa;
        int* nxt = fb;
        for (int round = 0; n_cur > 0; ++round) {
            for (int i = threadIdx.x; i < n_cur; i += kRouteNT) {
                const int u = ld_l2(&cur[i]);
                const float du = __int_as_float(ld_l2(&idist[u]));
                for (int k = in_off[u]; k < in_off[u + 1]; ++k) {
                    const int e = in_edge[k];
                    const int v = edge_from[e];
                    const float c = cost[e] + du;
                    const int old = atomicMin(&idist[v], __float_as_int(c));
                    if (c < __int_as_float(old) && atomicExch(&mark[v], round) != round)
                        st_l2(&nxt[atomicAdd(&n_next, 1)], v);
                }
            }
            settle_and_sync();
            n_cur = n_next;
            __syncthreads();   // every thread has read the count before it is reset
            if (threadIdx.x == 0) n_next = 0;
            int* t = cur;
            cur = nxt;
            nxt = t;
        }
        __syncthreads();
    }
}

// One thread per query: walk from the origin to the destination over the
// labels of its destination (slot).  fill == 0: write the number of edges to
// len[q] (-1: origin == destination, unreachable, or longer than V edges);
// fill == 1: write the edges at route_edges[off[q] ...].
__global__ void __launch_bounds__(256) k_route_walk(int V, const int* out_off, const int* out_edge,
                                                   const int* edge_to, const float* cost, const float* dist_all,
                                                   const int* slot, const int* origin, const int* dest, int nq,
                                                   int fill, int* len, const int64_t* off, int* route_edges) {
    for (int q = blockIdx.x * 256 + threadIdx.x; q < nq; q += gridDim.x * 256) {
        const float* dist = dist_all + (size_t)slot[q] * V;
        const int o = origin[q], d = dest[q];
        int n = 0;
        bool ok = o != d && dist[o] < INFINITY;
        int v = o;
        while (ok && v != d) {
            int be = -1;
            float bc = INFINITY;
            for (int k = out_off[v]; k < out_off[v + 1]; ++k) {   // ascending edge id within a node
                const int e = out_edge[k];
                const float c = cost[e] + dist[edge_to[e]];
                if (be < 0 || c < bc) {
                    be = e;
                    bc = c;
                }
            }
            if (be < 0 || n >= V) {
                ok = false;
                break;
            }
            if (fill) route_edges[off[q] + n] = be;
            ++n;
            v = edge_to[be];
        }
        if (!fill) len[q] = ok ? n : -1;
    }
}

}  // namespace manta
