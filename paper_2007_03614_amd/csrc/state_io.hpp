// Reading and writing a handle's state on the device.
//
// The caller's arrays are by vehicle id, the device's layout is sorted by lane:
// the kernels here gather one into the other, so that a read is one kernel and
// one copy (or, for a large state, one per field) and a write is the copies in
// and a counting sort by lane.  Done on the host, a written state of 470,000
// vehicles took 63 ms of sorting and copying, and a read of 50 vehicles 250 us of
// small copies, each waited for.
#pragma once
#include "step_kernels.hpp"

namespace manta {

// The head of a state on its way in or out
struct IoHead {
    int t;
    int err;            // out: the handle's device checks
    int bad;            // a check of this state failed
    int n_act;
    int departed;       // in: vehicles that have left the departure queues
    int set_counters;   // in
    long long counters[cNumCounters];
};

// A state's arrays by vehicle id, in one block of memory
struct StateIo {
    IoHead* head;
    double *tau_in, *t_arr;
    float *x, *v;
    int *edge, *lane, *cursor, *held_since, *ww;
    uint8_t *status, *mand;
};

// The arrays of n vehicles in a block at `base`; returns its size.
inline size_t state_io_at(char* base, int n, StateIo* io) {
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char* p = base + o;
        o += (bytes + 255) & ~(size_t)255;
        return p;
    };
    const size_t N = (size_t)n;
    StateIo s;
    s.head = (IoHead*)take(sizeof(IoHead));
    s.tau_in = (double*)take(8 * N);
    s.t_arr = (double*)take(8 * N);
    s.x = (float*)take(4 * N);
    s.v = (float*)take(4 * N);
    s.edge = (int*)take(4 * N);
    s.lane = (int*)take(4 * N);
    s.cursor = (int*)take(4 * N);
    s.held_since = (int*)take(4 * N);
    s.ww = (int*)take(4 * N);
    s.status = (uint8_t*)take(N);
    s.mand = (uint8_t*)take(N);
    if (io) *io = s;
    return o;
}

// What the kernels need besides the handle's own arrays
struct IoWork {
    const uint32_t* entry;    // [vehicle] first route edge | entry lane << 24
    const int* dep;           // [vehicle] departure step
    const int* q0;            // [queue + 1] first index of each departure queue
    int* list;                // [vehicle] active vehicles by lane, unordered within
    int* cnt;                 // [lane] vehicles still to be placed; zero between calls
    int lane_max;             // vehicles that a lane can hold without an overlap, at most
    int* off;                 // [lane] first slot, relative to the lane's block
    int* blk;                 // [commit block] vehicles, then first slot
    int* qmin;                // [queue] first index that still waits, last that has left
    int* qmax;
};

__device__ inline int route_edge_at(const Dev& d, const IoWork& w, int i, int cursor) {
    return cursor == 0 ? (int)(w.entry[i] & kLaneEdgeMask) : word_next(d.rnext[d.roff[i] + cursor - 1]);
}

// ---- read --------------------------------------------------------------------
__global__ void __launch_bounds__(kNT) k_io_read(Dev d, IoWork w, StateIo o) {
    const StepHead sh = step_head(d.ctl);
    const int par = sh.t_a & 1, na = par ? sh.n1 : sh.n0, tid = threadIdx.x;
    const Slots S = d.s[par];
    for (int i = blockIdx.x * kNT + tid; i < max(d.n_veh, na); i += gridDim.x * kNT) {
        if (i < d.n_veh) {
            const uint8_t st = d.status[i];
            const int cur = d.cursor[i];
            o.status[i] = st;
            o.cursor[i] = cur;
            o.held_since[i] = d.held_since[i];
            o.tau_in[i] = d.tau_in[i];
            o.t_arr[i] = d.t_arr[i];
            if (st == kArrived) {
                const uint32_t m = d.fin_meta[i];
                o.x[i] = d.fin_x[i];
                o.v[i] = d.fin_v[i];
                o.edge[i] = route_edge_at(d, w, i, cur);
                o.lane[i] = m_lane(m);
                o.mand[i] = m_mand(m);
                o.ww[i] = m_ww(m);
            } else if (st == kWaiting) {
                o.x[i] = 0.0f;
                o.v[i] = 0.0f;
                o.edge[i] = (int)(w.entry[i] & kLaneEdgeMask);
                o.lane[i] = (int)(w.entry[i] >> kLaneEdgeBits);
                o.mand[i] = 0;
                o.ww[i] = 0;
            }
        }
        if (i < na) {                              // an active vehicle, by its slot
            const uint32_t vid = S.vid[i], m = S.meta[i];
            if (vid >= (uint32_t)d.n_veh || d.status[vid] != kActive) {
                o.head->bad = 1;
                continue;
            }
            o.x[vid] = S.x[i];
            o.v[vid] = S.v[i];
            o.edge[vid] = S.edge[i];
            o.lane[vid] = m_lane(m);
            o.mand[vid] = m_mand(m);
            o.ww[vid] = m_ww(m);
        }
    }
    if (blockIdx.x < cNumCounters) {               // one workgroup per counter (at least as many are launched)
        __shared__ unsigned long long sum;
        if (tid == 0) sum = 0;
        __syncthreads();
        unsigned long long s = 0;
        for (int k = tid; k < kCounterCopies; k += kNT) s += d.counters[blockIdx.x * kCounterCopies + k];
        atomicAdd(&sum, s);
        __syncthreads();
        if (tid == 0) o.head->counters[blockIdx.x] = (long long)sum;
    }
    if (blockIdx.x == 0 && tid == 0) {
        o.head->t = sh.t_a;
        o.head->err = d.ctl->err;
        o.head->n_act = na;
    }
}

// ---- write -------------------------------------------------------------------
__global__ void __launch_bounds__(kNT) k_io_clear(IoWork w, int nq) {
    for (int q = blockIdx.x * kNT + threadIdx.x; q < nq; q += gridDim.x * kNT) {
        w.qmin[q] = INT_MAX;
        w.qmax[q] = -1;
    }
}

// The vehicles of a wavefront that share a key (their lane, their queue), one
// key after another: f(key, the set of them), up to kIoKeys keys; returns the
// set left over.  One atomic for each such group: 32,000 atomics on the one
// counter of a lane or queue take 0.35 ms.  (All lanes of the wavefront call.)
constexpr int kIoKeys = 2;
template <class F>
__device__ inline unsigned long long io_groups(bool have, int key, F&& f) {
    unsigned long long todo = __ballot(have);
    for (int r = 0; r < kIoKeys && todo != 0ull; ++r) {
        const int k = __builtin_amdgcn_readlane(key, __ffsll((long long)todo) - 1);
        const unsigned long long m = __ballot(have && key == k);
        f(k, m);
        todo &= ~m;
    }
    return todo;
}

// Every check of one vehicle's fields, its lane's count and its queue's bounds.
__global__ void __launch_bounds__(kNT) k_io_check(Dev d, IoWork w, StateIo in) {
    int left = 0;
    bool bad = false;
    const int lane = threadIdx.x & 63;
    for (int i0 = blockIdx.x * kNT; i0 < d.n_veh; i0 += gridDim.x * kNT) {
        const int i = i0 + threadIdx.x;
        const bool have = i < d.n_veh;
        int4 vq = make_int4(0, 0, 0, 0);
        int waits = -1, gone = -1;                 // place in its queue from the end, or from the front
        int gl = -1;
        if (have) {
            const uint8_t st = in.status[i];
            const int cur = in.cursor[i];
            vq = d.vq[i];
            if (st == kWaiting) waits = INT_MAX - vq.y;
            else gone = vq.y;
            left += st != kWaiting;
            bool ok = st <= kArrived && cur >= 0 && cur < d.roff[i + 1] - d.roff[i];
            if (ok && st == kActive) {
                const int e = route_edge_at(d, w, i, cur), l = in.lane[i], ww = in.ww[i];
                const EdgeC c = d.ec[e];
                const float x = in.x[i], v = in.v[i];
                ok = in.edge[i] == e && l >= 0 && l < c.lanes && x >= 0.0f && x <= c.L && v >= 0.0f && v < INFINITY &&
                     ww >= 0 && ww <= kPatience;
                if (ok) gl = c.lane_base + l;
            }
            bad = bad || !ok;
        }
        unsigned long long rest = io_groups(have, vq.x, [&](int q, unsigned long long m) {
            const bool in_q = (m >> lane) & 1ull;
            const int a = __builtin_amdgcn_readlane(wave_incl_max(in_q ? waits : -1), 63);
            const int b = __builtin_amdgcn_readlane(wave_incl_max(in_q ? gone : -1), 63);
            if (lane == 0 && a >= 0) atomicMin(&w.qmin[q], INT_MAX - a);
            if (lane == 0 && b >= 0) atomicMax(&w.qmax[q], b);
        });
        if ((rest >> lane) & 1ull) {
            if (waits >= 0) atomicMin(&w.qmin[vq.x], vq.y);
            else atomicMax(&w.qmax[vq.x], vq.y);
        }
        rest = io_groups(gl >= 0, gl, [&](int g, unsigned long long m) {
            if (lane == 0) atomicAdd(&w.cnt[g], (int)__popcll(m));
        });
        if ((rest >> lane) & 1ull) atomicAdd(&w.cnt[gl], 1);
    }
    left = (int)__ockl_wfred_add_u32((unsigned)left);
    if (lane == 0 && left) atomicAdd(&in.head->departed, left);
    if (bad) in.head->bad = 1;
}

// A lane with more vehicles than it can hold has two that overlap: the state
// is refused here, before anything is done for each pair of a lane's vehicles.
template <int NT>
__global__ void __launch_bounds__(NT) k_io_lanes(IoWork w, IoHead* head) {
    __shared__ int wsh[NT / 64];
    const int gl = blockIdx.x * NT + threadIdx.x;
    const int c = w.cnt[gl];
    if (c > w.lane_max) head->bad = 1;
    const int o = wg_exclusive_sum<NT>(c, wsh);
    w.off[gl] = o;
    if (threadIdx.x == NT - 1) w.blk[blockIdx.x] = o + c;
}

__global__ void __launch_bounds__(kBigNT) k_io_blocks(Dev d, IoWork w, IoHead* head) {
    __shared__ int wsh[kBigNT / 64];
    __shared__ int tot;
    __shared__ int stage[kScanLdsMax];
    const int n = scan_block_sums_staged<kBigNT>(w.blk, d.n_blk, w.blk, stage, kScanLdsMax, wsh, &tot);
    if (threadIdx.x == 0) head->n_act = n;
}

__device__ inline int io_start(const Dev& d, const IoWork& w, int gl, int n_act) {
    return gl < d.n_lanes_total ? w.blk[gl >> d.lane_shift] + w.off[gl] : n_act;
}

// The active vehicles of every lane, in any order (a state with a bad vehicle
// is refused in the end; here its vehicles that passed are placed all the
// same, which takes every lane's count back to zero).
__global__ void __launch_bounds__(kNT) k_io_place(Dev d, IoWork w, StateIo in) {
    const int lane = threadIdx.x & 63;
    for (int i0 = blockIdx.x * kNT; i0 < d.n_veh; i0 += gridDim.x * kNT) {
        const int i = i0 + threadIdx.x;
        int gl = -1;
        if (i < d.n_veh && in.status[i] == kActive) {
            const int cur = in.cursor[i];
            if (cur >= 0 && cur < d.roff[i + 1] - d.roff[i]) {
                const int e = route_edge_at(d, w, i, cur), l = in.lane[i], ww = in.ww[i];
                const EdgeC c = d.ec[e];
                const float x = in.x[i], v = in.v[i];
                if (in.edge[i] == e && l >= 0 && l < c.lanes && x >= 0.0f && x <= c.L && v >= 0.0f && v < INFINITY &&
                    ww >= 0 && ww <= kPatience)
                    gl = c.lane_base + l;
            }
        }
        int at = 0;                                // vehicles of the lane up to this one
        const unsigned long long rest = io_groups(gl >= 0, gl, [&](int g, unsigned long long m) {
            const int n = (int)__popcll(m);
            int last = 0;
            if (lane == 0) last = atomicSub(&w.cnt[g], n);
            last = __builtin_amdgcn_readfirstlane(last);
            if ((m >> lane) & 1ull) at = last - bits_below(m);
        });
        if ((rest >> lane) & 1ull) at = atomicSub(&w.cnt[gl], 1);
        if (gl >= 0) w.list[w.blk[gl >> d.lane_shift] + w.off[gl] + at - 1] = i;
    }
}

// On lanes of more than kIoLong vehicles a rank is looked up in sorted pieces:
// the list in chunks of kIoChunk, each by lane and then front first, in LDS.
// (Comparing with every vehicle of the lane takes 0.17 us each: a state of
// 32,000 vehicles on one lane is written in 5.4 ms, so in 0.35, and sorted on the
// host in 2.4.  Chunks without such a lane are left as they are, and networks
// that cannot have one do not launch this.)
constexpr int kIoLong = 256;
constexpr int kIoChunk = 1024;

struct IoKey {                // order within a chunk: first slot of the lane, then x and id, both descending
    int lo;
    float x;
    int id;
};
__device__ inline bool io_before(const IoKey& a, const IoKey& b) {
    return a.lo != b.lo ? a.lo < b.lo : a.x != b.x ? a.x > b.x : a.id > b.id;
}

__global__ void __launch_bounds__(kIoChunk / 2) k_io_sort(Dev d, IoWork w, StateIo in) {
    __shared__ IoKey key[kIoChunk];
    const int na = in.head->n_act, tid = threadIdx.x;
    if (in.head->bad) return;
    for (int c0 = blockIdx.x * kIoChunk; c0 < na; c0 += gridDim.x * kIoChunk) {
        bool any = false;
        for (int k = tid; k < kIoChunk; k += kIoChunk / 2) {
            key[k] = IoKey{INT_MAX, 0.0f, 0};
            if (c0 + k >= na) continue;
            const int i = w.list[c0 + k], gl = d.ec[in.edge[i]].lane_base + in.lane[i], lo = io_start(d, w, gl, na);
            key[k] = IoKey{lo, in.x[i], i};
            any = any || io_start(d, w, gl + 1, na) - lo > kIoLong;
        }
        if (!__syncthreads_or(any)) continue;
        for (int m = 2; m <= kIoChunk; m *= 2)                  // bitonic
            for (int h = m / 2; h > 0; h /= 2) {
                const int k = 2 * tid - (tid & (h - 1));        // and its partner, h further
                const IoKey a = key[k], b = key[k + h];
                const bool up = (k & m) == 0;
                if (up ? io_before(b, a) : io_before(a, b)) {
                    key[k] = b;
                    key[k + h] = a;
                }
                __syncthreads();
            }
        for (int k = tid; k < kIoChunk && c0 + k < na; k += kIoChunk / 2) w.list[c0 + k] = key[k].id;
        __syncthreads();
    }
}

// Each vehicle's rank in its lane (front first: x, then id, descending) and its
// record in layout B.  sorted: k_io_sort has run.
__global__ void __launch_bounds__(kNT) k_io_rank(Dev d, IoWork w, StateIo in, Slots B, bool sorted) {
    const int na = in.head->n_act;
    if (in.head->bad) return;
    for (int s = blockIdx.x * kNT + threadIdx.x; s < na; s += gridDim.x * kNT) {
        const int i = w.list[s], e = in.edge[i], l = in.lane[i], cur = in.cursor[i];
        const float x = in.x[i];
        const int gl = d.ec[e].lane_base + l;
        const int lo = io_start(d, w, gl, na), hi = io_start(d, w, gl + 1, na);
        const auto ahead = [&](int k) {
            const int j = w.list[k];
            const float xj = in.x[j];
            return xj > x || (xj == x && j > i);
        };
        int dst = lo;
        if (sorted && hi - lo > kIoLong) {
            // eight chunks' searches at once, so that their loads overlap
            constexpr int kU = 8;
            for (int c0 = lo / kIoChunk * kIoChunk; c0 < hi; c0 += kU * kIoChunk) {
                int at[kU];                       // those before it, of the chunk's part of the lane, end here
#pragma unroll
                for (int u = 0; u < kU; ++u) at[u] = max(lo, c0 + u * kIoChunk);
                for (int h = kIoChunk; h > 0; h /= 2) {
#pragma unroll
                    for (int u = 0; u < kU; ++u) {
                        const int k = at[u] + h - 1;
                        const bool in_part = k < min(hi, c0 + (u + 1) * kIoChunk);
                        if (ahead(in_part ? k : lo) && in_part) at[u] += h;
                    }
                }
#pragma unroll
                for (int u = 0; u < kU; ++u) dst += at[u] - max(lo, c0 + u * kIoChunk);
            }
        } else {
            for (int k = lo; k < hi; ++k) dst += ahead(k) ? 1 : 0;
        }
        const uint32_t rw = d.rnext[d.roff[i] + cur];
        B.x[dst] = x;
        B.v[dst] = in.v[i];
        B.vid[dst] = (uint32_t)i;
        B.edge[dst] = e;
        B.meta[dst] = m_make(l, in.mand[i] != 0, in.held_since[i] >= 0, in.ww[i], d.cls[i], rw >> 24);
        B.nxt[dst] = word_next(rw);
        if (d.v0_spread != 0.0f) B.lim[dst] = kLimUnknown;
    }
}

// No vehicle overlaps its leader, and the vehicles that have left a departure
// queue are a prefix of it.
__global__ void __launch_bounds__(kNT) k_io_verify(Dev d, IoWork w, StateIo in, Slots B) {
    const int na = in.head->n_act;
    if (in.head->bad) return;
    for (int s = blockIdx.x * kNT + threadIdx.x; s < max(na, d.nq); s += gridDim.x * kNT) {
        bool bad = false;
        if (s > 0 && s < na && B.edge[s] == B.edge[s - 1] && m_lane(B.meta[s]) == m_lane(B.meta[s - 1]))
            bad = B.x[s - 1] - d.cp[m_cls(B.meta[s - 1])].len < B.x[s];
        if (s < d.nq) bad = bad || w.qmax[s] > w.qmin[s];
        if (bad) in.head->bad = 1;
    }
}

// The checked state becomes the handle's.  B: the layout built above, in the
// buffer that the current step does not use; S: where step t reads it.
__global__ void __launch_bounds__(kNT) k_io_apply(Dev d, IoWork w, StateIo in, Slots B, Slots S) {
    const IoHead& h = *in.head;                // (a copy, its counters indexed, would live in scratch memory)
    if (h.bad) return;
    const int t = h.t, na = h.n_act, nl = d.n_lanes_total, nn = d.imode == 1 ? d.n_nodes : 0;
    const int most = max(max(max(d.n_veh, nl), max(d.nq, nn)), cNumCounters * kCounterCopies);
    for (int i = blockIdx.x * kNT + threadIdx.x; i < most; i += gridDim.x * kNT) {
        if (i < d.n_veh) {
            const uint8_t st = in.status[i];
            d.status[i] = st;
            d.cursor[i] = in.cursor[i];
            d.held_since[i] = in.held_since[i];
            d.tau_in[i] = in.tau_in[i];
            d.t_arr[i] = in.t_arr[i];
            const bool arr = st == kArrived;
            d.fin_x[i] = arr ? in.x[i] : 0.0f;
            d.fin_v[i] = arr ? in.v[i] : 0.0f;
            d.fin_meta[i] = arr ? m_make(in.lane[i], in.mand[i] != 0, false, in.ww[i], d.cls[i], 0) : 0u;
            const int4 vq = d.vq[i];
            if (st == kWaiting && w.qmin[vq.x] == vq.y) d.qhd[vq.x] = make_int2(w.dep[i], i);
        }
        if (i < d.nq) {
            const bool none = w.qmin[i] == INT_MAX;
            d.qhead[i] = none ? w.q0[i + 1] : w.qmin[i];
            if (none) d.qhd[i] = make_int2(INT_MAX, -1);
        }
        if (i < nl) {
            const int lo = io_start(d, w, i, na), hi = io_start(d, w, i + 1, na);
            LaneRear r{0.0f, 0.0f, -1, 0u};
            if (lo < hi) r = LaneRear{B.x[hi - 1] - d.cp[m_cls(B.meta[hi - 1])].len, B.v[hi - 1], t, B.vid[hi - 1]};
            d.rear[i] = r;
            d.post[i].stamp = -1;              // no stamp of another run: requests, claims, big tiles
            d.req_stamp[i] = d.exit_stamp[i] = d.enter_stamp[i] = -1;
            d.win[i] = ~0ull;
            d.big_lane[i] = make_int2(-1, -1);
        }
        if (i < na && S.x != B.x) {
            S.x[i] = B.x[i];
            S.v[i] = B.v[i];
            S.vid[i] = B.vid[i];
            S.edge[i] = B.edge[i];
            S.meta[i] = B.meta[i];
            S.nxt[i] = B.nxt[i];
            if (d.v0_spread != 0.0f) S.lim[i] = B.lim[i];
        }
        if (i < nn) {                          // the round-robin restarts
            d.rr[i] = -1;
            d.win_node[i] = ~0ull;
        }
        if (i < kMovedSlots) d.moved_at[i] = -1;
        if (i < kTileCtrInts) tile_counters(d)[i] = 0;
        if (h.set_counters && i < cNumCounters * kCounterCopies)
            d.counters[i] = i % kCounterCopies == 0 ? (unsigned long long)h.counters[i / kCounterCopies] : 0ull;
        if (i == 0) {
            Ctl c{};
            c.t_a = t;
            c.t_b = t;
            c.n_act[t & 1] = na;
            c.n_departed = h.departed;
            *d.ctl = c;
        }
    }
}

}  // namespace manta
