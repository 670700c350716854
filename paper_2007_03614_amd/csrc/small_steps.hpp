// Many steps of a small network in one launch.
//
// A step of the whole network is four launches that hand over through device
// memory: on a few hundred edges each lasts 4 to 14 us of launch, drain and
// dependent round trips to memory, whatever it has to do.  Here one workgroup
// runs every phase of one scenario (an ensemble: one workgroup each, as
// scenarios never touch) for as many steps as the launch is given, with a
// workgroup barrier where the four kernels have a launch boundary, the lanes'
// tables in LDS and the rest in the caches of one XCD.  The phases are the
// device functions of the four kernels, so the results are the same bit for
// bit.  What bounds it: the chain of dependent steps of one workgroup.
//
// Measured per step, four launches against this: a 50-vehicle ring 17.6 and
// 9.8 us, the 10x10 grid with 365 vehicles on the road 28.2 and 18.7, 32
// scenarios of it with 4,500 on the road 28.5 and 17.1, when it was written; by
// now the small kernel takes 6.7, 12.6 and 11.8.
#pragma once
#include "step_kernels.hpp"

namespace manta {

constexpr int kSmallNT = 512;            // threads per workgroup
constexpr int kSmallEdges = 1024;        // a scenario's edges, lanes and (case 1) nodes at most
constexpr int kSmallLanes = 1024;
constexpr int kSmallNodes = 1024;
constexpr int kSmallSteps = 1024;        // steps of one launch at most
constexpr int kSmallWords = kSmallSteps / 64;
constexpr int kSmallScen = 256;          // scenarios at most: one workgroup per CU
// Vehicles on the road up to which one workgroup is the faster way: two a thread, or three where it runs that many
// scenarios side by side (small_steps_ahead says how many there are expected to be).  us a step, the four launches
// and the one, 1,000 and 1,100 vehicles: 10x10 grid 22.2 and 20.9, 22.5 and 24.9; 16x16 streets of one lane 18.9 and
// 15.1, 19.3 and 18.3; 6x6 of three lanes 21.9 and 19.5, 21.7 and 23.6; a ring of 16 km 17.4 and 12.9, 17.2 and
// 15.9; at 2,900 it takes twice their time.  32 grids of 1,000 and of 1,200: 25.5 and 22.5, 25.4 and 26.9; 64 of 1,400
// and of 1,600 (two tiles): 29.8 and 27.3, 32.8 and 37.7; 128 of 1,400: 34.1 and 27.9.
constexpr int kSmallActive = 2 * kSmallNT;
constexpr int kSmallActiveMany = 3 * kSmallNT;
constexpr int kSmallMany = 64;

struct SmallRange {                      // what scenario k owns starts here (and ends at the next one's)
    int edge, lane, queue, node, veh;
};

struct Small {
    int n_scen;
    const SmallRange* range;             // [n_scen + 1]
    const int* due;                      // [n_scen][due_stride]: own vehicles with departure step <= t
    int due_stride;
    const int* q0;                       // first index of each departure queue
    Slots extra;                         // ensembles: the last step's layout, scenario k at its first vehicle
    int* n;                              // ensembles: [n_scen] vehicles after the run, then the step reached
    unsigned long long* moved;           // ensembles: [n_scen][kSmallWords] steps in which a vehicle moved
    unsigned long long* active;          //   and steps that began with one
    int* late;                           // ensembles: [n_scen][kSmallSteps] vehicles due less those that have departed
    unsigned long long* road;            // host memory: [n_scen] vehicles on the road after the launch | step << 32
                                         //   (null: not wanted)
    int cap, lanes, nodes;               // tile capacity (a multiple of 4), and the tables' entries in LDS
};

// LDS of the tables behind the tile: 64 bytes a lane, 8 a node
__host__ __device__ inline size_t small_table_bytes(int lanes, int nodes) {
    return (size_t)lanes * (sizeof(LaneRear) + sizeof(LanePost) + 8 + 6 * 4) + (size_t)nodes * 8;
}

__device__ inline Slots slots_at(const Slots& s, int o) {
    return Slots{s.x + o, s.v + o, s.vid + o, s.edge + o, s.meta + o, s.nxt + o, s.gl + o, s.lim ? s.lim + o : nullptr};
}

// first slot of [0, n) on edge e or a later one
__device__ inline int first_slot_of(const int32_t* edge, int n, int e) {
    int lo = 0, hi = n;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (edge[mid] < e) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// what the kernels of the next step expect to find cleared
__device__ inline void small_end_step(const Dev& d, int t) {
    d.ctl->t_a = t;
    d.ctl->t_b = t - 1;
    d.ctl->n_big[0] = d.ctl->n_big[1] = 0;
    d.ctl->big_done = 0;
    d.ctl->n_defer = 0;
    for (int k = 0; k < 2 * kTileGroups; ++k) tile_counters(d)[k * kTileCtrStride] = 0;
}

template <int NT, bool kSpread>
__global__ void __launch_bounds__(NT) k_small_steps(Dev d, Small sm, int nsteps) {
    extern __shared__ __align__(16) char lds[];
    __shared__ Totals wsh3[NT / 64];
    __shared__ int wsh[2 * (NT / 64)];
    __shared__ unsigned shc[cNumCounters];
    __shared__ ClassParams scp[16];
    __shared__ float slen[16];
    __shared__ uint16_t dlist[2 * NT], dfresh[kSpread ? 2 * NT : 1];
    __shared__ int dcount[3];
    __shared__ int smoved, sdep, stot, sreq, shead;
    const int tid = threadIdx.x, k = blockIdx.x;
    const DrawQ dq{dlist, dcount, 2 * NT, dfresh};
    const SmallRange r0 = sm.range[k], r1 = sm.range[k + 1];
    const int nl = r1.lane - r0.lane;
    // the tile, where the exits of a step and its claiming queues are kept once its tiles are done; then the lanes' tables
    LaneTabs tb;
    char* p = lds + (size_t)sm.cap * kTileBytesPerVeh + 64;
    tb.rear = (LaneRear*)p;
    p += sizeof(LaneRear) * (size_t)sm.lanes;
    tb.post = (LanePost*)p;
    p += sizeof(LanePost) * (size_t)sm.lanes;
    tb.win = (unsigned long long*)p;
    p += 8 * (size_t)sm.lanes;
    tb.win_node = (unsigned long long*)p;
    p += 8 * (size_t)sm.nodes;
    tb.req_stamp = (int*)p;
    tb.exit_stamp = tb.req_stamp + sm.lanes;
    tb.enter_stamp = tb.exit_stamp + sm.lanes;
    tb.lane_off = tb.enter_stamp + sm.lanes;
    tb.lane_newcnt = tb.lane_off + sm.lanes;
    tb.req_list = tb.lane_newcnt + sm.lanes;
    tb.n_req = &sreq;
    tb.lane0 = r0.lane;
    tb.node0 = r0.node;
    const Exits ex{(uint32_t*)(lds + 8 * (size_t)sm.lanes), (double*)lds, (uint32_t*)(lds + 12 * (size_t)sm.lanes)};
    int* const heads = (int*)(lds + 16 * (size_t)sm.lanes);

    if (tid < cNumCounters) shc[tid] = 0;
    if (tid < 3) dcount[tid] = 0;
    if (tid == 0) smoved = sdep = sreq = shead = 0;
    if (tid < 16) {
        scp[tid] = d.cp[tid];
        slen[tid] = d.cp[tid].len;
    }
    for (int i = tid; i < nl; i += NT) {
        tb.rear[i] = d.rear[r0.lane + i];
        tb.post[i] = LanePost{-1, 0, 0, 0.0f};
        tb.win[i] = ~0ull;
        tb.req_stamp[i] = tb.exit_stamp[i] = tb.enter_stamp[i] = -1;
    }
    for (int i = tid; i < sm.nodes; i += NT) tb.win_node[i] = ~0ull;
    const StepHead sh = step_head(d.ctl);
    const int t0 = sh.t_a, par0 = t0 & 1;
    const int n_all = par0 ? sh.n1 : sh.n0;
    const bool alone = sm.n_scen == 1;
    const int a0 = alone ? 0 : first_slot_of(d.s[par0].edge, n_all, r0.edge);
    int n = (alone ? n_all : first_slot_of(d.s[par0].edge, n_all, r1.edge)) - a0;
    // A scenario with nothing on the road still loads the first slot of its layout (scatter_load_record, dropped):
    // behind every vehicle there is none, and it takes the last there is.
    const int slot_max = max(d.n_veh - 1, 0), v0 = min(r0.veh, slot_max);
    __syncthreads();
    // vehicles that have left the departure queues
    int dep = 0;
    for (int q = r0.queue + tid; q < r1.queue; q += NT) dep += d.qhead[q] - sm.q0[q];
    if (dep) atomicAdd(&sdep, dep);
    __syncthreads();
    const int dep0 = sdep;
    dep = dep0;
    __syncthreads();
    if (tid == 0) sdep = 0;
    CounterAcc acc;
    acc.zero();
    unsigned long long act_sum = 0, denied = 0, grid_steps = 0, mv_bits = 0, ac_bits = 0;
    int run = alone ? d.ctl->stall_run : 0;
    Slots S = slots_at(d.s[par0], min(a0, slot_max));
    for (int j = 0; j < nsteps; ++j) {
        const int t = t0 + j;
        // an ensemble's scenarios write no buffer that another may still read as its first layout
        const Slots B = alone ? d.s[(t + 1) & 1] : slots_at((nsteps - 1 - j) & 1 ? d.s[par0 ^ 1] : sm.extra, v0);
        if (d.trace && tid == 0) d.nact_hist[t % d.trace_period] = n;
        tile_pieces<NT, kSpread, false>(d, tb, S, lds, sm.cap, 0, n, t, acc, wsh3, wsh, scp, dq, &smoved);
        for (int i = tid; i < nl; i += NT) {       // (the tile's space is free after its last barrier)
            ex.vid[i] = ~0u;
            ex.n[i] = 0u;
        }
        // admission: the listed requests, and the due queue heads, which are listed where they claim a lane
        const int nr = sreq;
        for (int i = tid; i < nr; i += NT) admit_request<false>(d, tb, S, tb.req_list[i], t);
        for (int q = r0.queue + tid; q < r1.queue; q += NT) {
            const int2 hd = d.qhd[q];
            if (hd.x <= t && admit_head<false>(d, tb, q, hd, t)) heads[atomicAdd(&shead, 1)] = q;
        }
        __syncthreads();
        // commit: the requests, and from the next wavefront on the heads whose key won their lane (in case 1 this
        // node's crossing into it comes first)
        const int h0 = (nr + 63) & ~63, nh = shead;
        for (int i = tid; i < h0 + nh; i += NT) {
            if (i < nr) {
                const int gl = tb.req_list[i];
                const uint32_t le = d.lane_edge[gl];
                const bool out = commit_request(d, tb, S, gl, (int)(le & kLaneEdgeMask), (int)(le >> kLaneEdgeBits),
                                                gl - r0.lane, t, acc, ex, &smoved);
                if (d.imode == 1 && out) {
                    const int target = d.outbox[gl].target;
                    if (target >= 0) tb.enter_stamp[target - r0.lane] = t;
                }
            } else if (i >= h0) {
                const int q = heads[i - h0], gl = d.qlane[q];
                const unsigned long long w = tb.win[gl - r0.lane];
                if ((w >> 63) && (int)(uint32_t)w == d.qhd[q].y) {
                    const uint32_t le = d.lane_edge[gl];
                    const int e = (int)(le & kLaneEdgeMask);
                    if (!crossing_into(d, tb, e, gl)) {
                        commit_departure(d, tb, gl, e, (int)(le >> kLaneEdgeBits), t, acc, &smoved);
                        atomicAdd(&sdep, 1);
                    }
                }
            }
        }
        __syncthreads();
        for (int i = tid; i < nr; i += NT) {
            const int gl = tb.req_list[i], li = gl - r0.lane;
            if (ex.vid[li] != ~0u) {
                const uint32_t le = d.lane_edge[gl];
                commit_travel_time<false>(d, (int)(le & kLaneEdgeMask), (int)(le >> kLaneEdgeBits), li, ex);
            }
        }
        // the lanes of the next layout
        int nnew = 0;
        for (int i0 = 0; i0 < nl; i0 += NT) {
            const int i = i0 + tid;
            int c = 0;
            if (i < nl) {
                const LanePost p = tb.post[i];
                c = (p.stamp == t ? p.cnt : 0) - (tb.exit_stamp[i] == t ? 1 : 0) + (tb.enter_stamp[i] == t ? 1 : 0);
                tb.lane_newcnt[i] = c;
            }
            const int o = nnew + wg_exclusive_sum<NT>(c, wsh);
            if (i < nl) tb.lane_off[i] = o;
            if (tid == NT - 1) stot = o + c;
            __syncthreads();
            nnew = stot;
        }
        for (int i = tid; i < max(n, nl); i += NT) {
            ScatterItem r;
            scatter_load_record<kSpread>(S, i < n ? i : -1, r);
            scatter_load_tables(d, tb, i < nl && tb.enter_stamp[i] == t ? r0.lane + i : -1, r);
            scatter_store<kSpread>(d, tb, B, r, nnew, t, slen, [](int) { return 0; });
        }
        if (d.imode == 1)
            for (int i = tid; i < sm.nodes; i += NT) tb.win_node[i] = ~0ull;
        if (tid == 0) {
            act_sum += (unsigned long long)n;
            dep += sdep;
            sdep = sreq = shead = 0;
            const int due = d.max_dep < 0 ? 0 : sm.due[(size_t)k * sm.due_stride + min(t, d.max_dep)];
            if (alone) denied += due > dep ? (unsigned long long)(due - dep) : 0ull;
            else sm.late[(size_t)k * kSmallSteps + j] = due - dep;   // (counted over all scenarios, k_small_gather)
            const bool mv = smoved != 0;
            smoved = 0;
            if (alone) {
                run = n > 0 && !mv ? run + 1 : 0;
                grid_steps += run >= kGridlockSteps ? 1ull : 0ull;
            } else {
                mv_bits |= (unsigned long long)mv << (j & 63);
                ac_bits |= (unsigned long long)(n > 0) << (j & 63);
                if ((j & 63) == 63 || j == nsteps - 1) {
                    sm.moved[(size_t)k * kSmallWords + (j >> 6)] = mv_bits;
                    sm.active[(size_t)k * kSmallWords + (j >> 6)] = ac_bits;
                    mv_bits = ac_bits = 0;
                }
            }
        }
        __syncthreads();
        n = nnew;
        S = B;
    }
    for (int i = tid; i < nl; i += NT) d.rear[r0.lane + i] = tb.rear[i];
    if (tid == 0) {
        atomicAdd(&d.counters[cActiveSum * kCounterCopies], act_sum);
        if (denied) atomicAdd(&d.counters[cInsertDenied * kCounterCopies], denied);
        atomicAdd(&d.ctl->n_departed, dep - dep0);
        if (sm.road) sm.road[k] = (unsigned long long)(uint32_t)(t0 + nsteps) << 32 | (uint32_t)n;
        if (alone) {
            if (grid_steps) d.counters[cGridlock * kCounterCopies] += grid_steps;
            d.ctl->stall_run = run;
            d.ctl->n_act[(t0 + nsteps) & 1] = n;
            small_end_step(d, t0 + nsteps);
        } else {
            sm.n[k] = n;
            if (k == 0) sm.n[sm.n_scen] = t0 + nsteps;
        }
    }
    flush_counters_lds(d, acc, shc);
}

// Ensembles: the scenarios' last layouts, one after another, and the end of
// the run (control block, gridlock detector and refused departures over all
// scenarios: a written state may have more departures than are due in one).
__global__ void __launch_bounds__(kSmallNT) k_small_gather(Dev d, Small sm, int nsteps) {
    __shared__ int scnt[kSmallScen + 1];
    __shared__ unsigned long long smv[kSmallWords], sac[kSmallWords];
    __shared__ int slate[kSmallSteps];
    const int tid = threadIdx.x, k = blockIdx.x;
    for (int i = tid; i < sm.n_scen; i += kSmallNT) scnt[i] = sm.n[i];
    if (tid < kSmallWords) smv[tid] = sac[tid] = 0;
    for (int j = tid; j < nsteps; j += kSmallNT) slate[j] = 0;
    __syncthreads();
    int o = 0, total = 0;
    for (int i = 0; i < sm.n_scen; ++i) {
        if (i == k) o = total;
        total += scnt[i];
    }
    const int t = sm.n[sm.n_scen];
    const Slots A = slots_at(sm.extra, sm.range[k].veh), B = slots_at(d.s[t & 1], o);
    for (int i = tid; i < scnt[k]; i += kSmallNT) {
        B.x[i] = A.x[i];
        B.v[i] = A.v[i];
        B.vid[i] = A.vid[i];
        B.edge[i] = A.edge[i];
        B.meta[i] = A.meta[i];
        B.nxt[i] = A.nxt[i];
        if (d.v0_spread != 0.0f) B.lim[i] = A.lim[i];
    }
    if (k != 0) return;
    const int nw = (nsteps + 63) / 64;
    for (int i = tid; i < sm.n_scen * nw; i += kSmallNT) {
        const int s = i / nw, w = i % nw;
        atomicOr(&smv[w], sm.moved[(size_t)s * kSmallWords + w]);
        atomicOr(&sac[w], sm.active[(size_t)s * kSmallWords + w]);
    }
    for (int i = tid; i < sm.n_scen * nsteps; i += kSmallNT) {
        const int s = i / nsteps, j = i % nsteps;
        atomicAdd(&slate[j], sm.late[(size_t)s * kSmallSteps + j]);
    }
    __syncthreads();
    unsigned long long denied = 0;
    for (int j = tid; j < nsteps; j += kSmallNT) denied += (unsigned long long)max(slate[j], 0);
    if (denied) atomicAdd(&d.counters[cInsertDenied * kCounterCopies], denied);
    if (tid != 0) return;
    int run = d.ctl->stall_run;
    unsigned long long grid_steps = 0;
    for (int w = 0; w < nw; ++w) {
        const int m = min(64, nsteps - 64 * w);
        const unsigned long long all = m == 64 ? ~0ull : (1ull << m) - 1ull;
        const unsigned long long stalled = sac[w] & ~smv[w] & all;
        if (stalled == 0ull) {
            run = 0;
            continue;
        }
        for (int j = 0; j < m; ++j) {
            run = (stalled >> j) & 1ull ? run + 1 : 0;
            grid_steps += run >= kGridlockSteps ? 1ull : 0ull;
        }
    }
    if (grid_steps) d.counters[cGridlock * kCounterCopies] += grid_steps;
    d.ctl->stall_run = run;
    d.ctl->n_act[t & 1] = total;
    small_end_step(d, t);
}

// ---- the reverse sweep of a small network --------------------------------------
// The steps [0, steps) of a traced segment, last first, in one launch of one
// workgroup (k_backward, k_bw_looks and k_bw_gather as phases between workgroup
// barriers: three launches a step take 32 us on the 10x10 grid, whose 370
// records are one a thread).  The adjoints are updated in place: a vehicle's are
// read by its own record and written after that, and one that was not yet on the
// road is never read again.  The lists of look-ahead records are in LDS, the
// parts in device memory, gpart: [5 * n_classes][kSmallBwNT], each thread's own.
constexpr int kSmallBwNT = 512;
// Vehicles on the road at most, on average over the run.  The re-run and the sweep of 1,200 steps with 700, 1,150, 1,350
// and 1,700 on the road, three kernels a step 50, 52, 53 and 54 ms, in one workgroup 34, 45, 51 and 62.
constexpr int kSmallBwActive = 1536;

template <int NC>
__global__ void __launch_bounds__(kSmallBwNT) k_small_backward(Dev d, const TraceRec* trace, size_t stride,
                                                              const int* nact, int steps, int n_classes, double* lx,
                                                              double* lv, double* lt, const double* w, BwPart* part,
                                                              double* gpart) {
    __shared__ int lk_cnt[kSmallLanes];
    __shared__ int lk_rec[kSmallLanes * kLookListCap];
    __shared__ double lk_x[kSmallLanes], lk_v[kSmallLanes];
    const EdgeC last = d.ec[d.n_edges - 1];
    const int tid = threadIdx.x, nl = min(last.lane_base + last.lanes, kSmallLanes), np = 5 * n_classes;
    ParamGrad<NC> acc{};
#pragma unroll
    for (int k = 0; k < 5 * NC; ++k)
        if (k < np) acc.g[k] = gpart[k * kSmallBwNT + tid];
    for (int g = tid; g < nl; g += kSmallBwNT) lk_cnt[g] = 0;
    __syncthreads();
    for (int i = steps - 1; i >= 0; --i) {
        const TraceRec* rec = trace + (size_t)i * stride;
        const int n = nact[i];
        for (int r = tid; r < n; r += kSmallBwNT) {
            const TraceRec R = rec[r];
            const BwRecord o = backward_record(d, R, lx, lv, lt, w);
            part[r] = o.part;
            acc.add(o);
            if (follows(R) && (r == 0 || (int)rec[r - 1].vid != R.partner)) atomicOr(&d.ctl->err, kErrTrace);
            if (looks_ahead(R)) {
                const int k = atomicAdd(&lk_cnt[R.look_gl], 1);
                if (k < kLookListCap) lk_rec[R.look_gl * kLookListCap + k] = r;
                else atomicOr(&d.ctl->err, kErrTrace);
            }
        }
        __syncthreads();
        // own part and the follower's; meanwhile the lanes' look-ahead sums, in record order
        for (int r = tid; r < n; r += kSmallBwNT) {
            const int v = (int)rec[r].vid;
            const BwPart P = part[r];
            double ax = P.sx, av = P.sv;
            if (r + 1 < n) {
                const TraceRec F = rec[r + 1];
                if (F.partner == v && follows(F)) {
                    const BwPart Q = part[r + 1];
                    ax += Q.px;
                    av += Q.pv;
                }
            }
            lx[v] = ax;
            lv[v] = av;
        }
        for (int g = tid; g < nl; g += kSmallBwNT) {
            const int m = min(lk_cnt[g], kLookListCap);
            double sx = 0.0, sv = 0.0;
            for (int k = 0, from = 0; k < m; ++k) {
                int next = INT_MAX;
                for (int q = 0; q < m; ++q) {
                    const int r = lk_rec[g * kLookListCap + q];
                    if (r >= from) next = min(next, r);
                }
                sx += part[next].px;
                sv += part[next].pv;
                from = next + 1;
            }
            lk_x[g] = sx;
            lk_v[g] = sv;
        }
        __syncthreads();
        for (int g = tid; g < nl; g += kSmallBwNT)
            if (lk_cnt[g] > 0) {
                const int v = rec[lk_rec[g * kLookListCap]].partner;   // the lane's rear, the partner of all of them
                lx[v] += lk_x[g];
                lv[v] += lk_v[g];
                lk_cnt[g] = 0;
            }
        __syncthreads();
    }
#pragma unroll
    for (int k = 0; k < 5 * NC; ++k)
        if (k < np) gpart[k * kSmallBwNT + tid] = acc.g[k];
}

}  // namespace manta
