// group.h -- the persistent iteration of a mid-sized instance: a group of
// workgroups that stays resident runs every iteration of a call in one
// launch, with one barrier between its workgroups per iteration.
// Internal: included by twa.hip inside its unnamed namespace (it runs the
// per-factor device code defined there).
//
// Three launches per iteration cost such an instance more than its work: the
// launches themselves, and in each of them cold instruction and scalar
// caches and a chain of dependent loads (queue lengths, entry, factor
// position, records) before a minimiser can start.  Here every workgroup
// keeps
//   - its own copy of all node records in LDS (last iteration's too in the
//     dense form, whose test of last iteration's activity reads them),
//   - its share of the factors for the whole launch: (column, break-point
//     interval block) items of the collision walk, a range of wall factors,
//     a range of energy and fixed factors, with their activity bits in LDS,
//   - its own work queue in LDS.
// An iteration is: test the share's collision and wall factors on the LDS
// records, run the minimisers of the queued ones and the energy and fixed
// factors, add the contributions to the consensus sums in global memory
// (the same exact integer atomics as everywhere, so neither the partition
// nor the order changes a bit), barrier, then every workgroup computes all
// new node records into its own LDS copy.  The sums rotate over three
// buffers: the one read after barrier t is cleared after barrier t + 1, when
// every member has read it, and written again from iteration t + 3 on; so
// one barrier per iteration is enough.
//
// No barrier waits for a workgroup that does not run yet.  Workgroups register;
// the first one waits for the rest, for a bounded time (see group_join), and
// then freezes the group at whoever came.  Later workgroups see
// the frozen mark and leave, the members share out all the shares.  No
// assumption about residency or dispatch order is needed for progress or for
// the result (fewer members are just slower).
//
// What bounds an iteration: the chain of latencies of one wave (100-agent
// swap, 461 queued factors, 32 members, 24 k cycles = 10.4 us against 19.5 us
// in three launches): tests 6 k, minimisers 8.5 k and their contributions 2.5 k,
// barrier 2 k and waiting for the slowest member 4 k, node records 2.2 k.
// 512 lanes: 256 made the walk slower (12 us), 1024 nothing faster.  Two
// intervals per item: four measured the same on this instance, 9.0 against
// 8.3 us on 32 agents; eight 10.8 us.
//
// Data that members exchange (sums, counts, barrier, totals) moves by
// agent-scope atomics only, each complete before its workgroup arrives at the
// barrier, so no cache is written back or invalidated.
#pragma once

constexpr int kGroupBlock = 512;      // lanes per workgroup of one instance's group
constexpr int kGroupBatchBlock = 256; // and of a batch's groups, two or more of which share a compute unit
constexpr int kGroupMinChunk = 16;    // least entries a wave takes from the collision queue

// An item of the walk covers kGroupCpw intervals of one row's chunk, or, in a
// batch's groups (cyclic), of kGroupSpan offsets d, 1 <= d <= p / 2, of the 64
// agents i = 64 b + lane: pairs i, i + d (mod p), every pair once (d = p / 2 of an
// even p from its lower half).  There lanes stay full where the rows of the pair
// triangle leave half of them idle (68 agents: 68 chunks of 64 lanes instead of
// 130): 256 instances 48 us per iteration instead of 69.  An instance with a
// group to itself has few items per wave, and the walk is short beside the
// minimisers: there the rows, whose words are the solver's own, are as fast or
// faster (32 agents 8.3 us per iteration against 8.8, 64 agents 9.0 against 9.4).
constexpr bool group_cyclic(int T) { return T == kGroupBatchBlock; }
// activity words of an item
constexpr int group_words(int T) { return (group_cyclic(T) ? kGroupSpan : 1) * kGroupCpw; }
// items per block of intervals
__host__ __device__ __forceinline__ int group_items(int p, int cps, int T) {
    return group_cyclic(T) ? cyclic_items(p) : cps;
}

// entries of the LDS queues of a workgroup of T lanes
constexpr int group_queue(int T) { return (T == kGroupBatchBlock ? 12 : 16) * T; }
constexpr int group_wall_queue(int T) { return 2 * T; }

// Queue length from which a wave sums the contributions to equal nodes before
// the atomics: the shuffles cost a short queue 1 us, the atomics on the same
// nodes a crowded one more (start of the 100-agent swap 22 against 17 us per
// iteration, ADMM of 32 agents 20 against 10.4).
constexpr int kGroupSums = 64;
constexpr unsigned kGroupFrozen = 0x80000000u;

// Shared words of a group, each on a line of its own where it is polled.
struct GroupCtl {
    unsigned reg, pad0[31];  // workgroups that came; bit 31 once the group is frozen
    unsigned size, pad1[31]; // members (0 until frozen)
    unsigned bar, pad2[31];  // barrier arrivals
    unsigned total[3];       // last iteration: active collision, active wall, queued factors
    unsigned pad3[29];
    unsigned turn;           // buffer the next iteration adds to (kept between launches)
    unsigned stuck;          // a wait ran out (never, short of a fault): results invalid from here on
};

// byte offsets in the dynamic LDS
struct GroupLds {
    unsigned zc, zp, rad, item, word, wbit, q, qw;
    int items, walls32; // items and 32-factor wall units of the largest share
};

struct GroupArgs {
    GroupCtl *ctl;
    unsigned long long *acc; // [3][dim][N]
    int *cnt;                // [3][N]
    unsigned long long *words; // the shares' activity words, where a member runs several
    float *xe;               // [Fe][2 * dim] x of the per-segment factors, last iteration; [p][dim] of a
                             // velocity-obstacle epoch's goal factors
    unsigned char *sent;     // [Fe] whether they sent rho0
    GroupLds L;
    int want;                // shares, and workgroups that may join
    int stride;              // every stride-th workgroup of the launch belongs to the group
    int K;
};

__device__ __forceinline__ unsigned agent_load(const unsigned *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A wait gives up after this many polls (ten seconds or so): a member that
// left abnormally must not hang the device.  The first one to give up says so
// in `stuck`, which every wait looks at now and then: the rest of the launch
// ends without waiting that long again, and later launches end at once.  What
// the solver holds is invalid from then on, and whatever reads it says so
// (GaveUp).
constexpr unsigned kGroupPatience = 1u << 24;

__device__ __forceinline__ void group_give_up(GroupCtl *c) {
    __hip_atomic_store(&c->stuck, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Join the group for K iterations: members get their rank in *rank and the
// member count in *size; false for a workgroup that came too late, or where a
// wait ran out.
//
// A group that starts short stays short for all K iterations, however soon the
// card is free again, so the first member waits for the rest for as long as
// running without them would take longer: rounds of shares past the first, at
// kGroupRound each, and 50 us at least.  What is lost by not starting, or by
// starting and staying short, is then at most about the time that is needed
// anyway.  (On an idle card all are there within a few us.  256 agents and 32
// walls, 50 iterations, beside matrix products of 1 ms each on another stream:
// with a fixed wait of 50 us some launches started short and took 26-34 ms,
// now 1.9-2.7.)
constexpr unsigned long long kGroupRound = 1000; // 10 us of the 100 MHz wall clock
__device__ __forceinline__ bool group_join(GroupCtl *c, int want, int K, unsigned *rank, unsigned *size) {
    const unsigned stuck = agent_load(&c->stuck), r = atomicAdd(&c->reg, 1u);
    if (stuck || (r & kGroupFrozen)) return false;
    if (r == 0u) {
        const unsigned long long t0 = wall_clock64();
        unsigned m = 1u;
        for (unsigned n = 0; n < kGroupPatience / 8; ++n) {
            if ((m = agent_load(&c->reg)) >= (unsigned)want) break;
            const unsigned long long more = ((unsigned)want + m - 1u) / m - 1u;
            if (wall_clock64() - t0 > max(5 * kGroupRound, kGroupRound * K * more)) break;
            __builtin_amdgcn_s_sleep(1);
        }
        m = min(atomicOr(&c->reg, kGroupFrozen), (unsigned)want);
        __hip_atomic_store(&c->size, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *size = m;
    } else {
        unsigned m = 0u;
        for (unsigned n = 0; n < kGroupPatience && (m = agent_load(&c->size)) == 0u; ++n) __builtin_amdgcn_s_sleep(1);
        if (m == 0u) group_give_up(c);
        *size = m;
    }
    *rank = r;
    return r < *size;
}

// Barrier `n` (1, 2, ...) of the group.  Every memory operation of the
// workgroup's waves is complete before it arrives.  *gone (LDS) is set where
// the wait ran out, here or in another member.
__device__ __forceinline__ void group_barrier(GroupCtl *c, unsigned size, unsigned n, int *gone) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(&c->bar, 1u);
        const unsigned all = size * n;
        unsigned k = 0;
        while (agent_load(&c->bar) < all)
            if ((++k & 1023u) == 0u && (k >= kGroupPatience || agent_load(&c->stuck))) {
                group_give_up(c);
                *gone = 1;
                break;
            }
    }
    __syncthreads();
}

// A share of the factors: items sh, sh + want, ... of the collision walk;
// ranges of 32-factor wall units and of energy and fixed factors.
struct GroupShare {
    int nitems, u0, nu, nwall, e0, ne, f0, nf;
    __device__ __forceinline__ void take(const Params &P, int want, int sh, int nitems_all) {
        auto cut = [&](long long n, int k) { return (int)(n * k / want); };
        const int units = (int)((P.Fw + 31) / 32);
        nitems = (nitems_all - sh + want - 1) / want;
        u0 = cut(units, sh), nu = cut(units, sh + 1) - u0;
        nwall = (int)min(32LL * (u0 + nu), P.Fw) - 32 * u0;
        e0 = cut(P.Fe, sh), ne = cut(P.Fe, sh + 1) - e0;
        f0 = cut(P.Ff, sh), nf = cut(P.Ff, sh + 1) - f0;
    }
};

// wave-aggregated append to an LDS queue; all lanes call
__device__ __forceinline__ void group_push(unsigned *q, int *len, bool pred, unsigned val) {
    const unsigned long long mask = __ballot(pred);
    if (mask == 0ull) return;
    const int lane = __lane_id(), leader = __ffsll((long long)mask) - 1;
    int base = 0;
    if (lane == leader) base = atomicAdd(len, __popcll(mask));
    base = __shfl(base, leader);
    if (pred) q[base + __popcll(mask & ((1ull << lane) - 1ull))] = val;
}

// Goal factor of a velocity-obstacle epoch, as vo_goal_stream, with the x kept
// from the last iteration (first: computed again from its records).
template <int D>
__device__ __forceinline__ void group_vo_goal(const Params &P, const Rec &Z, const GroupArgs &A, long long f, bool first) {
    const int i = (int)(f >> 1);
    const long long nd = (long long)P.eta * P.p + i;
    const float C = P.C[i];
    const float4 xr = P.xfix[f];
    float *up = P.u_fixed + f * D, *xp = A.xe + P.Fe * 2 * D + (long long)i * D;
    float u[3], n[3], x[3], zc[3];
    for (int c = 0; c < D; ++c) u[c] = up[c], x[c] = xp[c];
    const float4 rc = Z.cur[nd];
    node_xyz(rc, zc, D);
    const int k = wcode(rc);
    if (first) {
        const float4 rp = P.zr_prev[nd];
        float zp[3];
        node_xyz(rp, zp, D);
        for (int c = 0; c < D; ++c) n[c] = zp[c] - u[c];
        vo_cost_prox<D>(xr, C, n, wcode(rp), P.rho_prev, x);
    }
    for (int c = 0; c < D; ++c) u[c] = (k == W_STD) ? u[c] + P.step_prev * (x[c] - zc[c]) : 0.f, up[c] = u[c];
    for (int c = 0; c < D; ++c) n[c] = zc[c] - u[c];
    vo_cost_prox<D>(xr, C, n, k, P.rho, x);
    for (int c = 0; c < D; ++c) xp[c] = x[c], x[c] = x[c] + u[c];
    contribute(P, nd, 0, x, D);
}

// Fixed factor f of the three-weight method: u resets to zero (its
// outgoing weight is infinite) and the node takes the constant itself, which
// group_nodes knows, so only the range check of the sums is left to do.
template <int D>
__device__ __forceinline__ void group_fixed(const Params &P, const Rec &Z, const GroupArgs &A, long long f, bool first) {
    if (P.vo && (f & 1) && !P.admm) {
        group_vo_goal<D>(P, Z, A, f, first);
        return;
    }
    if (P.admm) {
        fixed_stream<D, M_FUSED>(P, Z, f);
        return;
    }
    const float4 xf = P.xfix[f];
    const float x[3] = {xf.x, xf.y, xf.z};
    for (int c = 0; c < D; ++c) {
        P.u_fixed[f * D + c] = 0.f;
        if (!(fabsf((x[c] + 0.f) * P.scalef) <= P.sat_lim)) P.counters[5] = 1;
    }
}

// Per-segment factor f between break-points of the workgroup's records: the
// u update of the last iteration with the x kept from it (first: x computed
// again from last iteration's records, as energy_stream does every time), then
// x and the contributions of this one.
template <int D>
__device__ __forceinline__ void group_energy(const Params &P, const Rec &Z, const GroupArgs &A, long long f, bool first) {
    const int i = (int)f / P.eta, s = (int)f - i * P.eta;
    const long long na = (long long)s * P.p + i, nb = na + P.p;
    const float C = P.C[f];
    float *up = P.u_energy + f * 2 * D, *xp = A.xe + f * 2 * D;
    float u[2 * D], n[2 * D], x[2 * D], zc[2 * D];
    for (int q = 0; q < 2 * D; ++q) u[q] = up[q], x[q] = xp[q];
    bool sent = A.sent[f] != 0;
    const float4 ca = Z.cur[na], cb = Z.cur[nb];
    node_xyz(ca, zc, D);
    node_xyz(cb, zc + D, D);
    const int ka = wcode(ca), kb = wcode(cb);
    if (first) {
        const float4 pa = P.zr_prev[na], pb = P.zr_prev[nb];
        float zp[2 * D];
        node_xyz(pa, zp, D);
        node_xyz(pb, zp + D, D);
        for (int q = 0; q < 2 * D; ++q) n[q] = zp[q] - u[q];
        sent = segment_prox<D>(P, C, n, wcode(pa), wcode(pb), P.rho_prev, x);
    }
    for (int c = 0; c < D; ++c) {
        u[c] = (sent && ka == W_STD) ? u[c] + P.step_prev * (x[c] - zc[c]) : 0.f;
        u[D + c] = (sent && kb == W_STD) ? u[D + c] + P.step_prev * (x[D + c] - zc[D + c]) : 0.f;
    }
    for (int q = 0; q < 2 * D; ++q) up[q] = u[q], n[q] = zc[q] - u[q];
    const bool send = segment_prox<D>(P, C, n, ka, kb, P.rho, x);
    for (int q = 0; q < 2 * D; ++q) xp[q] = x[q];
    if (send != sent || first) A.sent[f] = send ? 1 : 0;
    if (send) {
        for (int q = 0; q < 2 * D; ++q) x[q] = x[q] + u[q];
        if (!fixed_node(P, s)) contribute(P, na, 0, x, D);
        if (!fixed_node(P, s + 1)) contribute(P, nb, 0, x + D, D);
    }
}

// All nodes: z and <-rho of the next iteration from the sums of buffer b,
// into the workgroup's own records (as node_update); those of [w0, w1) also
// into the solver's.
template <int D, bool DENSE, int T>
__device__ __forceinline__ void group_nodes(const Params &P, const GroupArgs &A, int b, float4 *zc, float4 *zp, int w0,
                                            int w1) {
    constexpr int U = 4;
    const int N = (int)P.N, goal0 = P.eta * P.p;
    const unsigned long long *acc = A.acc + (long long)b * D * N;
    const int *cnt = A.cnt + (long long)b * N;
    for (int n0 = threadIdx.x; n0 < N; n0 += U * T) {
        unsigned long long a[U][D];
        int c[U];
        float4 fx[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int nd = n0 + k * T;
            c[k] = 0;
            if (nd < N) {
                if (!P.admm && (nd < P.p || (nd >= goal0 && !P.vo))) {
                    fx[k] = P.xfix[nd < P.p ? 2 * nd : 2 * (nd - goal0) + 1];
                    c[k] = -1;
                } else {
                    c[k] = __hip_atomic_load(&cnt[nd], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    for (int d = 0; d < D; ++d)
                        a[k][d] = __hip_atomic_load(&acc[(long long)d * N + nd], __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int nd = n0 + k * T;
            if (nd < N) {
                const float4 cur = zc[nd];
                float4 nw = cur;
                if (c[k] < 0) {
                    nw.x = fx[k].x + 0.f, nw.y = fx[k].y + 0.f;
                    if (D == 3) nw.z = fx[k].z + 0.f;
                    nw.w = (float)W_INF;
                } else if (c[k] > 0) {
                    const double den = (double)c[k] * P.scale;
                    nw.x = (float)((double)(long long)a[k][0] / den);
                    nw.y = (float)((double)(long long)a[k][1] / den);
                    if constexpr (D == 3) nw.z = (float)((double)(long long)a[k][2] / den);
                    nw.w = (float)W_STD;
                } else {
                    nw.w = (float)W_ZERO;
                }
                if (DENSE) zp[nd] = cur;
                zc[nd] = nw;
                if (nd >= w0 && nd < w1) P.zr_prev[nd] = cur, P.zr_cur[nd] = nw;
            }
        }
    }
}

// The activity tests of one item of the walk (packed s0, b, d0 or s0, i, 64 J), its
// factors to queue appended to q as (item and word) << 6 | lane.
template <int D, bool DENSE, int T>
__device__ __forceinline__ void group_item(const Params &P, const Rec &Z, unsigned long long item, int l, int lane,
                                           const float *rad, unsigned long long *word, unsigned *q, int *len) {
    constexpr int NS = kGroupCpw, WORDS = group_words(T);
    static_assert(!DENSE || !group_cyclic(T), "the cyclic walk is of the activity-bit form");
    const unsigned long long pk = uniform64(item);
    const int s0 = (int)(pk >> 48), ns = min(NS, P.eta - s0), p = P.p;
    // the lanes of the masks into the queue, as entries of the words from w on
    auto append = [&](const unsigned long long (&queue)[NS], const unsigned long long (&prev)[NS], int w) {
        const unsigned long long me = 1ull << lane;
        int n = 0;
#pragma unroll
        for (int k = 0; k < NS; ++k) n += __popcll(queue[k]);
        if (n == 0) return;
        int base = 0;
        if (lane == 0) base = atomicAdd(len, n);
        base = __builtin_amdgcn_readfirstlane(base);
#pragma unroll
        for (int k = 0; k < NS; ++k) {
            if (queue[k] & me)
                q[base + __popcll(queue[k] & (me - 1ull))] =
                    ((prev[k] & me) ? kPrev : 0u) | (unsigned)((l * WORDS + w + k) << 6) | (unsigned)lane;
            base += __popcll(queue[k]);
        }
    };
    if constexpr (!group_cyclic(T)) {
        const int i0 = (int)((pk >> 24) & 0xffffffull), j = (int)(pk & 0xffffffull) + lane, jj = min(j, p - 1);
        const float4 *c = Z.cur + s0 * p;
        const float R = rad[i0] + rad[jj];
        const bool valid = j > i0 && j < p;
        unsigned long long queue[NS], prev[NS];
        if constexpr (!DENSE) {
            // (an inactive factor's u is zero, so its n is z)
            float4 ri[NS + 1], rj[NS + 1];
#pragma unroll
            for (int k = 0; k <= NS; ++k) ri[k] = c[min(k, ns) * p + i0], rj[k] = c[min(k, ns) * p + jj];
            cpa_masks<D, NS>(ri, rj, R * R, queue);
            const unsigned long long all = __builtin_amdgcn_ballot_w64(valid);
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                prev[k] = uniform64(word[l * NS + k]);
                queue[k] = k < ns ? (queue[k] & all) | prev[k] : 0ull;
            }
            if (lane < NS) word[l * NS + lane] = 0ull;
        } else {
            const float4 *pr = Z.prev + s0 * p;
            const unsigned fr = (unsigned)((long long)i0 * (2 * p - i0 - 1) / 2 + (j - i0 - 1)), P2 = (unsigned)P.P2;
            float u[NS][4 * D];
#pragma unroll
            for (int k = 0; k < NS; ++k)
                if (k < ns && valid) load_u_coll<D>(P, (unsigned)(s0 + k) * P2 + fr, u[k]);
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                bool go = false;
                unsigned val = 0u;
                if (k < ns && valid) {
                    const float4 rc[4] = {c[k * p + i0], c[(k + 1) * p + i0], c[k * p + jj], c[(k + 1) * p + jj]};
                    const float4 rp[4] = {pr[k * p + i0], pr[(k + 1) * p + i0], pr[k * p + jj], pr[(k + 1) * p + jj]};
                    go = coll_factor<D, M_FUSED, true>(P, (unsigned)(s0 + k) * P2 + fr, R, rc, rp, u[k], 0ull, lane, &val);
                }
                queue[k] = __builtin_amdgcn_ballot_w64(go);
                prev[k] = __builtin_amdgcn_ballot_w64((val & kPrev) != 0u);
            }
        }
        append(queue, prev, 0);
    } else {
        // (the test does not depend on which of the two agents comes first)
        const int b = (int)((pk >> 24) & 0xffffffull), d0 = (int)(pk & 0xffffffull);
        const int i = 64 * b + lane, ii = min(i, p - 1), x0 = s0 * p;
        const float radi = rad[ii];
        float4 ri[NS + 1];
#pragma unroll
        for (int k = 0; k <= NS; ++k) ri[k] = Z.cur[x0 + min(k, ns) * p + ii];
        const unsigned long long mword = lane < WORDS ? word[l * WORDS + lane] : 0ull;
        if (lane < WORDS) word[l * WORDS + lane] = 0ull;
        const unsigned long long all = p - 64 * b < 64 ? (1ull << (p - 64 * b)) - 1ull : ~0ull;
        const int spans = min(kGroupSpan, p / 2 - d0 + 1);
#pragma unroll 1
        for (int r = 0; r < spans; ++r) {
            const int d = d0 + r;
            const int j = ii + d >= p ? ii + d - p : ii + d;
            const float R = radi + rad[j];
            float4 rj[NS + 1];
#pragma unroll
            for (int k = 0; k <= NS; ++k) rj[k] = Z.cur[x0 + min(k, ns) * p + j];
            unsigned long long queue[NS], prev[NS];
            cpa_masks<D, NS>(ri, rj, R * R, queue);
            const unsigned long long valid = 2 * d == p ? all & __builtin_amdgcn_ballot_w64(i < d) : all;
#pragma unroll
            for (int k = 0; k < NS; ++k) {
                prev[k] = lane_value(mword, r * NS + k);
                queue[k] = k < ns ? (queue[k] & valid) | prev[k] : 0ull;
            }
            append(queue, prev, r * NS);
        }
    }
}

// K iterations of the instance by member `rank` of `size`.
template <int D, bool DENSE, int T>
__device__ __forceinline__ void group_run(Params P, const GroupArgs &A, char *lds, unsigned rank, unsigned size) {
    constexpr int CPW = kGroupCpw;
    // known here, so that the code below carries no trace of the rest
    P.dense = DENSE ? 1 : 0;
    if (!DENSE) P.admm = 0;
    P.dbg_x = nullptr, P.dbg_rho = nullptr, P.adj_pool = nullptr;
    P.rho_prev = P.rho, P.step_prev = P.step;
    const int lane = threadIdx.x & 63, wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int N = (int)P.N, p = P.p;
    float4 *zc = reinterpret_cast<float4 *>(lds + A.L.zc), *zp = reinterpret_cast<float4 *>(lds + A.L.zp);
    float *rad = reinterpret_cast<float *>(lds + A.L.rad);
    unsigned long long *item = reinterpret_cast<unsigned long long *>(lds + A.L.item);
    unsigned long long *word = reinterpret_cast<unsigned long long *>(lds + A.L.word);
    unsigned *wbit = reinterpret_cast<unsigned *>(lds + A.L.wbit);
    unsigned *q = reinterpret_cast<unsigned *>(lds + A.L.q), *qw = reinterpret_cast<unsigned *>(lds + A.L.qw);
    // queue lengths; iteration + 1 where some wave has items left; whether a
    // wait ran out (read together, once a round)
    __shared__ int len[4];
    __shared__ unsigned totals[3];   // this iteration's active and queued factors
    for (int nd = threadIdx.x; nd < N; nd += T) {
        zc[nd] = P.zr_cur[nd];
        if (DENSE) zp[nd] = P.zr_prev[nd];
    }
    for (int i = threadIdx.x; i < p; i += T) rad[i] = P.radii[i];
    if (threadIdx.x < 4) len[threadIdx.x] = 0;
    if (threadIdx.x < 3) totals[threadIdx.x] = 0u;
    P.radii = rad;
    constexpr bool CYC = group_cyclic(T);
    constexpr int WORDS = group_words(T);
    const int cps = (int)P.cps, nsb = (P.eta + CPW - 1) / CPW;
    const int per = group_items(p, cps, T);
    const int nitems_all = per * nsb;
    GroupShare S;
    const unsigned P2 = (unsigned)P.P2;
    const unsigned turn = agent_load(&A.ctl->turn);
    const bool many = size < (unsigned)A.want; // a member runs several shares in turn
    const int n0 = (int)((long long)N * rank / size), n1 = (int)((long long)N * (rank + 1) / size);
    const Rec Z{zc, zp};
    const int spans = max(1, (p / 2 + kGroupSpan - 1) / kGroupSpan);
    auto take_items = [&](int sh) {
        for (int l = threadIdx.x; l < S.nitems; l += T) {
            const int g = l * A.want + sh, sb = g / per, m = g - sb * per;
            item[l] = ((unsigned long long)(sb * CPW) << 48) |
                      (CYC ? ((unsigned long long)(m / spans) << 24) | (unsigned)(1 + m % spans * kGroupSpan)
                           : P.chunk_coll[m]);
        }
    };
    // the solver's word that word t of share sh is (rows only), -1 past the last interval
    auto solver_word = [&](int sh, int t) {
        const int g = t / CPW * A.want + sh, sb = g / per, sw = sb * CPW + t % CPW;
        return sw < P.eta ? (long long)sw * cps + (g - sb * per) : -1ll;
    };
    __syncthreads();
    for (int it = 0; it < A.K; ++it) {
        const int b = (int)((turn + (unsigned)it) % 3u), bc = (int)((turn + (unsigned)it + 1u) % 3u);
        P.acc = A.acc + (long long)b * D * N;
        P.cnt = A.cnt + (long long)b * N;
        const bool last = it + 1 == A.K;
        {
            // the next iteration's buffer: every member has read it two
            // barriers ago, and adds to it only after the next barrier
            unsigned long long *acc = A.acc + (long long)bc * D * N;
            int *cnt = A.cnt + (long long)bc * N;
            for (int nd = n0 + (int)threadIdx.x; nd < n1; nd += T) {
                for (int d = 0; d < D; ++d)
                    __hip_atomic_store(&acc[(long long)d * N + nd], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&cnt[nd], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        for (int sh = (int)rank; sh < A.want; sh += (int)size) {
            if (it == 0 || many) {
                S.take(P, A.want, sh, nitems_all);
                take_items(sh);
                __syncthreads();
                if (!CYC) {
                    for (int t = threadIdx.x; t < S.nitems * WORDS; t += T) {
                        const long long at = solver_word(sh, t);
                        word[t] = at < 0 ? 0ull : P.bits_coll[at];
                    }
                } else if (it > 0) {
                    const unsigned long long *own = A.words + (long long)sh * A.L.items * WORDS;
                    for (int t = threadIdx.x; t < S.nitems * WORDS; t += T) word[t] = own[t];
                } else {
                    // the solver's words are cut by rows: lane by lane
                    for (int t = wave; t < S.nitems * WORDS; t += T / 64) {
                        const unsigned long long pk = item[t / WORDS];
                        const int sw = (int)(pk >> 48) + t % CPW;
                        int i, j;
                        bool bit = false;
                        if (sw < P.eta && group_pair(p, (int)((pk >> 24) & 0xffffffull),
                                                     (int)(pk & 0xffffffull) + t % WORDS / CPW, lane, &i, &j))
                            bit = (P.bits_coll[(long long)sw * cps + rowchunk(p, i) + (j >> 6)] >> (j & 63)) & 1ull;
                        const unsigned long long w = __builtin_amdgcn_ballot_w64(bit);
                        if (lane == 0) word[t] = w;
                    }
                }
                for (int u = threadIdx.x; u < S.nu; u += T) wbit[u] = P.bits_wall[S.u0 + u];
                __syncthreads();
            }
            const bool fits = S.nitems * WORDS * 64 <= group_queue(T); // (nobody need look at the queue)
            int l = wave, wt = 0; // this wave's next item, the next tile of wall factors
            for (bool end = false; !end;) {
                // Activity tests: items by waves, as long as the queue takes
                // whatever the items in flight may add; one wall factor per lane.
                constexpr int most = group_queue(T) - (T / 64) * WORDS * 64;
                static_assert(most > 0, "an item per wave fits the queue: every round makes progress");
                while (l < S.nitems && (fits || __hip_atomic_load(&len[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) <= most)) {
                    group_item<D, DENSE, T>(P, Z, item[l], l, lane, rad, word, q, &len[0]);
                    l += T / 64;
                }
                if (wt * T < S.nwall) {
                    const int lw = wt * T + (int)threadIdx.x;
                    bool queue = false;
                    unsigned val = 0u;
                    if (lw < S.nwall) {
                        const long long f = 32LL * S.u0 + lw;
                        const WallAt a = wall_at(P, f, P.wbase_wall[f >> 6], (int)(f & 63));
                        const bool bit = !DENSE && ((wbit[lw >> 5] >> (lw & 31)) & 1u);
                        queue = wall_test<M_FUSED>(P, Z, a, bit, &val);
                    }
                    // (the 32 lanes of a word are in one wave: all have read it)
                    if (!DENSE && lw < S.nwall && (lw & 31) == 0) wbit[lw >> 5] = 0u;
                    group_push(qw, &len[1], queue, (val & kPrev) | (unsigned)lw);
                    ++wt;
                }
                if (l < S.nitems && lane == 0) len[2] = it + 1;
                __syncthreads();
                const int nq = len[0], nqw = len[1];
                const bool items = len[2] == it + 1, gone = len[3] != 0;
                end = !items && wt * T >= S.nwall;
                __syncthreads();
                if (gone) return; // (the same on every lane: set before the last barrier's end)
                if (threadIdx.x == 0) len[2] = 0;
                // (room left for another round: the minimisers wait for it)
                if (!end && nq <= most && nqw <= group_wall_queue(T) - T) {
                    __syncthreads();
                    continue;
                }
                if (threadIdx.x == 0) {
                    len[0] = len[1] = 0;
                    totals[2] += (unsigned)(nq + nqw);
                }
                // minimisers of the queued factors, 64 collision or 32 wall
                // entries per wave, then the energy and fixed factors
                const int cc = min(64, max(kGroupMinChunk, (nq + (T / 64) - 1) / (T / 64)));
                const int kc = (nq + cc - 1) / cc, kw = (2 * nqw + 63) >> 6;
                const int ke = end ? (S.ne + 63) >> 6 : 0, kf = end ? (S.nf + 63) >> 6 : 0;
                for (int k = wave; k < kc + kw + ke + kf; k += (T / 64)) {
                    if (k < kc + kw) {
                        bool ac = false, aw = false;
                        float n[4 * D];
                        Contrib out;
                        if (k < kc) {
                            const int t = cc * k + lane;
                            if (lane < cc && t < nq) {
                                const unsigned e = q[t];
                                const int wi = (int)((e & kIdx) >> 6), ln = (int)(e & 63u);
                                const unsigned long long pk = item[wi / WORDS];
                                CollAt c;
                                c.s = (int)(pk >> 48) + wi % CPW;
                                if (!CYC) c.i = (int)((pk >> 24) & 0xffffffull), c.j = (int)(pk & 0xffffffull) + ln;
                                else group_pair(p, (int)((pk >> 24) & 0xffffffull),
                                                (int)(pk & 0xffffffull) + wi % WORDS / CPW, ln, &c.i, &c.j);
                                c.f = (long long)((unsigned)c.s * P2 +
                                                  (unsigned)((long long)c.i * (2 * p - c.i - 1) / 2 + (c.j - c.i - 1)));
                                coll_nodes(P, c.s, c.i, c.j, c.nd);
                                c.R = rad[c.i] + rad[c.j];
                                ac = coll_minimise<D, M_FUSED, false>(P, Z, c, (e & kPrev) != 0, n, out);
                                if (ac) atomicOr(&word[wi], 1ull << ln);
                            }
                        } else {
                            const int t = 64 * (k - kc) + lane;
                            if (t < 2 * nqw) {
                                const unsigned e = qw[t >> 1];
                                const int lf = (int)(e & kIdx);
                                const long long f = 32LL * S.u0 + lf;
                                const WallAt a = wall_at(P, f, P.wbase_wall[f >> 6], (int)(f & 63));
                                aw = wall_minimise<M_FUSED, false>(P, Z, a, (e & kPrev) != 0, t & 1, n, out) &&
                                     (t & 1) == 0;
                                if (aw) atomicOr(&wbit[lf >> 5], 1u << (lf & 31));
                            }
                        }
                        if ((k < kc ? nq : 2 * nqw) >= kGroupSums) contribute_wave<true>(P, out, D);
                        else contribute_wave<false>(P, out, D);
                        if (last) {
                            const int a = __popcll(__ballot(ac)), w = __popcll(__ballot(aw));
                            if (lane == 0 && a) atomicAdd(&totals[0], (unsigned)a);
                            if (lane == 0 && w) atomicAdd(&totals[1], (unsigned)w);
                        }
                    } else if (k < kc + kw + ke) {
                        const int t = 64 * (k - kc - kw) + lane;
                        if (t < S.ne) group_energy<D>(P, Z, A, S.e0 + t, it == 0);
                    } else {
                        const int t = 64 * (k - kc - kw - ke) + lane;
                        if (t < S.nf) group_fixed<D>(P, Z, A, S.f0 + t, it == 0);
                    }
                }
                if (!end) __syncthreads(); // (the queues are free again)
            }
            if (many || last) {
                __syncthreads();
                if (!CYC) {
                    for (int t = threadIdx.x; t < S.nitems * WORDS; t += T) {
                        const long long at = solver_word(sh, t);
                        if (at >= 0) P.bits_coll[at] = word[t];
                    }
                } else if (many) {
                    unsigned long long *own = A.words + (long long)sh * A.L.items * WORDS;
                    for (int t = threadIdx.x; t < S.nitems * WORDS; t += T) own[t] = word[t];
                }
                for (int u = threadIdx.x; u < S.nu; u += T) P.bits_wall[S.u0 + u] = wbit[u];
                __syncthreads();
            }
        }
        if (last) {
            __syncthreads();
            if (threadIdx.x < 3 && totals[threadIdx.x]) atomicAdd(&A.ctl->total[threadIdx.x], totals[threadIdx.x]);
        }
        group_barrier(A.ctl, size, (unsigned)it + 1u, &len[3]);
        if (threadIdx.x == 0) totals[2] = 0u;
        group_nodes<D, DENSE, T>(P, A, b, zc, zp, last ? n0 : 0, last ? n1 : 0);
        __syncthreads();
    }
    if (!CYC) return;
    // The solver's words, cut by rows: cleared, then the bits of the shares added.
    const long long c0 = P.nch * rank / size, c1 = P.nch * (rank + 1) / size;
    for (long long w = c0 + threadIdx.x; w < c1; w += T)
        __hip_atomic_store(&P.bits_coll[w], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    group_barrier(A.ctl, size, (unsigned)A.K + 1u, &len[3]);
    for (int sh = (int)rank; sh < A.want; sh += (int)size) {
        if (many) {
            S.take(P, A.want, sh, nitems_all);
            __syncthreads();
            take_items(sh);
            const unsigned long long *own = A.words + (long long)sh * A.L.items * WORDS;
            for (int t = threadIdx.x; t < S.nitems * WORDS; t += T) word[t] = own[t];
            __syncthreads();
        }
        for (int t = wave; t < S.nitems * WORDS; t += T / 64) {
            const unsigned long long w = uniform64(word[t]);
            if (w == 0ull || !((w >> lane) & 1ull)) continue;
            const unsigned long long pk = item[t / WORDS];
            int i, j;
            group_pair(p, (int)((pk >> 24) & 0xffffffull), (int)(pk & 0xffffffull) + t % WORDS / CPW, lane, &i, &j);
            atomicOr(&P.bits_coll[((pk >> 48) + t % CPW) * cps + rowchunk(p, i) + (j >> 6)], 1ull << (j & 63));
        }
    }
}

// K iterations of one instance (at the steady rho0, a u update pending).
template <int D, bool DENSE>
__global__ __launch_bounds__(kGroupBlock) void k_group(Params P, GroupArgs A) {
    if (blockIdx.x % (unsigned)A.stride) return;
    extern __shared__ __align__(16) char lds[];
    __shared__ unsigned who[3];
    if (threadIdx.x == 0) {
        unsigned r = 0u, m = 0u;
        who[2] = group_join(A.ctl, A.want, A.K, &r, &m) ? 1u : 0u;
        who[0] = r, who[1] = m;
    }
    __syncthreads();
    if (!who[2]) return;
    const unsigned rank = __builtin_amdgcn_readfirstlane(who[0]), size = __builtin_amdgcn_readfirstlane(who[1]);
    group_run<D, DENSE, kGroupBlock>(P, A, lds, rank, size);
    if (rank == 0 && threadIdx.x == 0) {
        for (int k = 0; k < 3; ++k) P.stats[k] = (int)agent_load(&A.ctl->total[k]);
        A.ctl->turn = (A.ctl->turn + (unsigned)A.K) % 3u;
    }
}

// A pointer read from memory, taken as an offset from a kernel argument (base,
// at address at), so that the compiler knows it to be global and does not use
// generic accesses.
template <class Q>
__device__ __forceinline__ void in_global(Q *&p, char *base, unsigned long long at) {
    p = reinterpret_cast<Q *>(base + (long long)((unsigned long long)p - at));
}

// A structure that the kernel does not write, at an address that is the same
// for the whole wave, through the scalar cache: its fields are uniform values.
template <class S>
__device__ __forceinline__ S load_struct(const S *src) {
    static_assert(sizeof(S) % 4 == 0, "read as 32-bit words");
    int raw[sizeof(S) / 4];
#pragma unroll
    for (int k = 0; k < (int)(sizeof(S) / 4); ++k) raw[k] = load_uniform(reinterpret_cast<const int *>(src), k);
    S out;
    __builtin_memcpy(&out, raw, sizeof(S));
    return out;
}

// A batch: block b belongs to the group of instance slots[b]; every instance
// has its own parameters and group.  The phased launches wait in each of their
// three phases for the slowest block of the whole batch and move every
// instance's records through memory; here an instance waits for its own shares
// alone, its records stay in LDS, and what bounds the launch is the walk's issue
// on the compute units and the longest share.  256 instances of up to 128 agents
// 75 -> 48 us per iteration (first iterations, which queue most factors, 390 ->
// 570, paid back within five), 64 instances 39 -> 23, 16 of up to 60 agents 30 -> 16.
// Three workgroups per compute unit: four spill (52 us), 384 lanes leave waves
// idle.  The parameters come from memory by scalar loads, and the pointers among
// them as offsets of a kernel argument: loaded as they are, every access through
// them was a flat one and the branches on them divergent (2x).
__global__ __launch_bounds__(kGroupBatchBlock, 3) void kp_group(const Params *insts, const GroupArgs *groups, const int *slots,
                                                             int K, char *base, unsigned long long at) {
    extern __shared__ __align__(16) char lds[];
    __shared__ unsigned who[3];
    const int inst = __builtin_amdgcn_readfirstlane(slots[blockIdx.x]);
    if (inst < 0) return;
    GroupArgs A = load_struct(groups + inst);
    A.K = K;
    in_global(A.ctl, base, at), in_global(A.acc, base, at), in_global(A.cnt, base, at), in_global(A.xe, base, at);
    in_global(A.words, base, at), in_global(A.sent, base, at);
    if (threadIdx.x == 0) {
        unsigned r = 0u, m = 0u;
        who[2] = group_join(A.ctl, A.want, A.K, &r, &m) ? 1u : 0u;
        who[0] = r, who[1] = m;
    }
    __syncthreads();
    if (!who[2]) return;
    const unsigned rank = __builtin_amdgcn_readfirstlane(who[0]), size = __builtin_amdgcn_readfirstlane(who[1]);
    Params P = load_struct(insts + inst);
    // (every pointer that group_run uses: one that is left out still works, at the
    // price above.  A field added to Params or GroupArgs belongs here if it is one.)
    static_assert(sizeof(Params) == 520 && sizeof(GroupArgs) == 104, "see above");
    in_global(P.zr_prev, base, at), in_global(P.zr_cur, base, at), in_global(P.radii, base, at), in_global(P.walls, base, at), in_global(P.C, base, at);
    in_global(P.xfix, base, at), in_global(P.u_coll, base, at), in_global(P.u_wall, base, at), in_global(P.u_energy, base, at), in_global(P.u_fixed, base, at);
    in_global(P.bits_coll, base, at), in_global(P.bits_wall, base, at), in_global(P.chunk_coll, base, at), in_global(P.counters, base, at), in_global(P.stats, base, at);
    in_global(P.x_coll, base, at), in_global(P.x_wall, base, at), in_global(P.wbase_wall, base, at);
    if (P.dim == 2) group_run<2, false, kGroupBatchBlock>(P, A, lds, rank, size);
    else group_run<3, false, kGroupBatchBlock>(P, A, lds, rank, size);
    if (rank == 0 && threadIdx.x == 0) {
        for (int k = 0; k < 3; ++k) P.stats[k] = (int)agent_load(&A.ctl->total[k]);
        A.ctl->turn = (A.ctl->turn + (unsigned)K) % 3u;
    }
}

// the words of n groups before a launch
__global__ void k_group_arm(GroupCtl *c, int n) {
    const int g = (int)blockIdx.x * (int)(blockDim.x / 4) + (int)(threadIdx.x >> 2), k = (int)(threadIdx.x & 3);
    if (g >= n) return;
    if (k == 0) c[g].reg = c[g].size = c[g].bar = 0u;
    if (k < 3) c[g].total[k] = 0u;
}
