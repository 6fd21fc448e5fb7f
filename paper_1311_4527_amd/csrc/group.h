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
// Only workgroups that already run are ever waited for.  They register; the
// first one waits a bounded time for the rest and then freezes the group at
// whoever came.  Later workgroups see the frozen mark and leave, the members
// share out all the shares.  No assumption about residency or dispatch order
// is needed for progress or for the result (fewer members are just slower).
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

constexpr int kGroupBlock = 512;                // lanes per workgroup
constexpr int kGroupWaves = kGroupBlock / 64;
constexpr int kGroupCpw = 2;                    // break-point intervals per item of the collision walk
constexpr int kGroupTile = 32;                  // items of a tile (walked between two looks at the queue)
constexpr int kGroupQueue = 2 * kGroupTile * kGroupCpw * 64;  // entries of the LDS collision queue
constexpr int kGroupMinChunk = 16;              // least entries a wave takes from the collision queue
// Queue length from which a wave sums the contributions to equal nodes before
// the atomics: the shuffles cost a short queue 1 us, the atomics on the same
// nodes a crowded one more (start of the 100-agent swap 22 against 17 us per
// iteration, ADMM of 32 agents 20 against 10.4).
constexpr int kGroupSums = 64;
constexpr int kGroupWallQueue = 2 * kGroupBlock;
constexpr unsigned kGroupFrozen = 0x80000000u;

// Shared words of a group, each on a line of its own where it is polled.
struct GroupCtl {
    unsigned reg, pad0[31];  // workgroups that came; bit 31 once the group is frozen
    unsigned size, pad1[31]; // members (0 until frozen)
    unsigned bar, pad2[31];  // barrier arrivals
    unsigned total[4];       // last iteration: active collision, active wall, queued factors
    unsigned pad3[28];
    unsigned turn;           // buffer the next iteration adds to (kept between launches)
    unsigned stuck;          // a wait ran out (never, short of a fault): results invalid
};

// byte offsets in the dynamic LDS
struct GroupLds {
    unsigned zc, zp, rad, item, word, wbit, q, qw, total;
    int items, walls32; // items and 32-factor wall units of the largest share
};

struct GroupArgs {
    GroupCtl *ctl;
    unsigned long long *acc; // [3][dim][N]
    int *cnt;                // [3][N]
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

// a wait gives up after about this many polls (seconds): a member that left
// abnormally must not hang the device
constexpr unsigned kGroupPatience = 1u << 25;

// Join the group: members get their rank in *rank and the member count in
// *size; false for a workgroup that came too late.
__device__ __forceinline__ bool group_join(GroupCtl *c, int want, unsigned *rank, unsigned *size) {
    const unsigned r = atomicAdd(&c->reg, 1u);
    if (r & kGroupFrozen) return false;
    if (r == 0u) {
        // about 50 us for the rest of the launch to arrive
        for (int n = 0; n < 128 && agent_load(&c->reg) < (unsigned)want; ++n) __builtin_amdgcn_s_sleep(1);
        const unsigned m = min(atomicOr(&c->reg, kGroupFrozen), (unsigned)want);
        __hip_atomic_store(&c->size, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *size = m;
    } else {
        unsigned m = 0u;
        for (unsigned n = 0; n < kGroupPatience && (m = agent_load(&c->size)) == 0u; ++n) __builtin_amdgcn_s_sleep(1);
        if (m == 0u) c->stuck = 1u;
        *size = m;
    }
    *rank = r;
    return r < *size;
}

// Barrier `n` (1, 2, ...) of the group.  Every memory operation of the
// workgroup's waves is complete before it arrives.
__device__ __forceinline__ void group_barrier(GroupCtl *c, unsigned size, unsigned n) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        atomicAdd(&c->bar, 1u);
        const unsigned all = size * n;
        unsigned k = 0;
        while (agent_load(&c->bar) < all)
            if (++k == kGroupPatience) {
                c->stuck = 1u;
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
template <int D, bool DENSE>
__device__ __forceinline__ void group_nodes(const Params &P, const GroupArgs &A, int b, float4 *zc, float4 *zp, int w0,
                                            int w1) {
    constexpr int U = 4;
    const int N = (int)P.N, goal0 = P.eta * P.p;
    const unsigned long long *acc = A.acc + (long long)b * D * N;
    const int *cnt = A.cnt + (long long)b * N;
    for (int n0 = threadIdx.x; n0 < N; n0 += U * kGroupBlock) {
        unsigned long long a[U][D];
        int c[U];
        float4 fx[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int nd = n0 + k * kGroupBlock;
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
            const int nd = n0 + k * kGroupBlock;
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

// K iterations of the instance by member `rank` of `size`.
template <int D, bool DENSE>
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
    __shared__ int len[2];           // queue lengths
    __shared__ unsigned totals[4];   // this iteration's active and queued factors
    for (int nd = threadIdx.x; nd < N; nd += kGroupBlock) {
        zc[nd] = P.zr_cur[nd];
        if (DENSE) zp[nd] = P.zr_prev[nd];
    }
    for (int i = threadIdx.x; i < p; i += kGroupBlock) rad[i] = P.radii[i];
    if (threadIdx.x < 2) len[threadIdx.x] = 0;
    if (threadIdx.x < 4) totals[threadIdx.x] = 0u;
    P.radii = rad;
    const int cps = (int)P.cps, nsb = (P.eta + CPW - 1) / CPW;
    const int nitems_all = cps * nsb;
    GroupShare S;
    const unsigned P2 = (unsigned)P.P2;
    const unsigned turn = agent_load(&A.ctl->turn);
    const bool many = size < (unsigned)A.want; // a member runs several shares in turn
    const int n0 = (int)((long long)N * rank / size), n1 = (int)((long long)N * (rank + 1) / size);
    const Rec Z{zc, zp};
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
            for (int nd = n0 + (int)threadIdx.x; nd < n1; nd += kGroupBlock) {
                for (int d = 0; d < D; ++d)
                    __hip_atomic_store(&acc[(long long)d * N + nd], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(&cnt[nd], 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        for (int sh = (int)rank; sh < A.want; sh += (int)size) {
            if (it == 0 || many) {
                S.take(P, A.want, sh, nitems_all);
                for (int l = threadIdx.x; l < S.nitems; l += kGroupBlock) {
                    const int g = l * A.want + sh;
                    const int sb = g / cps, col = g - sb * cps, s0 = sb * CPW;
                    item[l] = ((unsigned long long)s0 << 48) | P.chunk_coll[col];
                    for (int k = 0; k < CPW; ++k)
                        word[l * CPW + k] = s0 + k < P.eta ? P.bits_coll[(long long)(s0 + k) * cps + col] : 0ull;
                }
                for (int u = threadIdx.x; u < S.nu; u += kGroupBlock) wbit[u] = P.bits_wall[S.u0 + u];
                __syncthreads();
            }
            const int tiles = max(1, max((S.nitems + kGroupTile - 1) / kGroupTile,
                                         (S.nwall + kGroupBlock - 1) / kGroupBlock));
            for (int tile = 0; tile < tiles; ++tile) {
                // activity tests of a tile: items by waves, one wall factor per lane
                for (int l = tile * kGroupTile + wave; l < min((tile + 1) * kGroupTile, S.nitems); l += kGroupWaves) {
                    const unsigned long long pk = item[l];
                    const int s0 = (int)__builtin_amdgcn_readfirstlane((int)(pk >> 48));
                    const int i = (int)__builtin_amdgcn_readfirstlane((int)((pk >> 24) & 0xffffffull));
                    const int j0 = (int)__builtin_amdgcn_readfirstlane((int)(pk & 0xffffffull));
                    const int ns = min(CPW, P.eta - s0);
                    const int j = j0 + lane;
                    const bool valid = j > i && j < p;
                    const int jj = min(j, p - 1);
                    const unsigned long long act = __builtin_amdgcn_ballot_w64(valid);
                    const float R = rad[i] + rad[jj];
                    const float4 *ci = zc + s0 * p + i, *cj = zc + s0 * p + jj;
                    unsigned long long queue[CPW], prev[CPW]; // lanes to queue, and those active last iteration
                    if constexpr (!DENSE) {
                        float4 ri[CPW + 1], rj[CPW + 1];
#pragma unroll
                        for (int k = 0; k <= CPW; ++k) ri[k] = ci[min(k, ns) * p], rj[k] = cj[min(k, ns) * p];
                        // an inactive factor's u is zero, so its n is z
                        cpa_masks<D, CPW>(ri, rj, R * R, queue);
#pragma unroll
                        for (int k = 0; k < CPW; ++k) {
                            prev[k] = uniform64(word[l * CPW + k]);
                            queue[k] = k < ns ? (queue[k] & act) | prev[k] : 0ull;
                        }
                        if (lane < CPW) word[l * CPW + lane] = 0ull;
                    } else {
                        const float4 *pi = zp + s0 * p + i, *pj = zp + s0 * p + jj;
                        const unsigned fr = (unsigned)((long long)i * (2 * p - i - 1) / 2 + (j - i - 1));
                        float u[CPW][4 * D];
#pragma unroll
                        for (int k = 0; k < CPW; ++k)
                            if (k < ns && valid) load_u_coll<D>(P, (unsigned)(s0 + k) * P2 + fr, u[k]);
#pragma unroll
                        for (int k = 0; k < CPW; ++k) {
                            bool go = false;
                            unsigned val = 0u;
                            if (k < ns && valid) {
                                const float4 rc[4] = {ci[k * p], ci[(k + 1) * p], cj[k * p], cj[(k + 1) * p]};
                                const float4 rp[4] = {pi[k * p], pi[(k + 1) * p], pj[k * p], pj[(k + 1) * p]};
                                go = coll_factor<D, M_FUSED, true>(P, (unsigned)(s0 + k) * P2 + fr, R, rc, rp, u[k], 0ull,
                                                                   lane, &val);
                            }
                            queue[k] = __ballot(go);
                            prev[k] = __ballot((val & kPrev) != 0u);
                        }
                    }
                    int n = 0;
#pragma unroll
                    for (int k = 0; k < CPW; ++k) n += __popcll(queue[k]);
                    if (n == 0) continue;
                    int base = 0;
                    if (lane == 0) base = atomicAdd(&len[0], n);
                    base = __builtin_amdgcn_readfirstlane(base);
                    const unsigned long long below = (1ull << lane) - 1ull, me = 1ull << lane;
#pragma unroll
                    for (int k = 0; k < CPW; ++k) {
                        if (queue[k] & me)
                            q[base + __popcll(queue[k] & below)] = ((prev[k] & me) ? kPrev : 0u) |
                                                                   (unsigned)((l * CPW + k) << 6) | (unsigned)lane;
                        base += __popcll(queue[k]);
                    }
                }
                const int lw = tile * kGroupBlock + (int)threadIdx.x;
                if (tile * kGroupBlock < S.nwall) {
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
                }
                __syncthreads();
                const int nq = len[0], nqw = len[1];
                const bool end = tile + 1 == tiles;
                __syncthreads();
                if (!end && nq <= kGroupQueue / 2 && nqw <= kGroupWallQueue - kGroupBlock) continue;
                if (threadIdx.x == 0) {
                    len[0] = len[1] = 0;
                    totals[2] += (unsigned)(nq + nqw);
                }
                // minimisers of the queued factors, 64 collision or 32 wall
                // entries per wave, then the energy and fixed factors
                const int cc = min(64, max(kGroupMinChunk, (nq + kGroupWaves - 1) / kGroupWaves));
                const int kc = (nq + cc - 1) / cc, kw = (2 * nqw + 63) >> 6;
                const int ke = end ? (S.ne + 63) >> 6 : 0, kf = end ? (S.nf + 63) >> 6 : 0;
                for (int k = wave; k < kc + kw + ke + kf; k += kGroupWaves) {
                    if (k < kc + kw) {
                        bool ac = false, aw = false;
                        float n[4 * D];
                        Contrib out;
                        if (k < kc) {
                            const int t = cc * k + lane;
                            if (lane < cc && t < nq) {
                                const unsigned e = q[t];
                                const int wi = (int)((e & kIdx) >> 6), ln = (int)(e & 63u);
                                const unsigned long long pk = item[wi / CPW];
                                CollAt c;
                                c.s = (int)(pk >> 48) + wi % CPW, c.i = (int)((pk >> 24) & 0xffffffull);
                                c.j = (int)(pk & 0xffffffull) + ln;
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
                        if (nq >= kGroupSums) contribute_wave<true>(P, out, D);
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
                for (int l = threadIdx.x; l < S.nitems; l += kGroupBlock) {
                    const int g = l * A.want + sh;
                    const int sb = g / cps, col = g - sb * cps, s0 = sb * CPW;
                    for (int k = 0; k < CPW && s0 + k < P.eta; ++k)
                        P.bits_coll[(long long)(s0 + k) * cps + col] = word[l * CPW + k];
                }
                for (int u = threadIdx.x; u < S.nu; u += kGroupBlock) P.bits_wall[S.u0 + u] = wbit[u];
                __syncthreads();
            }
        }
        if (last) {
            __syncthreads();
            if (threadIdx.x < 3 && totals[threadIdx.x]) atomicAdd(&A.ctl->total[threadIdx.x], totals[threadIdx.x]);
        }
        group_barrier(A.ctl, size, (unsigned)it + 1u);
        if (threadIdx.x == 0) totals[2] = 0u;
        group_nodes<D, DENSE>(P, A, b, zc, zp, last ? n0 : 0, last ? n1 : 0);
        __syncthreads();
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
        who[2] = group_join(A.ctl, A.want, &r, &m) ? 1u : 0u;
        who[0] = r, who[1] = m;
    }
    __syncthreads();
    if (!who[2]) return;
    const unsigned rank = __builtin_amdgcn_readfirstlane(who[0]), size = __builtin_amdgcn_readfirstlane(who[1]);
    group_run<D, DENSE>(P, A, lds, rank, size);
    if (rank == 0 && threadIdx.x == 0) {
        for (int k = 0; k < 3; ++k) P.stats[k] = (int)agent_load(&A.ctl->total[k]);
        A.ctl->turn = (A.ctl->turn + (unsigned)A.K) % 3u;
    }
}

// a group's words before a launch
__global__ void k_group_arm(GroupCtl *c) {
    if (threadIdx.x == 0) c->reg = c->size = c->bar = 0u;
    if (threadIdx.x < 4) c->total[threadIdx.x] = 0u;
}
