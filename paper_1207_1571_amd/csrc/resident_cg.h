// Resident pressure CG (device code, included by kernels.hip): a whole FP64
// Jacobi CG solve in one launch, its state on the chip.
//
// What bounded the launched iterations at these sizes: three kernels per
// iteration that each stream the vectors through the caches and end in a
// grid reduction, whose chain of device-scope accesses and tickets costs
// 5 us at 1e5 cells and 17 us at 1e6 (an update of 1e6 cells took 24 us, the
// direction kernel, which reduces nothing, 7 us).  Here the mesh is split
// into compact parts of at most kResCells cells (mesh_parts: bisection of
// the cell centres, whatever the numbering); one workgroup holds one part
// for the whole solve: r, p, z or q, the reciprocal diagonal and the
// coefficients of its cells in registers (8 cells of about 24 registers per
// thread), x, the diagonal, and p of the part and its halo (the neighbours
// in other parts: 1 000 to 2 500 cells) in LDS, where the product's gathers
// go.  Between workgroups an iteration moves only z of the cells in other
// parts' halos, and two reductions:
//   p = z + beta p          own cells and halo (each part repeats its
//                           neighbours' update, so p needs no exchange)
//   q = A p, p.q            from LDS
//   reduction 1             alpha
//   x += alpha p, r -= alpha q, z = r / diag, |r|, r.z; publish z
//   reduction 2             stop test, beta; every z is visible after it
//
// Every workgroup of a case must be on the device at once: a launch has at
// most one per CU, and the host starts it beside other launches only where
// the CUs suffice for all of them (case.cpp, resident_batch).  Should other
// work keep a workgroup from starting all the same (another process on the
// card), the waits end after a time limit: whoever waited marks the solve and
// leaves, and the host runs the launched iterations from the saved start
// value instead, for a while without trying again (resident_outcome).
//
// The arithmetic per cell and its order are the launched kernels'; only the
// order of the sums over cells differs, and it depends on the case's parts
// alone: a case computes the same bits alone and in any batch.

constexpr int kResThreads = 512;
constexpr int kResWaves = kResThreads / 64;
// limit of the first wait, which ends when every part has started: a second.
// The host starts a launch only where its account leaves the CUs free, so a
// longer wait is for work it knows nothing of.
constexpr long kResStartTicks = 100000000L;
constexpr int kHaloStep = 5;   // halo cells a thread loads at once (a 16^3 brick's halo: 3 to 5 per thread)

// value of one lane, in scalar registers
__device__ __forceinline__ double lane_value(double x, int lane)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), lane),
                            __builtin_amdgcn_readlane(__double2loint(x), lane));
}

// a value that is the same in every lane, in scalar registers
__device__ __forceinline__ double uniform(double x)
{
    return __hiloint2double(__builtin_amdgcn_readfirstlane(__double2hiint(x)),
                            __builtin_amdgcn_readfirstlane(__double2loint(x)));
}

// wave sum in a fixed order, in every lane.  Row shifts and row broadcasts
// cost a few cycles a step where a shuffle goes through the LDS unit.
__device__ __forceinline__ double wave_total(double x)
{
    x += dpp_move<0x111, 0xf>(x);   // row_shr 1, 2, 4, 8: lane 15 of a row has its sum
    x += dpp_move<0x112, 0xf>(x);
    x += dpp_move<0x114, 0xf>(x);
    x += dpp_move<0x118, 0xf>(x);
    x += dpp_move<0x142, 0xa>(x);   // row_bcast 15: rows 1 and 3 take rows 0 and 2
    x += dpp_move<0x143, 0xc>(x);   // row_bcast 31: rows 2 and 3 take row 1
    return lane_value(x, 63);
}

// the wave's own stores and loads have completed
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// a published word: local = a plain store, which ends in the L2 of this XCD
// (for readers known to run on it), else written through to memory.  Readers
// use device-scope loads (gld) either way.
__device__ __forceinline__ void put_word(double *a, unsigned long long b, bool local)
{
    if (local) __hip_atomic_store((gword *)a, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else gst(a, b);
}
__device__ __forceinline__ unsigned long long slot_word(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return b == kSentinel ? kQNaN : b;
}

struct ResRed {
    double part[2][kResMaxSum][kResWaves];
    double tot[2][kResMaxSum];
    int late, local;
};

// What a workgroup needs to take part in its case's reductions.  The case's
// parts form groups of at most kResGroup consecutive parts, and a launch
// places a group on one XCD (workgroups are dispatched round robin over the
// XCDs).  That is checked, not assumed: `local` is set once the group's
// parts have all reported the same XCD, and only speeds up the stores.
struct ResTeam {
    double *slots;   // [kResGens]: own sums [kResMaxSum][ngrp][kResGroup], then
                     // group sums [kResMaxSum][reader's group][kResGroups]
    int part, G, gen;
    int grp, ngrp, first, size;   // group, groups, the group's first part and its parts
    bool local;
    long ticks, later;   // limit of one wait (100 MHz clock): at present, after the first reduction
};

// NV words at a + k * stride, polled by the wave until none is empty; false
// when the time limit passes first.  Lanes past n read nothing and get 0.
template <int NV>
__device__ __forceinline__ bool poll_slots(const double *a, int stride, int n, long ticks, double (&out)[NV])
{
    const int lane = threadIdx.x & 63;
    unsigned long long b[NV];
    const long t0 = wall_clock64();
    bool ok = true;
    for (int spin = 0;; ++spin) {
        bool miss = false;
#pragma unroll
        for (int k = 0; k < NV; ++k) b[k] = lane < n ? gld(a + k * stride + lane) : 0ull;
#pragma unroll
        for (int k = 0; k < NV; ++k) miss = miss || b[k] == kSentinel;
        if (!__any(miss)) break;
        if ((spin & 63) == 63 && wall_clock64() - t0 > ticks) {
            ok = false;
            break;
        }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) out[k] = __longlong_as_double((long long)b[k]);
    return ok;
}

// Totals of NV values over all parts of the case, in every thread; false
// when a part did not arrive in time.  Two workgroup barriers (one where the
// case is a single part).
//
// Each part stores its sums in its own slots; a slot is empty while it holds
// the NaN sentinel.  With one group every part reads all slots (one hop
// through the L2); with several the group's first part reads its group's
// slots and stores the group's sums, a copy per reading group, and every
// part reads those (a hop through the L2 and one through memory; every part
// reading 256 slots through memory took 3.4 us, this 2 us).  All parts add
// the same numbers in the same order, so they take the same decisions
// without a broadcast.  Slots rotate over kResGens generations: a part that
// has passed reduction g knows that every part has finished reading g - 1,
// and empties its own slots of g - 1.  Each wave waits for its earlier
// stores (published z among them) before the barrier in front of the slot's
// store, so whoever sees the sums sees z.
template <int NV, bool FIRST = false>
__device__ __forceinline__ bool res_reduce(double (&v)[NV], ResTeam &tm, ResRed &sh)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, par = tm.gen & 1;
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = wave_total(v[k]);
    if (lane == 0 && wv < kResWaves)   // further waves have no cells
#pragma unroll
        for (int k = 0; k < NV; ++k) sh.part[par][k][wv] = v[k];
    wait_vmem();
    __syncthreads();
    if (tm.G == 1) {
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double t = sh.part[par][k][0];
            for (int w = 1; w < kResWaves; ++w) t += sh.part[par][k][w];
            v[k] = t;
        }
        tm.gen += 1;
        return true;
    }
    if (wv == 0) {
        const int S = tm.ngrp * kResGroup;   // own slots of a value
        const size_t words = res_gen_words(tm.ngrp);
        double *own = tm.slots + (tm.gen & (kResGens - 1)) * words;
        double *old = tm.slots + ((tm.gen - 1) & (kResGens - 1)) * words;
        double *all = own + kResMaxSum * S, *all_old = old + kResMaxSum * S;
        const int me = tm.grp * kResGroup + tm.part - tm.first;
        const bool one = tm.ngrp == 1, leads = tm.part == tm.first;
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            double t = sh.part[par][k][0];
#pragma unroll
            for (int w = 1; w < kResWaves; ++w) t += sh.part[par][k][w];
            if (lane == 0) put_word(own + k * S + me, slot_word(t), tm.local);
        }
        double t[NV];
        bool ok = true;
        if (one || leads) {
            ok = poll_slots<NV>(own + tm.grp * kResGroup, S, tm.size, tm.ticks, t);
#pragma unroll
            for (int k = 0; k < NV; ++k) t[k] = wave_total(t[k]);
            if (!one && ok && lane < tm.ngrp)
#pragma unroll
                for (int k = 0; k < NV; ++k)
                    gst(all + (k * kResGroups + lane) * kResGroups + tm.grp, slot_word(t[k]));
        }
        bool same_xcd = FIRST && one && tm.size * t[NV > 2 ? 2 : 0] == t[NV > 1 ? 1 : 0] * t[NV > 1 ? 1 : 0];
        if (!one && ok) {
            ok = poll_slots<NV>(all + tm.grp * kResGroups, kResGroups * kResGroups, tm.ngrp, tm.ticks, t);
            if (FIRST) {
                const double x = lane_value(t[NV > 1 ? 1 : 0], tm.grp), xx = lane_value(t[NV > 2 ? 2 : 0], tm.grp);
                same_xcd = tm.size * xx == x * x;
            }
#pragma unroll
            for (int k = 0; k < NV; ++k) t[k] = wave_total(t[k]);
        }
        // empty the previous generation's slots
        if (lane < kResMaxSum) put_word(old + lane * S + me, kSentinel, tm.local);
        if (!one && leads)
            for (int e = lane; e < kResMaxSum * kResGroups; e += 64) gst(all_old + e * kResGroups + tm.grp, kSentinel);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) sh.tot[par][k] = t[k];
            if (!ok) sh.late = 1;
            if (FIRST) sh.local = same_xcd;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = sh.tot[par][k];
    tm.gen += 1;
    if (FIRST) tm.ticks = tm.later;
    return !sh.late;
}

// controls of the solve: src 0 the case's pressure controls, 1 the values
// given; serial names the solve (a part that has written its x says so)
struct ResCtl {
    double tol, rel_tol;
    int max_iter, src, serial;
};

// r / d from the rounded reciprocal y of d: one correction step gives the
// quotient to the last bit but for rare halfway cases, in 3 operations
// instead of the division's 14 (the update phase of 4096 cells: 2.0 -> 1.0 us)
__device__ __forceinline__ double quotient(double r, double d, double y)
{
    const double q = r * y;
    return fma(fma(-d, q, r), y, q);
}

// One part's share of the solve; false when a wait ran out.  lds: the part's
// local vector (own cells in [0, n), halo in [n, n + H)), x and the diagonal
// of the own cells, the halo's positions.  A part's cells that lie in other
// parts' halos come first, those read from another group before the rest.
// On return (true) x is in d.p and, in part 0, the record in d.ks[3].
template <int W, int U>
__device__ bool res_solve(const DevCase &d, ResTeam &tm, const ResCtl &ctl, ResRed &sh, double *lds)
{
    const int tid = threadIdx.x, part = tm.part;
    const int p0 = d.res_start[part], n = d.res_start[part + 1] - p0;
    const int h0 = d.res_hstart[part], H = d.res_hstart[part + 1] - h0;
    const int far = d.res_far[part], shown = d.res_shown[part];   // cells read from other groups / other parts
    const auto *__restrict__ cell = gmem((const int32_t *)d.res_cell + p0);
    double *const zx = d.q;    // published z (part order)
    double *const xx = d.qt;   // published x
    double *const loc = lds, *const xl = lds + d.res_local, *const dl = xl + kResCells;
    int32_t *const hid = reinterpret_cast<int32_t *>(dl + kResCells);

    double r[U], p[U], y[U], a[U][W];
    double w[U];   // z = r / diag between the update and the direction, q = A p between the product and the update
    unsigned int ix[U][W / 2];
    if (tid == 0) {
        sh.late = 0;
        sh.local = 0;
    }
    for (int h = tid; h < H; h += kResThreads) hid[h] = gmem((const int32_t *)d.res_halo + h0)[h];
    double v3[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int l = u * kResThreads + tid;
        r[u] = p[u] = w[u] = 0.0;
        y[u] = 1.0;
#pragma unroll
        for (int k = 0; k < W; ++k) a[u][k] = 0.0;
#pragma unroll
        for (int k = 0; k < W / 2; ++k) ix[u][k] = 0;
        if (l < n) {
            const auto *__restrict__ fe = gmem((const int32_t *)d.res_fe + (size_t)W * p0);
            const auto *__restrict__ idx = gmem((const uint16_t *)d.res_idx + (size_t)W * p0);
            const int i = cell[l];
            const double x0 = gmem((const double *)d.p)[i], di = gmem((const double *)d.pdiag)[i];
            gmem(d.rt)[i] = x0;   // start value, for a solve that has to be begun again
            xl[l] = loc[l] = x0;
            dl[l] = di;
            y[u] = 1.0 / di;
            if (l < shown) gst(xx + p0 + l, (unsigned long long)__double_as_longlong(x0));
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const int f = fe[k * n + l];
                a[u][k] = f >= 0 ? gmem((const double *)d.poff)[f >> 1] : 0.0;
                ix[u][k / 2] |= (unsigned int)idx[k * n + l] << (16 * (k & 1));
            }
            v3[0] += x0;
        }
    }
    auto at = [&](int u, int k) { return (int)((ix[u][k / 2] >> (16 * (k & 1))) & 0xffffu); };
    // z of a cell that others read
    auto publish = [&](int l, double z) {
        if (l < far) gst(zx + p0 + l, (unsigned long long)__double_as_longlong(z));
        else if (l < shown) put_word(zx + p0 + l, (unsigned long long)__double_as_longlong(z), tm.local);
    };

    // ---- start: residual, normalisation (k_pcg_sumx, k_pcg_init); the first
    // reduction also tells whether the group's parts share an XCD
    if (tid == 0) {
        v3[1] = (double)xcc_id();
        v3[2] = v3[1] * v3[1];
    }
    if (!res_reduce<3, true>(v3, tm, sh)) return false;
    tm.local = sh.local;
    const double xbar = uniform(v3[0] / (double)d.N);
    for (int h = tid; h < H; h += kResThreads) loc[n + h] = __longlong_as_double((long long)gld(xx + hid[h]));
    __syncthreads();
    v3[0] = v3[1] = v3[2] = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int l = u * kResThreads + tid;
        if (l >= n) continue;
        // upper entries, then lower ones: the order of row_apply and row_sum
        const auto *__restrict__ fe = gmem((const int32_t *)d.res_fe + (size_t)W * p0);
        double ax = dl[l] * xl[l], a1 = dl[l];
#pragma unroll
        for (int side = 0; side < 2; ++side)
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const int f = fe[k * n + l];
                if (f >= 0 && (f & 1) == side) {
                    ax += a[u][k] * loc[at(u, k)];
                    a1 += a[u][k];
                }
            }
        const double b = gmem((const double *)d.pb)[cell[l]];
        r[u] = b - ax;
        w[u] = quotient(r[u], dl[l], y[u]);
        publish(l, w[u]);
        v3[0] += fabs(ax - xbar * a1) + fabs(b - xbar * a1);
        v3[1] += fabs(r[u]);
        v3[2] += r[u] * w[u];
    }
    if (!res_reduce<3>(v3, tm, sh)) return false;
    KState s{};
    s.xbar = xbar;
    s.tol = ctl.src ? ctl.tol : d.p_tol;
    s.rel_tol = ctl.src ? ctl.rel_tol : d.p_rel_tol;
    s.max_iter = ctl.src ? ctl.max_iter : d.p_max_iter;
    s.nf = uniform(v3[0] + 1e-20);
    s.nres0 = s.nres = uniform(v3[1] / s.nf);
    s.tol_eff = uniform(fmax(s.tol, s.rel_tol * s.nres0));
    s.first = 1;
    if (!isfinite(s.nres0)) set_done(s, FVM_ENUMERIC);
    else if (s.nres0 <= s.tol_eff) set_done(s, FVM_OK);
    else if (!(v3[2] > 0.0) || !isfinite(v3[2])) { set_done(s, FVM_ENUMERIC); s.iters = 1; }
    else s.rho = uniform(v3[2]);

    while (!s.done) {
        // the packed indices stay packed: unpacked ahead of the loop they
        // would take twice the registers
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < W / 2; ++k) asm volatile("" : "+v"(ix[u][k]));
        // p = z + beta p: own cells and, from the published z, the halo
        const double beta = s.beta;
        const bool first = s.first;
        auto halo_step = [&](int base, auto between) {
            // every load of the step is issued before the first use
            unsigned long long zb[kHaloStep];
#pragma unroll
            for (int j = 0; j < kHaloStep; ++j) {
                const int h = base + j * kResThreads;
                zb[j] = h < H ? gld(zx + hid[h]) : 0ull;
            }
            between();
#pragma unroll
            for (int j = 0; j < kHaloStep; ++j) {
                const int h = base + j * kResThreads;
                const double z = __longlong_as_double((long long)zb[j]);
                if (h < H) loc[n + h] = first ? z : z + beta * loc[n + h];
            }
        };
        halo_step(tid, [&] {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int l = u * kResThreads + tid;
                if (l < n) {
                    p[u] = first ? w[u] : w[u] + beta * p[u];
                    loc[l] = p[u];
                }
            }
        });
        for (int base = tid + kHaloStep * kResThreads; base < H; base += kHaloStep * kResThreads) halo_step(base, [] {});
        __syncthreads();
        double pq[1] = {0.0};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = u * kResThreads + tid;
            if (l >= n) continue;
            double q = dl[l] * p[u];
#pragma unroll
            for (int k = 0; k < W; ++k) q += a[u][k] * loc[at(u, k)];
            w[u] = q;
            pq[0] += p[u] * q;
        }
        if (!res_reduce<1>(pq, tm, sh)) return false;
        if (!(pq[0] > 0.0) || !isfinite(pq[0])) {
            set_done(s, FVM_ENUMERIC);
            s.iters += 1;
            break;
        }
        s.alpha = uniform(s.rho / pq[0]);
        double v2[2] = {0.0, 0.0};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = u * kResThreads + tid;
            if (l >= n) continue;
            r[u] = r[u] - s.alpha * w[u];
            w[u] = quotient(r[u], dl[l], y[u]);
            publish(l, w[u]);
            v2[0] += fabs(r[u]);
            v2[1] += r[u] * w[u];
            xl[l] += s.alpha * p[u];
        }
        if (!res_reduce<2>(v2, tm, sh)) return false;
        s.iters += 1;
        s.nres = uniform(v2[0] / s.nf);
        s.first = 0;
        if (!isfinite(s.nres)) set_done(s, FVM_ENUMERIC);
        else if (s.nres <= s.tol_eff) set_done(s, FVM_OK);
        else if (s.iters >= s.max_iter) set_done(s, FVM_WARN_MAXITER);
        else if (!(v2[1] > 0.0) || !isfinite(v2[1])) { set_done(s, FVM_ENUMERIC); s.iters += 1; }
        else {
            s.beta = uniform(v2[1] / s.rho);
            s.rho = uniform(v2[1]);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int l = u * kResThreads + tid;
        if (l < n) gmem(d.p)[cell[l]] = xl[l];
    }
    if (tid == 0) d.res_fin[part] = ctl.serial;
    if (part == 0 && tid == 0) d.ks[3] = s;
    return true;
}

// Workgroup b of a launch holds part pt[b] of case cs[b] (255: none); a
// group's parts have the same b % 8, one XCD.
struct ResMap {
    uint8_t cs[kResParts], pt[kResParts];
};

__device__ __forceinline__ ResTeam res_team(const DevCase &d, int part, long ticks)
{
    ResTeam tm;
    tm.slots = d.res_slots;
    tm.part = part;
    tm.G = d.res_G;
    tm.gen = *d.res_gen;
    tm.ngrp = res_groups(tm.G);
    tm.grp = res_group_of(tm.part, tm.G);
    tm.first = res_group_first(tm.grp, tm.G);
    tm.size = res_group_first(tm.grp + 1, tm.G) - tm.first;
    tm.local = false;
    tm.ticks = min(ticks, kResStartTicks);
    tm.later = ticks;
    return tm;
}

// the next solve goes on with the generation after this one's last (its
// slots are emptied then)
__device__ __forceinline__ void res_end(const DevCase &d, const ResTeam &tm, bool ok)
{
    if (threadIdx.x != 0) return;
    if (!ok) d.ks[kNumKs - 1].pad[0] = 1;
    else if (tm.part == 0) *d.res_gen = tm.gen & (kResGens - 1);
}

template <int W, int U>
__global__ void __launch_bounds__(kResThreads) k_res_cg(Batch bt, ResMap map, ResCtl ctl, long ticks)
{
    extern __shared__ __align__(16) double res_lds[];
    __shared__ ResRed sh;
    const int c = map.cs[blockIdx.x];
    if (c >= bt.n) return;
    const DevCase &d = *bt.dc[c];
    ResTeam tm = res_team(d, map.pt[blockIdx.x], ticks);
    const bool ok = res_solve<W, U>(d, tm, ctl, sh, res_lds);
    res_end(d, tm, ok);
}

// slots empty, generation 0, no wait run out (ks[kNumKs - 1].pad[0]; case
// creation, the static descriptor, and after a solve that had to be begun
// again); serial > 0: parts that had finished that solve get their start
// value back
__global__ void k_res_reset(Batch bt, int serial)
{
    CASE_OF(bt);
    const long t = (long)K.raw * kBlock + threadIdx.x, stride = (long)K.G * kBlock;
    if (d.res_G > 0) {
        for (long i = t; i < d.res_words; i += stride) clear_word(d.res_slots, i);
        if (t == 0) {
            *d.res_gen = 0;
            d.ks[kNumKs - 1].pad[0] = 0;
        }
    }
    for (int part = K.raw; serial > 0 && part < d.res_G; part += K.G)
        if (d.res_fin[part] == serial)
            for (int q = d.res_start[part] + threadIdx.x; q < d.res_start[part + 1]; q += kBlock)
            {
                const int i = (int)((unsigned int)d.res_cell[q] & ~(kDicShown | kDicFar));
                d.p[i] = d.rt[i];
            }
}
