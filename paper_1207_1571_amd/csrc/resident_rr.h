// Resident mixed-precision pressure CG (device code, included by kernels.hip
// after resident_cg.h): the FP32 recurrence with FP64 solution and residual
// replacement (k_rr_*) of a whole solve in one launch.
//
// It is built like the FP64 one and gains for the same reason, but the parts
// are chosen by the order of the sums.  An FP32 recurrence forgets nothing: a
// dot product that differs in its last bit decorrelates the rounding of every
// later iteration, and after some hundred of them the solution differs by as
// much as it is off the exact one (measured 7e-8).  So the sums here are
// those of the launched kernels bit for bit: a part is four consecutive tiles
// of 1024 cells (the launched kernels' blocks), a thread holds four cells of
// a tile, 256 apart, for each of two tiles, and the sums go thread, wave,
// tile, 64 tiles, all, each in the launched kernels' order.  All vectors of
// the solve give the same bits as the launched iterations.
//
// x, r, p, z or q, the diagonal and the coefficients of a part's 4096 cells
// are in registers, p of the part and its halo (the cells of other parts its
// rows read: about two part sizes on a box numbered line by line) in LDS as
// FP32.  A halo too large for the LDS (random numbering) keeps the launched
// iterations.

typedef __attribute__((address_space(1))) unsigned int gword32;

constexpr int kRrTiles = kResCells / kRrTile;     // tiles of a part
constexpr int kRrU = kResCells / kResThreads;     // cells of a thread
constexpr int kRrHaloStep = 9;                    // halo cells a thread loads at once

struct RrRed {
    double part[2][2][kRrTiles][4];   // [generation's parity][value][tile][wave of the tile]
    double tot[2][2];
    int late, local;
};

// Totals of NV values in the launched kernels' order: va the thread's sums
// over its cells of tile tid / 256, vb of tile 2 + tid / 256.  As res_reduce
// otherwise; a group is 16 parts, the 64 tiles the launched reduction sums
// first.
template <int NV, bool FIRST = false>
__device__ __forceinline__ bool rr_reduce(double (&va)[NV], double (&vb)[NV], double (&out)[NV], ResTeam &tm, RrRed &sh)
{
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, par = tm.gen & 1;
    const int S = tm.ngrp * 64;   // slots of a value
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        va[k] = wave_tree(va[k]);
        vb[k] = wave_tree(vb[k]);
        if (lane == 0) {
            sh.part[par][k][wv >> 2][wv & 3] = va[k];
            sh.part[par][k][2 + (wv >> 2)][wv & 3] = vb[k];
        }
    }
    wait_vmem();
    __syncthreads();
    if (wv == 0) {
        const size_t words = rr_gen_words(tm.ngrp);
        double *own = tm.slots + (size_t)(tm.gen & (kResGens - 1)) * words;
        double *old = tm.slots + (size_t)((tm.gen - 1) & (kResGens - 1)) * words;
        double *all = own + 2 * S, *all_old = old + 2 * S;
        const bool one = tm.ngrp == 1, leads = tm.part == tm.first;
        const int q = lane & (kRrTiles - 1), kq = (lane / kRrTiles) & 1;   // lanes 0..3: value 0, lanes 4..7: value 1
        if (lane < NV * kRrTiles) {
            const double *w = sh.part[par][kq][q];
            double t = w[0];
            t += w[1];
            t += w[2];
            t += w[3];
            put_word(own + kq * S + tm.part * kRrTiles + q, slot_word(t), tm.local);
        }
        double t[NV], mine[NV];
        bool ok = true, same_xcd = false;
        if (one || leads) {
            ok = poll_slots<NV>(own + tm.grp * 64, S, tm.size * kRrTiles, tm.ticks, t);
#pragma unroll
            for (int k = 0; k < NV; ++k) t[k] = wave_tree(t[k]);
            if (!one && ok && lane < tm.ngrp)
#pragma unroll
                for (int k = 0; k < NV; ++k)
                    gst(all + (k * kRrGroups + lane) * kRrGroups + tm.grp, slot_word(t[k]));
        }
        if (!one && ok) {
            ok = poll_slots<NV>(all + tm.grp * kRrGroups, kRrGroups * kRrGroups, tm.ngrp, tm.ticks, t);
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                mine[k] = lane_value(t[k], tm.grp);
                t[k] = wave_tree(t[k]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < NV; ++k) mine[k] = t[k];
        }
        // FIRST: the values were each part's XCD and its square
        if (FIRST) same_xcd = tm.size * mine[NV - 1] == mine[0] * mine[0];
        if (lane < 2 * kRrTiles) put_word(old + kq * S + tm.part * kRrTiles + q, kSentinel, tm.local);
        if (!one && leads)
            for (int e = lane; e < 2 * kRrGroups; e += 64) gst(all_old + e * kRrGroups + tm.grp, kSentinel);
        if (lane == 0) {
#pragma unroll
            for (int k = 0; k < NV; ++k) sh.tot[par][k] = t[k];
            if (!ok) sh.late = 1;
            if (FIRST) sh.local = same_xcd;
        }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NV; ++k) out[k] = sh.tot[par][k];
    tm.gen += 1;
    if (FIRST) tm.ticks = tm.later;
    return !sh.late;
}

// One part's share of the solve, from the state the start kernels left
// (k_pcg_init, k_mx_cvt, k_rr_start); false when a wait ran out.  lds: p of
// the own cells and the halo, then the halo's positions.
template <int W>
__device__ bool rr_solve(const DevCase &d, ResTeam &tm, int serial, RrRed &sh, float *lds)
{
    constexpr int U = kRrU;
    const int tid = threadIdx.x, part = tm.part;
    const int p0 = d.res_start[part], n = d.res_start[part + 1] - p0;
    const int h0 = d.res_hstart[part], H = d.res_hstart[part + 1] - h0;
    float *const pl = lds;
    int32_t *const hid = reinterpret_cast<int32_t *>(lds + d.res_local);
    auto *const zf = gmem(d.f_q);   // published z
    double *const xx = d.q;         // published x
    KState s = d.ks[3];
    if (s.done) return true;        // solved (or failed) at the start: the same for every part

    auto place = [&](int u) { return ((u >> 2) * 2 + (tid >> 8)) * kRrTile + (u & 3) * kBlock + (tid & (kBlock - 1)); };
    double x[U], ex[U];   // ex: row sum minus the coefficients' sum (difference form, spmv_row)
    float r[U], p[U], w[U], dg[U], a[U][W];   // w: z = r / diag, or q = A p between the product and the update
    unsigned int ix[U][W / 2];
    unsigned int far = 0, shown = 0;   // bit u: the cell is read by another group / another part
    if (tid == 0) {
        sh.late = 0;
        sh.local = 0;
    }
    for (int h = tid; h < H; h += kResThreads) hid[h] = gmem((const int32_t *)d.res_halo + h0)[h];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int l = place(u), i = p0 + l;
        x[u] = ex[u] = 0.0;
        r[u] = p[u] = w[u] = 0.0f;
        dg[u] = 1.0f;
#pragma unroll
        for (int k = 0; k < W; ++k) a[u][k] = 0.0f;
#pragma unroll
        for (int k = 0; k < W / 2; ++k) ix[u][k] = 0;
        if (l < n) {
            const auto *__restrict__ fe = gmem((const int32_t *)d.res_fe + (size_t)W * p0);
            const auto *__restrict__ idx = gmem((const uint16_t *)d.res_idx + (size_t)W * p0);
            x[u] = gmem((const double *)d.p)[i];
            gmem(d.rt)[i] = x[u];   // start value, for a solve that has to be begun again
            r[u] = gmem((const float *)d.f_r)[i];
            dg[u] = gmem((const float *)d.f_pdiag)[i];
            const int pub = gmem((const uint8_t *)d.res_pub)[i];
            shown |= (pub > 0 ? 1u : 0u) << u;
            far |= (pub > 1 ? 1u : 0u) << u;
            double so = 0.0;
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const int f = fe[k * n + l];
                a[u][k] = f >= 0 ? (float)gmem((const double *)d.poff)[f >> 1] : 0.0f;
                so += (double)a[u][k];
                ix[u][k / 2] |= (unsigned int)idx[k * n + l] << (16 * (k & 1));
            }
            // row sums are exactly zero in slices of mode 2
            ex[u] = (d.sell_mode[i / kBlock] != 2 ? (double)gmem((const float *)d.f_pexc)[i] : 0.0) - so;
            w[u] = r[u] / dg[u];
        }
    }
    auto at = [&](int u, int k) { return (int)((ix[u][k / 2] >> (16 * (k & 1))) & 0xffffu); };
    auto publish = [&](int u) {
        if (!((shown >> u) & 1u)) return;
        gword32 *to = (gword32 *)(zf + p0 + place(u));
        const unsigned int b = __float_as_uint(w[u]);
        if (tm.local && !((far >> u) & 1u)) __hip_atomic_store(to, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        else __hip_atomic_store(to, b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
#pragma unroll
    for (int u = 0; u < U; ++u) publish(u);
    {
        double va[2] = {0.0, 0.0}, vb[2] = {0.0, 0.0}, xcd[2];
        if (tid == 0) {
            va[0] = (double)xcc_id();
            va[1] = va[0] * va[0];
        }
        if (!rr_reduce<2, true>(va, vb, xcd, tm, sh)) return false;
        tm.local = sh.local;
    }

    for (long it = 0; s.done != 1; ++it) {
        // indices and coefficients stay packed and in FP32
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int k = 0; k < W / 2; ++k) asm volatile("" : "+v"(ix[u][k]));
#pragma unroll
            for (int k = 0; k < W; ++k) asm volatile("" : "+v"(a[u][k]));
        }
        if (s.done == 0) {
            // p = z + beta p: own cells and, from the published z, the halo
            const float beta = (float)s.beta;
            const bool first = s.first;
            auto halo_step = [&](int base, auto between) {
                unsigned int zb[kRrHaloStep];
#pragma unroll
                for (int j = 0; j < kRrHaloStep; ++j) {
                    const int h = base + j * kResThreads;
                    zb[j] = h < H ? __hip_atomic_load((const gword32 *)(zf + hid[h]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                  : 0u;
                }
                between();
#pragma unroll
                for (int j = 0; j < kRrHaloStep; ++j) {
                    const int h = base + j * kResThreads;
                    const float z = __uint_as_float(zb[j]);
                    if (h < H) pl[n + h] = first ? z : z + beta * pl[n + h];
                }
            };
            halo_step(tid, [&] {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int l = place(u);
                    if (l < n) {
                        p[u] = first ? w[u] : w[u] + beta * p[u];
                        pl[l] = p[u];
                    }
                }
            });
            for (int base = tid + kRrHaloStep * kResThreads; base < H; base += kRrHaloStep * kResThreads)
                halo_step(base, [] {});
            __syncthreads();
            double va[1] = {0.0}, vb[1] = {0.0}, pq[1];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (place(u) >= n) continue;
                const double pi = (double)p[u];
                double qa = 0.0;
#pragma unroll
                for (int k = 0; k < W; ++k) qa += (double)a[u][k] * (double)pl[at(u, k)];
                w[u] = (float)(qa + ex[u] * pi);
                (u < 4 ? va : vb)[0] += pi * (double)w[u];
            }
            if (!rr_reduce<1>(va, vb, pq, tm, sh)) return false;
            if (!(pq[0] > 0.0) || !isfinite(pq[0])) {
                set_done(s, FVM_ENUMERIC);
                s.iters += 1;
                break;
            }
            s.alpha = uniform(s.rho / pq[0]);
            const float alf = (float)s.alpha;
            double ua[2] = {0.0, 0.0}, ub[2] = {0.0, 0.0}, v2[2];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (place(u) >= n) continue;
                x[u] = x[u] + s.alpha * (double)p[u];
                r[u] = r[u] - alf * w[u];
                w[u] = r[u] / dg[u];
                publish(u);
                (u < 4 ? ua : ub)[0] += fabs((double)r[u]);
                (u < 4 ? ua : ub)[1] += (double)r[u] * (double)w[u];
            }
            if (!rr_reduce<2>(ua, ub, v2, tm, sh)) return false;
            s.iters += 1;
            s.nres = uniform(v2[0] / s.nf);
            s.first = 0;
            s.xbar = s.rho;   // rho of the previous iteration (for a replacement)
            if (!isfinite(s.nres)) set_done(s, FVM_ENUMERIC);
            else if (s.nres <= s.tol_eff || s.iters >= s.max_iter) s.done = 2;   // verify on the true residual
            else if (!(v2[1] > 0.0) || !isfinite(v2[1])) { set_done(s, FVM_ENUMERIC); s.iters += 1; }
            else {
                s.beta = uniform(v2[1] / s.rho);
                s.rho = uniform(v2[1]);
            }
        }
        // residual replacement after every fourth iteration (k_rr_replace),
        // x of the other parts' cells read past the caches
        if ((it & 3) == 3 && s.done != 1 && (s.done == 2 || s.nres < 0.1 * s.scale)) {
            int t = tid;
            asm volatile("" : "+v"(t));   // nothing of this is to be loaded ahead of the loop
            double va[2] = {0.0, 0.0}, vb[2] = {0.0, 0.0}, v2[2];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int l = place(u) - tid + t;
                if (l < n) gst(xx + p0 + l, (unsigned long long)__double_as_longlong(x[u]));
            }
            if (!rr_reduce<2>(va, vb, v2, tm, sh)) return false;
            va[0] = va[1] = vb[0] = vb[1] = 0.0;
            const auto *__restrict__ fe = gmem((const int32_t *)d.res_fe + (size_t)W * p0);
            for (int u = 0; u < U; ++u) {
                const int l = place(u) - tid + t, i = p0 + l;
                double res = 0.0;
                if (l < n) {
                    double c[W], xj[W];
                    int side[W];
#pragma unroll
                    for (int k = 0; k < W; ++k) {
                        const int f = fe[k * n + l];
                        side[k] = f < 0 ? 2 : f & 1;
                        c[k] = f < 0 ? 0.0 : gmem((const double *)d.poff)[f >> 1];
                        const int j = f < 0 ? i : f & 1 ? gmem((const int32_t *)d.own)[f >> 1] : gmem((const int32_t *)d.nei)[f >> 1];
                        xj[k] = __longlong_as_double((long long)gld(xx + j));
                    }
                    // upper entries, then lower ones (row_apply)
                    double ax = gmem((const double *)d.pdiag)[i] * __longlong_as_double((long long)gld(xx + i));
#pragma unroll
                    for (int sd = 0; sd < 2; ++sd)
#pragma unroll
                        for (int k = 0; k < W; ++k)
                            if (side[k] == sd) ax += c[k] * xj[k];
                    res = gmem((const double *)d.pb)[i] - ax;
                }
                const float rf = (float)res;
#pragma unroll
                for (int v = 0; v < U; ++v)
                    if (v == u && l < n) {
                        r[v] = rf;
                        w[v] = rf / dg[v];
                        publish(v);
                        (v < 4 ? va : vb)[0] += fabs(res);
                        (v < 4 ? va : vb)[1] += (double)rf * (double)w[v];
                    }
            }
            if (!rr_reduce<2>(va, vb, v2, tm, sh)) return false;
            const double nres = uniform(v2[0] / s.nf);
            s.nres = s.scale = nres;
            if (!isfinite(nres)) set_done(s, FVM_ENUMERIC);
            else if (nres <= s.tol_eff) set_done(s, FVM_OK);
            else if (s.iters >= s.max_iter) set_done(s, FVM_WARN_MAXITER);
            else if (!(v2[1] > 0.0) || !isfinite(v2[1])) { set_done(s, FVM_ENUMERIC); s.iters += 1; }
            else {
                s.beta = s.first ? 0.0 : uniform(v2[1] / s.xbar);
                s.rho = uniform(v2[1]);
                s.done = 0;
            }
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
        if (place(u) < n) gmem(d.p)[p0 + place(u)] = x[u];
    if (tid == 0) d.res_fin[part] = serial;
    if (part == 0 && tid == 0) d.ks[3] = s;
    return true;
}

template <int W>
__global__ void __launch_bounds__(kResThreads) k_res_rr(Batch bt, ResMap map, int serial, long ticks)
{
    extern __shared__ __align__(16) float rr_lds[];
    __shared__ RrRed sh;
    const int c = map.cs[blockIdx.x];
    if (c >= bt.n) return;
    const DevCase &d = *bt.dc[c];
    ResTeam tm;
    tm.slots = d.res_slots;
    tm.part = map.pt[blockIdx.x];
    tm.G = d.res_G;
    tm.gen = *d.res_gen;
    tm.ngrp = (tm.G + kRrGroup - 1) / kRrGroup;
    tm.grp = tm.part / kRrGroup;
    tm.first = tm.grp * kRrGroup;
    tm.size = min(kRrGroup, tm.G - tm.first);
    tm.local = false;
    tm.ticks = min(ticks, kResStartTicks);
    tm.later = ticks;
    const bool ok = rr_solve<W>(d, tm, serial, sh, rr_lds);
    res_end(d, tm, ok);
}
