// Resident pressure CG with the DIC preconditioner (device code, included by
// kernels.hip after resident_cg.h): a whole FP64 solve in one launch, parts,
// reductions and state as in resident_cg.h.
//
// What bounded it: the two triangular sweeps, 298 dependent levels on 1M
// renumbered cells, at 1.1 us per level: every value went from one CU to the
// next through the L2 of the one XCD that ran the sweep.  With compact parts
// most dependencies lie inside a part: a value then goes from wave to wave
// through LDS (0.2 us per level), and only some 20 times on the longest chain,
// from part to part, through the L2 or memory.  All XCDs take part.  Measured
// on 1M cells: 660 -> 360 us per iteration (a PISO step 415 -> 207 ms); 36 us
// of it are the products, updates and reductions, the sweeps 150 and 170 us.
// They now go at the pace of a wave's chunks, about 1 us each: the loads for
// the next cells, and the published values' stores in front of them.
//
// A part's cells are ordered by dependency level (local index = place in
// that order), so chunk c of 64 cells belongs to wave c % 8, and a wave takes
// its chunks one after the other.  A lane waits until all values its cell
// depends on are in the LDS vector `sw`; a word is empty while it holds the
// NaN sentinel.  Values of other parts are brought there by four further
// waves, each lane taking its halo cells in level order from the published
// array (with those loads in the waves that compute, every look at LDS waited
// for one: 1.6 us per level; with further waves publishing as well, a value
// took 3 us longer from part to part).  The earliest unfinished cell never
// waits for a later one (its wave can only be at a chunk, the lane that brings
// a word only at a halo cell, of the same or a lower level), so a sweep always
// progresses; every wait has the time limit of the reductions.
//
// Published words are emptied again by their owner: y after the reduction of
// r.z (every part has finished its sweeps), z after the reduction of p.q
// (every part has taken z of its halo into p), each of them at least one
// reduction before the array is polled again.
//
// The sums per cell are those of the launched sweeps in the same order; the
// division by D* is a product with its rounded reciprocal, formed once.

constexpr int kDicBring = 4;       // waves that bring the halo
constexpr int kDicThreads = kResThreads + 64 * kDicBring;
constexpr int kDicFlight = 3;      // halo words a lane has under way
constexpr int kDicFew = 3;         // entries of a cell a sweep uses, but for few meshes
constexpr int kDicChunks = kResCells / 64;

// words of LDS shared by waves without a barrier
__device__ __forceinline__ double lds_word(const double *a)
{
    return __longlong_as_double((long long)__hip_atomic_load(reinterpret_cast<const unsigned long long *>(a), __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_WORKGROUP));
}
__device__ __forceinline__ void lds_put(double *a, double v)
{
    __hip_atomic_store(reinterpret_cast<unsigned long long *>(a), slot_word(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ bool lds_empty(double v) { return (unsigned long long)__double_as_longlong(v) == kSentinel; }

template <int W>
__device__ __forceinline__ bool res_solve_dic(const DevCase &d, ResTeam &tm, const ResCtl &ctl, ResRed &sh, double *lds)
{
    constexpr int U = kResCells / kResThreads;
    const int tid = threadIdx.x, part = tm.part;
    int own0 = tid < kResThreads ? tid : kResCells;   // first own cell (none: past the end)
    const int p0 = d.res_start[part], n = d.res_start[part + 1] - p0;
    const int h0 = d.res_hstart[part], H = d.res_hstart[part + 1] - h0;
    const auto *__restrict__ cell = gmem((const int32_t *)d.res_cell + p0);
    const auto *__restrict__ idx = gmem((const uint16_t *)d.res_idx + (size_t)W * p0);
    double *const zg = d.q, *const yg = d.q + d.N;   // published z and y (D* during its set-up), part order
    double *const xx = d.qt;                          // published x
    // the part's residual, diagonal, 1 / D*, x and coefficients (entry k of
    // cell l at k n + l): arrays only their own threads use, too many for LDS
    auto *const r = gmem(d.r) + p0, *const dl = gmem(d.r) + d.N + p0, *const rD = gmem(d.r) + 2 * (size_t)d.N + p0;
    auto *const xg = gmem(d.rt) + d.N + p0, *const coef = gmem(d.pp) + (size_t)W * p0;
    // LDS: p and a sweep's values, own cells then halo; y, then q = A p
    double *const loc = lds, *const sw = lds + d.res_local, *const w = sw + d.res_local + 1;
    // per chunk: the cells other parts, parts of other groups read
    unsigned long long *const shown = reinterpret_cast<unsigned long long *>(w + kResCells), *const far = shown + kDicChunks;
    uint32_t *const hid = reinterpret_cast<uint32_t *>(far + kDicChunks);
    const int none = n + H;                           // a word of sw that holds 1

    unsigned int more_lo = 0, more_up = 0;   // bit u: a cell of the wave's has more than kDicFew lower / upper entries
    unsigned int lower = 0, every = 0;  // 4 bits for each u: the cell's lower entries, all its entries
    if (tid == 0) {
        sh.late = 0;
        sh.local = 0;
        sw[none] = 1.0;
    }
    for (int h = tid; h < H; h += kDicThreads) {
        hid[h] = (uint32_t)gmem((const int32_t *)d.res_halo + h0)[h];
        reinterpret_cast<unsigned long long *>(sw)[n + h] = kSentinel;
    }
    // addresses are formed where they are used: 100 of them kept over the
    // iterations ran out of registers
    auto renew = [&] { asm volatile("" : "+v"(own0)); };
    auto index = [&](int l) { return (int)((unsigned int)cell[l] & ~(kDicShown | kDicFar)); };
    double v3[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int l = u * kResThreads + own0;
        const unsigned int c = l < n ? (unsigned int)cell[l] : 0u;
        const unsigned long long ms = __ballot(c & kDicShown), mf = __ballot(c & kDicFar);
        if (tid < kResThreads && (tid & 63) == 0) {
            shown[l >> 6] = ms;
            far[l >> 6] = mf;
        }
        unsigned int nl = 0, ne = 0;
        if (l < n) {
            const auto *__restrict__ fe = gmem((const int32_t *)d.res_fe + (size_t)W * p0);
            const int i = index(l);
            const double x0 = gmem((const double *)d.p)[i];
            gmem(d.rt)[i] = x0;   // start value, for a solve that has to be begun again
            xg[l] = loc[l] = x0;
            dl[l] = gmem((const double *)d.pdiag)[i];
            reinterpret_cast<unsigned long long *>(sw)[l] = kSentinel;
            if (c & kDicShown) {
                gst(xx + p0 + l, (unsigned long long)__double_as_longlong(x0));
                gst(yg + p0 + l, kSentinel);
                gst(zg + p0 + l, kSentinel);
            }
#pragma unroll
            for (int k = 0; k < W; ++k) {
                const int f = fe[k * n + l];
                coef[k * n + l] = f >= 0 ? gmem((const double *)d.poff)[f >> 1] : 0.0;
                nl += f >= 0 && (f & 1) ? 1u : 0u;
                ne += f >= 0 ? 1u : 0u;
            }
            lower |= nl << (4 * u);
            every |= ne << (4 * u);
            v3[0] += x0;
        }
        more_lo |= (__any(nl > kDicFew) ? 1u : 0u) << u;
        more_up |= (__any(ne - nl > kDicFew) ? 1u : 0u) << u;
    }
    // entries of a cell: nl lower ones first, then upper ones
    auto lowers = [&](int u) { return (int)((lower >> (4 * u)) & 15u); };
    auto entries = [&](int u) { return (int)((every >> (4 * u)) & 15u); };
    auto sweep_empty = [&] {
        renew();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = u * kResThreads + own0;
            if (l < n) reinterpret_cast<unsigned long long *>(sw)[l] = kSentinel;
        }
        for (int h = tid; h < H; h += kDicThreads) reinterpret_cast<unsigned long long *>(sw)[n + h] = kSentinel;
    };
    auto empty = [&](double *arr) {
        renew();
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = u * kResThreads + own0;
            if (l >= n) continue;
            const unsigned long long bit = 1ull << (tid & 63);
            if (shown[l >> 6] & bit) put_word(arr + p0 + l, kSentinel, tm.local && !(far[l >> 6] & bit));
        }
    };
    auto overdue = [&](int spin, long t0) {
        return (spin & 63) == 63 && (wall_clock64() - t0 > tm.ticks || *(volatile int *)&sh.late);
    };
    // the halo words a sweep needs (flag `need`), from the published array
    auto bring = [&](double *arr, uint32_t need, bool down) {
        constexpr int S = 64 * kDicBring;
        const int J = (H + kDicFlight * S - 1) / (kDicFlight * S);
        int j[kDicFlight], ha[kDicFlight], hl[kDicFlight];
        auto next = [&](int s) {
            ha[s] = -1;
            while (ha[s] < 0 && j[s] < J) {
                const int h = (tid - kResThreads) + S * (s + kDicFlight * (down ? J - 1 - j[s] : j[s]));
                const uint32_t v = h < H ? hid[h] : 0u;
                if (v & need) {
                    ha[s] = (int)(v & kDicPos);
                    hl[s] = n + h;
                }
                ++j[s];
            }
        };
#pragma unroll
        for (int s = 0; s < kDicFlight; ++s) {
            j[s] = hl[s] = 0;
            next(s);
        }
        const long t0 = wall_clock64();
#pragma unroll 1
        for (int spin = 0;; ++spin) {
            unsigned long long g[kDicFlight];
            bool more = false;
#pragma unroll
            for (int s = 0; s < kDicFlight; ++s) g[s] = ha[s] >= 0 ? gld(arr + ha[s]) : kSentinel;
#pragma unroll
            for (int s = 0; s < kDicFlight; ++s) {
                if (g[s] != kSentinel) {
                    lds_put(sw + hl[s], __longlong_as_double((long long)g[s]));
                    next(s);
                }
                more = more || ha[s] >= 0;
            }
            if (!__any(more)) break;
            if (overdue(spin, t0)) {
                sh.late = 1;
                break;
            }
        }
    };
    // A sweep over the thread's cells, first to last or (backward) last to
    // first:
    // MODE 0: D = A_ii - sum a^2 / D_j over the lower entries, into rD (1 / D)
    // MODE 1: y = (r - sum a y_j) rD, into w
    // MODE 2: z = y - (sum a z_j) rD over the upper entries, left in sw;
    //         returns the thread's sum of r z
    // A look forms the value from whatever is there: an empty word makes it
    // NaN.  State held in registers instead of LDS and the L2 made the change
    // from one cell to the next, 2.8 us, the bound of the sweep.
    auto compute = [&](auto mode, double *arr) {
        constexpr int MODE = decltype(mode)::value;
        constexpr bool down = MODE == 2;
        int ne[W];
        double na[W], nown = 0.0, nrd = 0.0, nr = 0.0, rz = 0.0;
        // what cell number at needs, on its way while the one before waits;
        // no branch but for the further entries
        auto ahead = [&](int at) {
            const int u = down ? U - 1 - at : at, first = down ? lowers(u) : 0, cnt = down ? entries(u) - first : lowers(u);
            const bool has = u * kResThreads + own0 < n;
            const unsigned int q = has ? (unsigned int)(u * kResThreads + own0) : 0u;
            auto entry = [&](int k) {
                const bool on = has && k < cnt;
                const unsigned int at_k = (on ? (unsigned int)((first + k) * n) : 0u) + q;
                const double v = coef[at_k];
                const int i = idx[at_k];
                na[k] = on ? v : 0.0;
                ne[k] = on ? i : none;
            };
#pragma unroll
            for (int k = 0; k < kDicFew; ++k) entry(k);
            if (((down ? more_up : more_lo) >> u) & 1u)
#pragma unroll
                for (int k = kDicFew; k < W; ++k) entry(k);
            nown = MODE == 0 ? dl[q] : MODE == 1 ? r[q] : w[q];
            if (MODE != 0) nrd = rD[q];
            if (MODE == 2) nr = r[q];
        };
        ahead(0);
        const long t0 = wall_clock64();
#pragma unroll 1
        for (int c = 0; c < U; ++c) {
            const int u = down ? U - 1 - c : c, l = u * kResThreads + own0;
            const bool live = l < n, many = ((down ? more_up : more_lo) >> u) & 1u;
            const double own = nown, rd = nrd, rl = nr;
            double a[W], out = 0.0;
            int e[W];
#pragma unroll
            for (int k = 0; k < W; ++k) {
                a[k] = na[k];
                e[k] = ne[k];
            }
            if (c + 1 < U) ahead(c + 1);
            // the looks, at the first K entries (those past the last are a
            // zero times the word that holds 1).  A value that is no number
            // by itself is told from an empty word at every 16th look only.
            const unsigned long long bit = 1ull << (tid & 63);
            const bool show = shown[l >> 6] & bit, near = tm.local && !(far[l >> 6] & bit);
            auto looks = [&](auto count) {
                constexpr int K = decltype(count)::value;
                unsigned long long open = __ballot(live);
#pragma unroll 1
                for (int spin = 0; open; ++spin) {
                    double b[K], acc = MODE == 2 ? 0.0 : own;
#pragma unroll
                    for (int k = 0; k < K; ++k) b[k] = lds_word(sw + e[k]);
#pragma unroll
                    for (int k = 0; k < K; ++k) {
                        if (MODE == 0) acc -= a[k] * a[k] / b[k];
                        else if (MODE == 1) acc -= a[k] * b[k];
                        else acc += a[k] * b[k];
                    }
                    out = MODE == 0 ? acc : MODE == 1 ? acc * rd : own - acc * rd;
                    unsigned long long full = __ballot(out == out);
                    if ((spin & 15) == 15) {
                        bool all = true;
#pragma unroll
                        for (int k = 0; k < K; ++k) all = all && !lds_empty(b[k]);
                        full = __ballot(all);
                        if (overdue(spin, t0)) {
                            sh.late = 1;
                            break;
                        }
                    }
                    full &= open;
                    if (full == 0) continue;
                    open &= ~full;
                    if ((full >> (tid & 63)) & 1ull) {
                        lds_put(sw + l, out);
                        if (show) put_word(arr + p0 + l, slot_word(out), near);
                    }
                }
            };
            if (!many) looks(std::integral_constant<int, kDicFew>{});
            else looks(std::integral_constant<int, W>{});
            if (live) {
                if (MODE == 0) {
                    rD[l] = 1.0 / out;
                    gmem(d.dstar)[index(l)] = out;
                } else if (MODE == 1) w[l] = out;
                else rz += rl * out;
            }
            renew();
        }
        return rz;
    };
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto sweep = [&](auto mode, double *arr) {
        constexpr bool down = decltype(mode)::value == 2;
        if (wave < kResWaves) return compute(mode, arr);
        bring(arr, down ? kDicHigh : kDicLow, down);
        return 0.0;
    };

    if (tid == 0) {
        v3[1] = (double)xcc_id();
        v3[2] = v3[1] * v3[1];
    }
    if (!res_reduce<3, true>(v3, tm, sh)) return false;
    tm.local = sh.local;
    const double xbar = uniform(v3[0] / (double)d.N);
    // the factor D*
    sweep(std::integral_constant<int, 0>{}, yg);
    for (int h = tid; h < H; h += kDicThreads) loc[n + h] = __longlong_as_double((long long)gld(xx + (hid[h] & kDicPos)));
    __syncthreads();
    if (sh.late) return false;
    sweep_empty();
    v3[0] = v3[1] = v3[2] = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int l = u * kResThreads + own0;
        if (l >= n) continue;
        // upper entries, then lower ones: the order of row_apply and row_sum
        const int nl = lowers(u);
        double ax = dl[l] * loc[l], a1 = dl[l];
        for (int up = 1; up >= 0; --up)
#pragma unroll
            for (int k = 0; k < W; ++k)
                if ((k >= nl) == (up != 0)) {
                    const double a = coef[k * n + l];
                    ax += a * loc[idx[k * n + l]];
                    a1 += a;
                }
        const double b = gmem((const double *)d.pb)[index(l)];
        const double rl = b - ax;
        r[l] = rl;
        v3[0] += fabs(ax - xbar * a1) + fabs(b - xbar * a1);
        v3[1] += fabs(rl);
    }
    if (!res_reduce<3>(v3, tm, sh)) return false;
    empty(yg);   // every part has its D*
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
    {
        double none[1] = {0.0};
        if (!res_reduce<1>(none, tm, sh)) return false;
    }

    while (!s.done) {
        renew();
        // z = M^-1 r: forward, backward
        sweep(std::integral_constant<int, 1>{}, yg);
        __syncthreads();
        if (sh.late) return false;
        sweep_empty();
        __syncthreads();
        double rz[1] = {sweep(std::integral_constant<int, 2>{}, zg)};
        if (!res_reduce<1>(rz, tm, sh) || sh.late) return false;   // its barrier ends the sweep in the part
        if (!(rz[0] > 0.0) || !isfinite(rz[0])) {
            set_done(s, FVM_ENUMERIC);
            s.iters += 1;
            break;
        }
        s.beta = s.iters == 0 ? 0.0 : uniform(rz[0] / s.rho);
        s.rho = uniform(rz[0]);
        empty(yg);
        // p = z + beta p: own cells and, from the published z, the halo
        renew();
        const double beta = s.beta;
        const bool first = s.first;
        for (int base = tid; base < H; base += kHaloStep * kDicThreads) {
            unsigned long long zb[kHaloStep];
#pragma unroll
            for (int j = 0; j < kHaloStep; ++j) {
                const int h = base + j * kDicThreads;
                zb[j] = h < H ? gld(zg + (hid[h] & kDicPos)) : 0ull;
            }
#pragma unroll
            for (int j = 0; j < kHaloStep; ++j) {
                const int h = base + j * kDicThreads;
                const double z = __longlong_as_double((long long)zb[j]);
                if (h < H) loc[n + h] = first ? z : z + beta * loc[n + h];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = u * kResThreads + own0;
            if (l < n) loc[l] = first ? sw[l] : sw[l] + beta * loc[l];
        }
        sweep_empty();   // each word by the thread that read it
        __syncthreads();
        renew();
        double pq[1] = {0.0};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = u * kResThreads + own0;
            if (l >= n) continue;
            const double pu = loc[l];
            double q = dl[l] * pu;
#pragma unroll
            for (int k = 0; k < W; ++k) q += coef[k * n + l] * loc[idx[k * n + l]];
            w[l] = q;
            pq[0] += pu * q;
        }
        if (!res_reduce<1>(pq, tm, sh)) return false;
        if (!(pq[0] > 0.0) || !isfinite(pq[0])) {
            set_done(s, FVM_ENUMERIC);
            s.iters += 1;
            break;
        }
        s.alpha = uniform(s.rho / pq[0]);
        empty(zg);
        double v1[1] = {0.0};
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int l = u * kResThreads + own0;
            if (l >= n) continue;
            const double rl = r[l] - s.alpha * w[l];
            r[l] = rl;
            v1[0] += fabs(rl);
            xg[l] += s.alpha * loc[l];
        }
        if (!res_reduce<1>(v1, tm, sh)) return false;
        s.iters += 1;
        s.nres = uniform(v1[0] / s.nf);
        s.first = 0;
        if (!isfinite(s.nres)) set_done(s, FVM_ENUMERIC);
        else if (s.nres <= s.tol_eff) set_done(s, FVM_OK);
        else if (s.iters >= s.max_iter) set_done(s, FVM_WARN_MAXITER);
    }
    renew();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int l = u * kResThreads + own0;
        if (l < n) gmem(d.p)[index(l)] = xg[l];
    }
    if (tid == 0) d.res_fin[part] = ctl.serial;
    if (part == 0 && tid == 0) d.ks[3] = s;
    return true;
}

template <int W>
__global__ void __launch_bounds__(kDicThreads) k_res_dic(Batch bt, ResMap map, ResCtl ctl, long ticks)
{
    extern __shared__ __align__(16) double res_lds[];
    __shared__ ResRed sh;
    const int c = map.cs[blockIdx.x];
    if (c >= bt.n) return;
    const DevCase &d = *bt.dc[c];
    ResTeam tm = res_team(d, map.pt[blockIdx.x], ticks);
    const bool ok = res_solve_dic<W>(d, tm, ctl, sh, res_lds);
    res_end(d, tm, ok);
}
