// The linear algebra and kinetics of the wave-per-cell integrator: one cell's
// right-hand side, Newton matrix and linear solve on 64 lanes.
//
// What bounds it: a cell is a serial chain of right-hand sides (400 per cell
// of the 35-species flame at dt = 1e-6), each a short piece of work for 64
// lanes, at two waves per SIMD; latency and FP64 issue, not memory.  So
//  * the tables come lane by lane (wave_tables.h), every load coalesced and
//    independent of the state, instead of each lane walking its species' list
//    of reactions and fetching 64-byte reaction records;
//  * production sums and Jacobian entries are dealt out evenly over the 64
//    lanes (the busiest of the 35 species takes part in 39 of 200 reactions,
//    the mean in 23), each with a fixed order of summation;
//  * the Newton matrix lives in registers, one row per lane, and is inverted
//    in place by Gauss-Jordan elimination with row pivoting: a refresh serves
//    about nine solves, and a solve is then one matrix-vector product of
//    independent multiply-adds instead of 2 N dependent substitution steps.
// Measured against the walk over species lists with an LU in LDS: 65,536
// cells of the 35-species flame 419 -> 158 ms (FP32 matrix, 16,383 cells:
// 72.8 -> 39.0), 20,011 cells of the 20-species one 17.5 -> 6.9 ms.  VALU issue
// is now 76 % of the time of the 35-species kernel.
// Included by bdf_wave.hip, inside its namespace.

// Largest |v| of the candidate lanes (lowest lane on ties), -1 if no
// candidate has a comparable value.  Compared by the bits of |v|, which order
// like the values: the high words first, the low words only among equals.
template <int CTRL>
__device__ __forceinline__ int dpp_max(int v)
{
    const int o = dpp_i32<CTRL>(v);
    return v > o ? v : o;
}

// maximum of v >= -1 over the lanes below NP, the same in all
template <int NP>
__device__ __forceinline__ int rows_max(int v)
{
    v = dpp_max<0xB1>(v);
    v = dpp_max<0x4E>(v);
    v = dpp_max<0x141>(v);
    v = dpp_max<0x140>(v);
    int best = __builtin_amdgcn_readlane(v, 15);
    if constexpr (NP > 16) best = max(best, __builtin_amdgcn_readlane(v, 31));
    if constexpr (NP > 32) best = max(best, __builtin_amdgcn_readlane(v, 47));
    if constexpr (NP > 48) best = max(best, __builtin_amdgcn_readlane(v, 63));
    return best;
}

template <int NP>
__device__ __forceinline__ int pivot_lane(double v, bool cand)
{
    const long long b = __double_as_longlong(v);
    const int hi = cand && v == v ? (int)(b >> 32) & 0x7fffffff : -1;
    const int best = rows_max<NP>(hi);
    if (best < 0) return -1;
    unsigned long long mask = __ballot(hi == best);
    if (mask & (mask - 1)) {
        // equal high words: the low words decide (as two 16-bit halves, to stay in signed range)
        const int lo = (int)(b & 0xffffffffll);
        int key = hi == best ? (lo >> 16) & 0xffff : -1;
        int top = rows_max<NP>(key);
        const bool in = key == top && hi == best;
        key = in ? lo & 0xffff : -1;
        top = rows_max<NP>(key);
        mask = __ballot(in && key == top);
    }
    return (int)__ffsll((long long)mask) - 1;
}

template <int NP>
__device__ __forceinline__ int pivot_lane(float v, bool cand)
{
    const int key = cand && v == v ? __float_as_int(v) & 0x7fffffff : -1;
    const int best = rows_max<NP>(key);
    if (best < 0) return -1;
    return (int)__ffsll((long long)__ballot(key == best)) - 1;
}

__device__ __forceinline__ float rcp_lt(float x) { return 1.0f / x; }
__device__ __forceinline__ double rcp_lt(double x) { return rcp_d(x); }

template <int NP, typename LT>
struct Wave64Lds {
    double C[64], g[64], h[64];   // concentrations, G/RT and H/RT of the species, the sentinel's at K
    double part[64];              // production: every lane's partial sum
    LT J[NP * (NP + 1) + 1];      // Jacobian rows; last: target of padded entries.  Entries no
                                  // reaction reaches stay 0 from the start
};

// RPL: reactions per lane, unrolled, whose rate constants a refresh keeps in
// registers (0: any number, their rate constants in the scratch); QLDS: the scratch
// is in LDS.
template <int NP, typename LT, int RPL, bool QLDS>
struct WaveSys {
    static constexpr int G = 64;
    static constexpr bool kUniformOrder = true;    // one cell per wave: one order
    static constexpr int LDJ = NP + 1;
    using Gp = Grp<64>;
    const DevMechView &m;
    const Wave64Tables &wt;
    Wave64Lds<NP, LT> &L;
    double *P;        // scratch, layout in wave_tables.h
    int K, R, lane;
    double W, invW;   // of this lane's species (0 beyond)
    double tmid;
    int xfirst, xcount;
    LT a[NP];         // this lane's row of the inverse, columns moved (see invert)
    LT rpl;           // reciprocal of this lane's pivot
    int pj, pk;       // pivot row of the column in a[lane], resp. of component `lane`

    __device__ WaveSys(const DevMechView &m_, const Wave64Tables &wt_, Wave64Lds<NP, LT> &L_, double *P_)
        : m(m_), wt(wt_), L(L_), P(P_), K(m_.K), R(m_.R), lane(Gp::lane())
    {
        W = lane < K ? m.W[lane] : 0.0;
        invW = lane < K ? m.invW[lane] : 0.0;
        tmid = wt.tmid[lane];
        const int x = wt.xseg[lane];
        xfirst = x & 0xff;
        xcount = x >> 8;
        for (int i = lane; i < NP * LDJ + 1; i += 64) L.J[i] = (LT)0;
        if (lane == 0) P[0] = 0.0;
        rpl = (LT)0;
        pj = pk = lane;
        sync();
    }

    // LDS (or scratch) written by some lanes of the wave, then read by others:
    // one wave's LDS instructions execute in order, so only the compiler has
    // to keep theirs; a scratch in global memory needs the wait
    __device__ __forceinline__ static void sync()
    {
        if constexpr (QLDS) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        } else {
            Gp::sync();
        }
    }

    // double at byte offset `off` of the scratch
    __device__ __forceinline__ double at_off(uint32_t off) const { return *(const double *)((const char *)P + off); }

    __device__ __forceinline__ void thermo(double T, double invT, double lnT, double &cp, double &h, double &g,
                                           double &dcp) const
    {
        const double2 *c = wt.th + (m.two_range && !(T < tmid) ? 7 * 64 : 0) + lane;
        const double2 c0 = c[0], c1 = c[64], c2 = c[128], c3 = c[192], c4 = c[256], c5 = c[320], c6 = c[384];
        cp = c0.x + T * (c0.y + T * (c1.x + T * (c1.y + T * c2.x)));
        h = c0.x + T * (c3.y + T * (c4.x + T * (c4.y + T * c5.x))) + c2.y * invT;
        g = h - (c0.x * lnT + T * (c0.y + T * (c5.y + T * (c6.x + T * c6.y))) + c3.x);
        dcp = c0.y + T * (2.0 * c1.x + T * (3.0 * c1.y + T * 4.0 * c2.x));
    }

    // sum over the reactions of net coefficient times the value at 1 + r (its
    // negative at 1 + R + r), for lane's species
    __device__ __forceinline__ double produce() const
    {
        double s = 0.0;   // in reaction order
        auto add = [&](const uint4 &e) __attribute__((always_inline)) {
            s += at_off(e.x);
            s += at_off(e.y);
            s += at_off(e.z);
            s += at_off(e.w);
        };
        // every table entry is fetched before the first sum and every value
        // read before the first addition, the quads counted at compile time
        auto quads = [&](auto nc, int i0 = 0) __attribute__((always_inline)) {
            constexpr int n = decltype(nc)::value;
            uint4 e[n];
#pragma unroll
            for (int i = 0; i < n; i++) e[i] = wt.gat[(i0 + i) * 64 + lane];
#pragma unroll
            for (int i = 0; i < n; i++) add(e[i]);
        };
        if constexpr (RPL == 0) {
            // many reactions: long sums, the more so from a scratch in global memory
            int i = 0;
            for (; i + 6 <= wt.gather4; i += 6) quads(std::integral_constant<int, 6>{}, i);
            for (; i < wt.gather4; i++) quads(std::integral_constant<int, 1>{}, i);
        } else {
            switch (wt.gather4) {
            case 1: quads(std::integral_constant<int, 1>{}); break;
            case 2: quads(std::integral_constant<int, 2>{}); break;
            case 3: quads(std::integral_constant<int, 3>{}); break;
            case 4: quads(std::integral_constant<int, 4>{}); break;
            case 5: quads(std::integral_constant<int, 5>{}); break;
            case 6: quads(std::integral_constant<int, 6>{}); break;
            default:
#pragma clang loop unroll(disable)
                for (int i = 0; i < wt.gather4; i++) add(wt.gat[i * 64 + lane]);
            }
        }
        L.part[lane] = s;
        sync();
#pragma clang loop unroll(disable)
        for (int j = 0; j < wt.extras; j++) {
            const double x = L.part[(xfirst + j) & 63];
            s += j < xcount ? x : 0.0;
        }
        return s;
    }

    // mixture sums at the state yi, species data to LDS
    struct Mix {
        double T, invT, lnT, cpk, hk, gk, dcpk, sumYW, rho, cpm;
    };
    __device__ __forceinline__ Mix mixture(double p, double yi)
    {
        Mix x;
        x.T = Gp::at(yi, K);
        x.invT = 1.0 / x.T;
        x.lnT = log(x.T);
        thermo(x.T, x.invT, x.lnT, x.cpk, x.hk, x.gk, x.dcpk);
        x.sumYW = Gp::sum(yi * invW);   // 0 beyond the species
        x.cpm = kRu * Gp::sum(yi * x.cpk * invW);
        x.rho = p / (kRu * x.T * x.sumYW);
        if (lane < K) {
            L.C[lane] = x.rho * yi * invW;
            L.g[lane] = x.gk;
            L.h[lane] = x.hk;
        } else if (lane == K) {
            L.C[lane] = 1.0;
            L.g[lane] = 0.0;
            L.h[lane] = 0.0;
        }
        sync();
        return x;
    }

    struct Slots {
        int r0, r1, p0, p1;
    };
    static __device__ __forceinline__ Slots slots(uint32_t w)
    {
        return Slots{(int)(w & 63u), (int)(w >> 6 & 63u), (int)(w >> 12 & 63u), (int)(w >> 18 & 63u)};
    }

    // f(i, record) for this lane's reactions i * 64 + lane.  Beyond the register
    // builds each record is fetched ahead of the work on the one before: the compiler
    // cannot move a table read over a write to a scratch in global memory.  (With the
    // other fetches ahead below and 48 rows where they suffice: 12,000 cells of 45
    // species and 900 elementary reactions 120 -> 93 ms, with FP32 matrix 97 -> 83.)
    struct Record {
        double2 ka, kb;
        uint32_t w;
    };
    template <class F>
    __device__ __forceinline__ void each_reaction(F &&f) const
    {
        auto fetch = [&](int i) __attribute__((always_inline)) {
            return Record{wt.rx[(2 * i) * 64 + lane], wt.rx[(2 * i + 1) * 64 + lane], wt.rw[i * 64 + lane]};
        };
        if constexpr (RPL > 0) {
#pragma unroll
            for (int i = 0; i < RPL; i++) f(i, fetch(i));
        } else {
            Record rec = fetch(0);
            for (int i = 0; i < wt.rounds; i++) {
                const Record next = fetch(i + 1 < wt.rounds ? i + 1 : 0);
                f(i, rec);
                rec = next;
            }
        }
    }

    // f(y): each lane passes its component yi and receives fi
    __device__ __forceinline__ double rhs(double p, double yi)
    {
        const Mix x = mixture(p, yi);
        const double ln_c0 = log(kPstd / kRu) - x.lnT;
        each_reaction([&](int i, const Record &rec) __attribute__((always_inline)) {
            const int r = i * 64 + lane;
            const double2 ka = rec.ka, kb = rec.kb;
            const uint32_t w = rec.w;
            const Slots s = slots(w);
            const double lnkf = ka.x + ka.y * x.lnT - kb.x * x.invT;
            const double dg = L.g[s.p0] + L.g[s.p1] - L.g[s.r0] - L.g[s.r1];
            const double lnkr = lnkf + dg - kb.y * ln_c0;
            const double fwd = exp(lnkf) * L.C[s.r0] * L.C[s.r1];
            double q = (w & kRxnWordIrrev) ? fwd : fwd - exp(lnkr) * L.C[s.p0] * L.C[s.p1];
            if constexpr (kPD) {
                const int kind = (int)(w >> 24 & 7u);
                if (kind != kRxnElem) {
                    const DevRxn rx = m.rxn[r];
                    const double M = third_body(rx, m.aux, x.rho * x.sumYW, [&](int l) { return L.C[l]; });
                    q *= pdep_rate<false>(kind, m.aux + rx.aux, M, x.T, x.lnT, x.invT, lnkf, 0.0).mult;
                }
            }
            if (r < R) {
                P[1 + r] = q;
                P[1 + R + r] = -q;
            }
        });
        sync();
        const double w0 = produce();
        const double wk = lane < K ? w0 : 0.0;
        const double heat = Gp::sum(x.hk * wk);
        sync();
        const double fk = W * wk / x.rho, fT = -(kRu * x.T) * heat / (x.rho * x.cpm);
        return lane < K ? fk : (lane == K ? fT : 0.0);
    }

    // Inverse of M = I - gamma J at the state yi; false if M is singular.
    __device__ __forceinline__ bool refresh(double p, double yi, double gamma)
    {
        const int N = K + 1;
        const Mix x = mixture(p, yi);
        const double T = x.T, invT = x.invT, rho = x.rho, cpm = x.cpm;
        const double wbar = 1.0 / x.sumYW;
        const double dcpm = kRu * Gp::sum(yi * x.dcpk * invW);
        const double ln_c0 = log(kPstd / kRu) - x.lnT;
        // per reaction: rate constants (registers, or behind the derivatives
        // in the scratch), G = dq/d[M] of a pressure-dependent one
        double *gM = P + 1 + 4 * R, *kfs = gM + (kPD ? R : 0), *krs = kfs + R;
        double kfv[RPL > 0 ? RPL : 1], krv[RPL > 0 ? RPL : 1];
        each_reaction([&](int i, const Record &rec) __attribute__((always_inline)) {
            const int r = i * 64 + lane;
            const double2 ka = rec.ka, kb = rec.kb;
            const uint32_t w = rec.w;
            const Slots s = slots(w);
            const double lnkf = ka.x + ka.y * x.lnT - kb.x * invT;
            const double dg = L.g[s.p0] + L.g[s.p1] - L.g[s.r0] - L.g[s.r1];
            const double dh = L.h[s.p0] + L.h[s.p1] - L.h[s.r0] - L.h[s.r1];
            const double lnkr = lnkf + dg - kb.y * ln_c0;
            const double dlnk = (ka.y + kb.x * invT) * invT;
            const double cr0 = L.C[s.r0], cr1 = L.C[s.r1], cp0 = L.C[s.p0], cp1 = L.C[s.p1];
            const double k0f = exp(lnkf), k0r = (w & kRxnWordIrrev) ? 0.0 : exp(lnkr);
            PdepRate pd{1.0, 0.0, 0.0};
            double M = 0.0;
            if constexpr (kPD) {
                const int kind = (int)(w >> 24 & 7u);
                if (kind != kRxnElem) {
                    const DevRxn rx = m.rxn[r];
                    M = third_body(rx, m.aux, rho * x.sumYW, [&](int l) { return L.C[l]; });
                    pd = pdep_rate<true>(kind, m.aux + rx.aux, M, T, x.lnT, invT, lnkf, dlnk);
                }
            }
            const double kf = kPD ? k0f * pd.mult : k0f, kr = kPD ? k0r * pd.mult : k0r;
            const double fwd = kf * cr0 * cr1, rev = kr * cp0 * cp1;
            const double mf = s.r1 != K ? 2.0 : 1.0, mr = s.p1 != K ? 2.0 : 1.0;
            const double dlnkf = kPD ? dlnk + pd.dlnT : dlnk;
            const double dlnkr = dlnkf - (dh - kb.y) * invT;
            double qh = mf * fwd - mr * rev;   // sum_l C_l dq/dC_l
            if constexpr (kPD) {
                const double g = pd.dM * (k0f * cr0 * cr1 - k0r * cp0 * cp1);
                qh += g * M;
                if (r < R) gM[r] = g;
            }
            if (r < R) {
                const double q = fwd - rev;
                P[1 + r] = q;
                P[1 + R + r] = -q;
                P[1 + 2 * R + r] = qh;
                P[1 + 3 * R + r] = fwd * dlnkf - rev * dlnkr;   // dq/dT
            }
            if constexpr (RPL > 0) {
                kfv[i] = kf;
                krv[i] = kr;
            } else if (r < R) {
                kfs[r] = kf;
                krs[r] = kr;
            }
        });
        auto all = [&](auto &&f) __attribute__((always_inline)) {
            if constexpr (RPL > 0) {
#pragma unroll
                for (int i = 0; i < RPL; i++) f(i);
            } else {
                for (int i = 0; i < wt.rounds; i++) f(i);
            }
        };
        // production sums of q, qh and dq/dT: each value in turn at the two
        // places the production table reads
        auto move = [&](int from) __attribute__((always_inline)) {
            auto put = [&](int r, double v) __attribute__((always_inline)) {
                P[1 + r] = v;
                P[1 + R + r] = -v;
            };
            if constexpr (RPL > 0) {
#pragma unroll
                for (int i = 0; i < RPL; i++) {
                    const int r = i * 64 + lane;
                    if (r < R) put(r, P[1 + from * R + r]);
                }
            } else {
                for (int i0 = 0; i0 < wt.rounds; i0 += 4) {
                    double v[4];   // read before the first is written
#pragma unroll
                    for (int i = 0; i < 4; i++) v[i] = P[1 + from * R + min((i0 + i) * 64 + lane, R - 1)];
#pragma unroll
                    for (int i = 0; i < 4; i++)
                        if ((i0 + i) * 64 + lane < R) put((i0 + i) * 64 + lane, v[i]);
                }
            }
            sync();
        };
        sync();
        const double w0 = produce();
        const double wk = lane < K ? w0 : 0.0;
        sync();
        move(2);
        const double w1 = produce();
        const double ACk = lane < K ? w1 : 0.0;
        sync();
        move(3);
        const double w2 = produce();
        const double wTk = lane < K ? w2 : 0.0;
        sync();
        all([&](int i) __attribute__((always_inline)) {
            const int r = i * 64 + lane;
            if (r < R) {
                const Slots s = slots(wt.rw[r]);
                const double kf = RPL > 0 ? kfv[RPL > 0 ? i : 0] : kfs[r], kr = RPL > 0 ? krv[RPL > 0 ? i : 0] : krs[r];
                P[1 + 4 * r + 0] = kf * L.C[s.r1];
                P[1 + 4 * r + 1] = kf * L.C[s.r0];
                P[1 + 4 * r + 2] = -kr * L.C[s.p1];
                P[1 + 4 * r + 3] = -kr * L.C[s.p0];
            }
        });
        sync();
        // entries of the species block
        for (int i = 0; i < wt.jrounds; i++) {
            const int2 c = wt.jcnt[i];
            const uint32_t rc = wt.jrc[i * 64 + lane];
            const uint32_t *con = wt.jcon + (size_t)c.x * 64 + lane;
            double s = 0.0;
            uint32_t e[4], f[4];   // the next four contributions are fetched while these are added
#pragma unroll
            for (int j = 0; j < 4; j++) e[j] = con[j * 64];
            auto add = [&](uint32_t k, double v) __attribute__((always_inline)) { s += (int)k < 0 ? -v : v; };
            if constexpr (QLDS) {
#pragma clang loop unroll(disable)
                for (int j0 = 4; j0 <= c.y; j0 += 4) {
                    const int jn = j0 < c.y ? j0 : 0;
#pragma unroll
                    for (int j = 0; j < 4; j++) f[j] = con[(jn + j) * 64];
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        add(e[j], at_off(e[j] & 0x7fffffffu));
                        e[j] = f[j];
                    }
                }
            } else {
                // and their values too, from global memory
                double v[4], u[4];
                const int j4 = c.y > 4 ? 4 : 0;
#pragma unroll
                for (int j = 0; j < 4; j++) f[j] = con[(j4 + j) * 64];
#pragma unroll
                for (int j = 0; j < 4; j++) v[j] = at_off(e[j] & 0x7fffffffu);
#pragma clang loop unroll(disable)
                for (int j0 = 4; j0 <= c.y; j0 += 4) {
                    const int jn = j0 + 4 < c.y ? j0 + 4 : 0;
                    uint32_t g[4];
#pragma unroll
                    for (int j = 0; j < 4; j++) g[j] = con[(jn + j) * 64];
#pragma unroll
                    for (int j = 0; j < 4; j++) u[j] = at_off(f[j] & 0x7fffffffu);
#pragma unroll
                    for (int j = 0; j < 4; j++) {
                        add(e[j], v[j]);
                        e[j] = f[j];
                        f[j] = g[j];
                        v[j] = u[j];
                    }
                }
            }
            const bool pad = rc == 0xFFFFu;
            const int row = pad ? 0 : (int)(rc & 0xff), col = pad ? 0 : (int)(rc >> 8);
            L.J[pad ? NP * LDJ : row * LDJ + col] = (LT)(s * (m.W[row] * wt.invw[col]));
        }
        sync();
        double uk = 0.0;
        if constexpr (kPD) {
            // through [M]: the default efficiency on every column (added with
            // the rank-one term below), the listed ones here
            for (int j = wt.poff[lane]; j < wt.poff[lane + 1]; j++) {
                const int2 ent = wt.pent[j];
                const DevRxn rx = m.rxn[ent.x];
                const double gn = (double)ent.y * gM[ent.x];
                uk += gn * rx.def_eff;
                const double *ef = m.aux + rx.aux + kAuxHead;
                for (int t = 0; t < rx.neff; t++) {
                    const int l = (int)ef[2 * t];
                    L.J[lane * LDJ + l] += (LT)(gn * ef[2 * t + 1] * W * m.invW[l]);
                }
            }
            sync();
        }
        const double RT = kRu * T;
        const double inv_rcp = 1.0 / (rho * cpm);
        const double S = RT * Gp::sum(x.hk * wk);
        const double hAC = Gp::sum(x.hk * ACk);
        const double dST = Gp::sum(kRu * x.cpk * wk + RT * x.hk * (wTk - ACk * invT));
        double hU = 0.0;
        if constexpr (kPD) hU = Gp::sum(x.hk * uk);
        // temperature row: lane j sums column j over the species rows
        double JT = 0.0;
        {
            double col = 0.0;
            const LT *Jc = L.J + (lane < K ? lane : 0);
#pragma unroll 4
            for (int k = 0; k < K; k++) col += (double)Jc[k * LDJ] * (L.h[k] * m.invW[k]);
            if constexpr (kPD) col += invW * hU;
            const double dS = RT * rho * (col - (wbar / rho) * invW * hAC);
            const double drcp = rho * invW * (kRu * x.cpk - cpm * wbar);
            const double drcpT = rho * dcpm - cpm * rho * invT;
            JT = lane < K ? (-dS + S * drcp * inv_rcp) * inv_rcp : (-dST + S * drcpT * inv_rcp) * inv_rcp;
        }
        const double gq = wbar / rho;
        const double u = W * (kPD ? gq * (wk - ACk) + uk : gq * (wk - ACk));   // 0 beyond the species
        if (lane < K) L.J[lane * LDJ + K] = (LT)(W / rho * (wTk + (wk - ACk) * invT));
        if (lane < N) L.J[K * LDJ + lane] = (LT)JT;
        sync();
        // this lane's row of M (columns from N on and lanes from N on: identity)
        {
            const LT *Jr = L.J + (lane < N ? lane : 0) * LDJ;
            const double gl = lane < N ? gamma : 0.0;
            int ln = lane;   // opaque, so that the identity is not kept in registers across the integration
            asm volatile("" : "+v"(ln));
#pragma unroll
            for (int c = 0; c < NP; c++)
                a[c] = (LT)((c == ln ? 1.0 : 0.0) - gl * ((double)Jr[c] + u * wt.invw[c]));
        }
        return invert(N);
    }

    // Gauss-Jordan inversion in place with row pivoting, four steps at a time:
    // steps k .. k + 3 eliminate the columns held in a[0] .. a[3], whose places
    // take the new columns of the inverse, then the columns move up by four
    // places (the new ones last), so that the loop body is the same code for
    // every k and every broadcast reads a fixed register.  In the end column j
    // of the inverse (belonging to the row that was pivot j) is in
    // a[shift + j]; rows stay on their lanes and unscaled, row p_k (pivot k)
    // holds component k.
    static __device__ __forceinline__ int shift(int N) { return NP - ((N + 3) & ~3); }
    __device__ __forceinline__ bool invert(int N)
    {
        static_assert(NP % 4 == 0, "four steps per pass");
        bool ok = true, used = lane >= N;
        pj = lane;
        pk = lane;
        const int sh = shift(N);
#pragma clang loop unroll(disable)
        for (int k0 = 0; k0 < N; k0 += 4) {
            static_for<0, 4>([&](auto sc) __attribute__((always_inline)) {
                constexpr int s = decltype(sc)::value;
                const int k = k0 + s;
                if (k < N) {
                    int p = pivot_lane<NP>(a[s], !used);
                    if (p < 0) {   // no comparable value (NaN column): any open row, fail below
                        p = (int)__ffsll((long long)__ballot(!used)) - 1;
                        ok = false;
                    }
                    p = __builtin_amdgcn_readfirstlane(p);
                    const LT piv = Gp::at(a[s], p);
                    ok = ok && piv != (LT)0;
                    const LT rp = rcp_lt(piv);
                    const bool is_p = lane == p;
                    used = used || is_p;
                    pj = lane == sh + k ? p : pj;
                    pk = lane == k ? p : pk;
                    rpl = is_p ? rp : rpl;
                    const LT t = is_p ? (LT)0 : a[s] * rp;
                    // broadcasts in groups ahead of their multiply-adds
                    static_for<0, (NP + 5) / 6>([&](auto gc) __attribute__((always_inline)) {
                        constexpr int c0 = decltype(gc)::value * 6;
                        LT u[6];
#pragma unroll
                        for (int c = 0; c < 6; c++)
                            if (c0 + c < NP && c0 + c != s) u[c] = Gp::at(a[c0 + c], p);
#pragma unroll
                        for (int c = 0; c < 6; c++)
                            if (c0 + c < NP && c0 + c != s) a[c0 + c] -= t * u[c];
                    });
                    a[s] = is_p ? (LT)1 : -t;
                }
            });
            LT b[4];
#pragma unroll
            for (int c = 0; c < 4; c++) b[c] = a[c];
#pragma unroll
            for (int c = 0; c + 4 < NP; c++) a[c] = a[c + 4];
#pragma unroll
            for (int c = 0; c < 4; c++) a[NP - 4 + c] = b[c];
        }
        return ok;
    }

    // x = M^-1 b
    __device__ __forceinline__ double solve(double bi) const
    {
        const int N = K + 1;
        const double bp = Gp::gather(bi, pj);
        const int sh = shift(N);
        const LT b = lane >= sh && lane < sh + N ? (LT)bp : (LT)0;
        LT s[3] = {(LT)0, (LT)0, (LT)0};
        static_for<0, (NP + 5) / 6>([&](auto gc) __attribute__((always_inline)) {
            constexpr int c0 = decltype(gc)::value * 6;
            LT u[6];
#pragma unroll
            for (int c = 0; c < 6; c++)
                if (c0 + c < NP) u[c] = Gp::at(b, c0 + c);
#pragma unroll
            for (int c = 0; c < 6; c++)
                if (c0 + c < NP) s[c % 3] += a[c0 + c] * u[c];
        });
        const double x = Gp::gather((double)((s[0] + s[1] + s[2]) * rpl), pk);
        return lane < N ? x : 0.0;
    }
};
