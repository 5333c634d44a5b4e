// sigk_team.h -- the forward sweep by teams of wavefronts, for launches whose
// time is the dependency chain of a few long pairs and not the chip's rate.
//
// A team is one workgroup: W compute waves on consecutive 64-row strips of a
// pair (the mapping and the cell map of sigk_strip.h) and one service wave.
// Consecutive strips of a team hand their frontier over through an LDS ring of
// edge columns, so a strip starts kSub + 64 steps behind the one below it; only
// the team's first strip reads, and its last one writes, the pair's frontier
// row in memory.  The service wave does everything that waits on memory: it
// fills the ring of x increments that all the team's waves read, polls the
// progress flag of the team below and fills the first strip's edge ring, and
// writes the last strip's edges out.  A compute wave's only wait is an LDS
// counter, tested once per kSub steps.
//
// Why: a lone wave issues a vector instruction about every 5.25 cycles, so a
// step takes its instruction count, and a pair of S strips takes
// (columns + S lags) steps.  With one wave per workgroup every strip pays the
// chunk's flag, frontier and increment round trips (about 3.8 us per 32 steps
// measured at order 6) and a lag of 95-127 steps.  Measured, one-wave kernel
// then team: 4096-point pair (d 8, order 6) 3.89 -> 3.05 ms, 200,001-point
// pair (d 8, order 5) 292 -> 227 ms, eight paths of 128 points (order 10) 214
// -> 188 us.  A step then costs about 290 ns at order 6 for 143 instructions,
// near the 5.25 cycles each that a lone wave needs.
//
// Progress counters (LDS, all counted from the team's start):
//   done[w]  steps completed by wave w; its top lane has then produced
//            columns below done - 63
//   x        columns of increments in the ring (service wave)
//   bot      columns in the first strip's edge ring (service wave)
//   out      columns of the last strip written to memory (service wave)
// A wave starts steps [t, t+kSub) once the strip below has produced their
// columns and the strip above has consumed what they overwrite.  Every wait is
// on a wave of the same workgroup, and the service wave waits only on teams
// with smaller tickets: no deadlock at any grid size.
#pragma once
#include "sigk_strip.h"

namespace sigk {

// Steps between two tests of the counters; the edge rings hold 4 kSub columns:
// a strip lags the one below it by at least 64 + kSub steps and its edge ring
// lets that one run at most 63 + 3 kSub ahead.  16 steps where a step is
// short; 8 where it is long (the test is nothing there and LDS is scarce).
template <int P>
constexpr int team_sub = team_steps(P);
template <int P>
constexpr int team_ec = 4 * team_sub<P>;

constexpr int kTeamX = 32;  // columns per increment chunk (and per Neumann depth)
constexpr int kTeamQ = 16;  // ring of the chunks' norm bounds

// Bytes of one column in the increment ring: its d channels, padded by 16
// bytes so that 16-byte reads of consecutive columns by consecutive lanes
// spread over all LDS banks.
template <int D>
constexpr int team_colb = D * 8 + 16;

// Columns of the increment ring for W compute waves: the last wave's 63 columns
// back, one chunk, and the waves' lags with half an edge ring of slack each.
__host__ __device__ constexpr int team_ring_cols(int sub, int W) {
    return (63 + kTeamX + (W - 1) * (64 + 2 * sub) + 2 * sub + kTeamX - 1) / kTeamX * kTeamX;
}

template <int P, int D>
__host__ __device__ constexpr size_t team_lds_bytes(int W) {
    const size_t edges = (size_t)(W + 1) * team_ec<P> * P * 8;
    const size_t coef = D > 0 ? (size_t)(team_ring_cols(team_sub<P>, W) + team_sub<P> + 1) *
                                    (D > 0 ? team_colb<D> : 0)
                              : (size_t)W * team_sub<P> * kWave * 8;
    return 256 + edges + coef;
}

// Workgroup-scope LDS counters.
__device__ __forceinline__ void lds_publish(int* f, int v) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (lane_id() == 0) __hip_atomic_store(f, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ int lds_peek(const int* f) {
    return __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// Whether a wait that began at t0 must be given up (watchdog, or raised by
// another wave).
__device__ __forceinline__ bool wait_expired(WsHeader* h, long long t0, long long ticks) {
    if (uniform((int)(load_status(h) & SIGK_ERR_WATCHDOG))) return true;
    if ((long long)__builtin_amdgcn_s_memrealtime() - t0 <= ticks) return false;
    raise_status(h, SIGK_ERR_WATCHDOG);
    return true;
}

struct TeamFlags {
    int done[8];
    int x, bot, out, ticket;
    int pad[4];
    float norm[kTeamQ];  // largest |dx|^2 over the columns a chunk's steps touch
};
static_assert(sizeof(TeamFlags) <= 256, "flag block");

// What a team's waves share about their strips.
struct TeamGeo {
    int W, nw;          // compute waves of the team, strips of this ticket
    int s0;             // first strip
    int rb;             // columns of the increment ring
    TeamFlags* f;
    char* edges;        // W + 1 edge rings
    char* coef;         // increment ring, or the coefficient rings (D = 0)
};

// ------------------------------------------------------------ service wave
template <int P, int D>
struct TeamService {
    static constexpr int SUB = team_sub<P>, EC = team_ec<P>, CB = D > 0 ? team_colb<D> : 1;
    const FwdArgs& a;
    const Geo& g;
    const TeamGeo& tg;

    // increments of columns [c0, c0 + 32), zero past the last one
    __device__ void load_x(int c0) {
        const int lane = lane_id();
        const int col = c0 + lane;
        float w = 0.0f;
        if (lane < kTeamX) {
            const bool in = col < g.m;
            const double* xp = g.x + (int64_t)min(col, g.m - 1) * a.d;
            const int slot = col % tg.rb;
            double* dst = (double*)(tg.coef + (size_t)slot * CB);
            double* dst2 = (double*)(tg.coef + (size_t)(slot + tg.rb) * CB);
            double n2 = 0.0;
#pragma unroll
            for (int ch0 = 0; ch0 < D; ch0 += 8) {
                double lo[8], hi[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const int cc = ch0 + k < a.d ? ch0 + k : 0;
                    lo[k] = xp[cc];
                    hi[k] = xp[a.d + cc];
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const double v = in && ch0 + k < a.d ? hi[k] - lo[k] : 0.0;
                    dst[ch0 + k] = v;
                    // the ring's first columns again behind its end, so that a
                    // block of steps reads them without a wrap
                    if (slot <= SUB) dst2[ch0 + k] = v;
                    n2 = fma(v, v, n2);
                }
            }
            // a float no smaller than n2 (as in the one-wave sweep)
            w = (float)fmax(n2 * (1.0 + 1e-6), n2 > 0.0 ? 1.2e-38 : 0.0);
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) w = fmaxf(w, __shfl_xor(w, o));
        // steps [c0, c0+32) touch columns [c0-63, c0+32): this chunk and the
        // two before it
        const float win = fmaxf(w, fmaxf(nprev, nprev2));
        nprev2 = nprev;
        nprev = w;
        if (lane == 0) tg.f->norm[(c0 / kTeamX) % kTeamQ] = win;
    }
    float nprev = 0.0f, nprev2 = 0.0f;

    // Runs until everything of this ticket is loaded and written out.
    __device__ bool run(const double* Fin, double* Fout, int* prog, bool below, bool above) {
        const int lane = lane_id();
        const int m = g.m;
        TeamFlags* f = tg.f;
        const int rows_last = min(kWave, g.n - (tg.s0 + tg.nw - 1) * kWave);
        // the last strip's steps, and the column read ahead of its last one
        // (earlier strips are full: no fewer columns)
        const int nx = D > 0 ? m + (tg.nw > 1 ? kWave : rows_last) : 0;
        double* ein = (double*)tg.edges;
        const double* eout = (const double*)(tg.edges + (size_t)tg.nw * EC * P * 8);
        int xc = 0, bc = below ? 0 : m, oc = above ? 0 : m;
        int avail = 0;
        long long idle0 = 0;
        int idle = 0;
        while (xc < nx || bc < m || oc < m) {
            bool moved = false;
            const int d0 = uniform(lds_peek(&f->done[0]));
            const int dl = uniform(lds_peek(&f->done[tg.nw - 1]));
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            if constexpr (D > 0) {
                if (xc < nx && xc + kTeamX - tg.rb <= dl - (kWave - 1)) {
                    load_x(xc);
                    xc += kTeamX;
                    lds_publish(&f->x, xc);
                    moved = true;
                }
            }
            if (bc < m) {
                if (avail < m && avail - bc < 2 * SUB)
                    avail = min(m, uniform(__hip_atomic_load(prog + tg.s0 - 1, __ATOMIC_RELAXED,
                                                             __HIP_MEMORY_SCOPE_AGENT)));
                int n = min(min(avail - bc, d0 + EC - bc), 2 * SUB);
                if (bc + n < m) n -= n % SUB;
                if (n > 0) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                    constexpr int NB = (2 * SUB * P + kWave - 1) / kWave;
                    const CoherentSpan src(Fin + (int64_t)bc * P, n * P);
                    double v[NB];
#pragma unroll
                    for (int k = 0; k < NB; ++k) v[k] = src.load(lane + k * kWave);
                    const int s0 = (bc % EC) * P;
#pragma unroll
                    for (int k = 0; k < NB; ++k) {
                        const int e = lane + k * kWave;
                        if (e < n * P) ein[(s0 + e) % (EC * P)] = v[k];
                    }
                    bc += n;
                    lds_publish(&f->bot, bc);
                    moved = true;
                }
            }
            if (oc < m) {
                int n = min(dl - (kWave - 1), m) - oc;
                if (oc + n < m && n < SUB) n = 0;
                if (n > 0) {
                    n = min(n, 2 * SUB);
                    double* dst = Fout + (int64_t)oc * P;
                    const int s0 = (oc % EC) * P;
                    for (int e = lane; e < n * P; e += kWave)
                        store_coherent(&dst[e], eout[(s0 + e) % (EC * P)]);
                    oc += n;
                    publish_coherent(prog + tg.s0 + tg.nw - 1, oc);
                    lds_publish(&f->out, oc);
                    moved = true;
                }
            }
            if (moved) {
                idle = 0;
            } else {
                if (idle == 0) idle0 = (long long)__builtin_amdgcn_s_memrealtime();
                __builtin_amdgcn_s_sleep(1);
                if ((++idle & 63) == 0 && wait_expired(a.hdr, idle0, a.watchdog_ticks))
                    return false;
            }
        }
        return true;
    }
};

// ------------------------------------------------------------ compute waves
template <int P, int D>
struct TeamWave {
    static constexpr int SUB = team_sub<P>, EC = team_ec<P>, CB = D > 0 ? team_colb<D> : 1;
    // the next step's coefficient is formed a step ahead where registers allow
    static constexpr bool kAhead = D > 0 && (P <= 8 || (P <= 12 && D <= 8));
    static constexpr int kUnroll = P <= 6 ? 4 : P <= 12 ? 2 : 1;
    const FwdArgs& a;
    const Geo& g;
    const TeamGeo& tg;
    Acc& acc;
    int s, w, nrows;
    bool has_below, has_above;
    const double* Ein;   // edge ring of the strip's bottom edges
    double* Eout;        // edge ring its top lane writes
    double B[P], Ac[P];
    double dy[D > 0 ? D : 1];
    double kpad;         // K at the end of the strip's bottom row
    bool padded;
    double cn;
    double dymax2;
    double tau;          // tau2[lane] (lanes 1..P-1; infinite elsewhere)
    double tacc, etot;   // as in StripCtx; etot per lane
    int kexp, q;
    Recip<P> R;

    __device__ TeamWave(const FwdArgs& a_, const Geo& g_, const TeamGeo& t_, Acc& acc_)
        : a(a_), g(g_), tg(t_), acc(acc_) {}

    __device__ __forceinline__ void tally(double c, const double (&E)[P]) {
        tacc = fma(fabs(c), fabs(E[P - 1]), tacc);
    }
    __device__ __forceinline__ void fold() {
        const double k1 = fabs(B[0]);
        const int e1 = k1 >= 1.0 && k1 <= 1.7e308 ? ilogb(k1) : 0;  // 0 also for NaN
        etot += ldexp(tacc, -min(kexp, e1));
        kexp = e1;
        tacc = 0.0;
    }
    // counters for steps [t0, t1) at depth qd
    __device__ void count(int t0, int t1, int qd) {
        const long long cnt = cells_before(t1, g.m, nrows) - cells_before(t0, g.m, nrows);
        acc.cells += (unsigned long long)cnt;
        acc.flops += (unsigned long long)(cnt * cell_flops(P, qd, D > 0 ? a.d : 0));
    }
    // depth of the cells with |c|^2 <= cmax2: lane n compares term n
    __device__ __forceinline__ void set_depth(double cmax2) {
        const uint64_t need = ballot(cmax2 > tau);
        q = need ? 63 - __builtin_clzll(need) : 0;
    }

    // Bottom edges of steps [t, te) past the last column: the constant K at the
    // row's end (as StripCtx::pad_bottom); the strip below writes no more then.
    __device__ void pad_bottom(int t, int te) {
        const int m = g.m;
        if (!padded) {
            const double* r = Ein + ((m - 1) & (EC - 1)) * P;
            double k = r[P - 1];
#pragma unroll
            for (int i = P - 2; i >= 0; --i) k = fma(k, R(i + 1), r[i]);
            kpad = uniform_d(k);
            padded = true;
        }
        for (int e = lane_id(); e < SUB * P; e += kWave) {
            const int col = t + e / P;
            if (col >= m && col < te) ((double*)Ein)[(col & (EC - 1)) * P + e % P] =
                e % P == 0 ? kpad : 0.0;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    }

    __device__ __forceinline__ double dot(const char* xp) const {
        double c0 = 0.0, c1 = 0.0;
#pragma unroll
        for (int ch = 0; ch < D; ch += 2) {
            const double2 v = *(const double2*)(xp + ch * 8);
            c0 = fma(dy[ch], v.x, c0);
            c1 = fma(dy[ch + 1], v.y, c1);
        }
        return c0 + c1;
    }

    // Step t.  xp: the column's increments (of step t + 1 where kAhead);
    // D = 0: the step's coefficient.
    template <int QC>
    __device__ __forceinline__ void step(int t, const char* xp) {
        const int lane = lane_id();
        const double* bsrc = Ein + (t & (EC - 1)) * P;
        double A[P], An[P], Bn[P];
        double c;
        if constexpr (P <= 12) {
            double bv[P];
            lds_copy<P>(bv, bsrc);
            double2 dxv[kAhead ? D / 2 : 1];
            if constexpr (kAhead) {
                c = cn;
#pragma unroll
                for (int k = 0; k < D / 2; ++k) dxv[k] = *(const double2*)(xp + k * 16);
            } else if constexpr (D > 0) {
                c = dot(xp);
            } else {
                c = *(const double*)xp;
            }
            SplitMap<P, QC> S;
            S.pre(B, c, Bn, R);
            tally(c, B);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < P; ++i) A[i] = shift_up(Ac[i], bv[i]);
            S.post(A, An, Bn, R);
            tally(c, A);
            if constexpr (kAhead) {
                __builtin_amdgcn_sched_barrier(0);
                double c0 = 0.0, c1 = 0.0;
#pragma unroll
                for (int k = 0; k < D / 2; ++k) {
                    c0 = fma(dy[2 * k], dxv[k].x, c0);
                    c1 = fma(dy[2 * k + 1], dxv[k].y, c1);
                }
                cn = c0 + c1;
            }
        } else {
#pragma unroll
            for (int i = 0; i < P; ++i) A[i] = shift_up(Ac[i], bsrc[i]);
            if constexpr (D > 0)
                c = dot(xp);
            else
                c = *(const double*)xp;
            tally(c, A);
            tally(c, B);
            cell_map<P>(A, B, c, An, Bn, QC, R);
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {
            B[i] = Bn[i];
            Ac[i] = An[i];
        }
        // (columns before the first land in slots that are written again
        // before they are read)
        if (has_above && lane == kWave - 1)
            lds_copy<P>(Eout + ((t + 1) & (EC - 1)) * P, Ac);  // column t - 63
    }

    template <int QD>
    __device__ __forceinline__ void run_depth(int t, int te, const char* xp) {
        if constexpr (QD < P - 1) {
            if (q > QD) {
                run_depth<QD + 1>(t, te, xp);
                return;
            }
        }
#pragma unroll kUnroll
        for (; t < te; ++t) {
            step<QD>(t, xp);
            xp += D > 0 ? CB : kWave * 8;
        }
    }

    __device__ bool sweep(double* out_est) {
        const int lane = lane_id();
        const int m = g.m;
        TeamFlags* f = tg.f;
        const int row0 = s * kWave;
        nrows = uniform(min(kWave, g.n - row0));
        const bool lane_ok = lane < nrows;
        R.init();
        const int l = row0 + lane;
        double n2 = 0.0;
        if constexpr (D > 0) {
#pragma unroll
            for (int ch = 0; ch < D; ++ch) {
                dy[ch] = (ch < a.d && lane_ok)
                             ? g.y[(int64_t)(l + 1) * a.d + ch] - g.y[(int64_t)l * a.d + ch]
                             : 0.0;
                n2 = fma(dy[ch], dy[ch], n2);
            }
            dymax2 = wave_max(n2);
        }
        tau = lane >= 1 && lane < P ? a.tau2[lane < kMaxP ? lane : 0] : __builtin_inf();
        q = P - 1;
        tacc = 0.0;
        etot = 0.0;
        kexp = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            B[i] = i == 0 ? 1.0 : 0.0;
            Ac[i] = B[i];
        }
        const int T = m + nrows - 1;
        // counters this wave waits on, one lane each: 0 the strip below, 1 the
        // increments (first wave), 2 the strip above
        const int* fl = lane == 0 ? (w > 0 ? &f->done[w - 1] : &f->bot)
                        : lane == 1 ? &f->x
                                    : (w + 1 < tg.nw ? &f->done[w + 1] : &f->out);
        int add = INT32_MIN / 2, cap = INT32_MIN / 2;
        if (lane == 0 && has_below) {
            add = SUB + (w > 0 ? kWave - 1 : 0);
            cap = m + (w > 0 ? kWave - 1 : 0);
        } else if (lane == 1 && w == 0 && D > 0) {
            add = SUB + 1;
            cap = T + 1;
        } else if (lane == 2 && has_above) {
            // (the service wave counts columns, a compute wave steps: its
            // bottom edges are read up to its step)
            add = SUB - (kWave - 1) - EC;
            cap = INT32_MAX;
        }
        char* cring = nullptr;
        double cbuf[D > 0 ? 1 : SUB];
        const double* csrc = nullptr;
        if constexpr (D == 0) {
            cring = tg.coef + (size_t)w * SUB * kWave * 8;
            csrc = a.delta + g.delta + (int64_t)s * delta_steps(m) * kWave + lane;
#pragma unroll
            for (int k = 0; k < SUB; ++k) cbuf[k] = csrc[(int64_t)k * kWave];
        }
        padded = false;
        kpad = 0.0;
        // slot of the block's first column (the one read ahead where kAhead)
        int slot = ((kAhead ? 1 : 0) - lane + tg.rb) % tg.rb;
        int trun = 0, qrun = q;  // steps since trun ran at depth qrun
        for (int t = 0; t < T;) {
            const int te = min(T, t + SUB);
            {
                const int need = min(t + add, cap);
                long long t0 = 0;
                for (int spin = 0;; ++spin) {
                    const int v = lds_peek(fl);
                    if (ballot(v < need) == 0) break;
                    __builtin_amdgcn_s_sleep(1);
                    if ((spin & 255) == 0) {
                        if (spin == 0) t0 = (long long)__builtin_amdgcn_s_memrealtime();
                        else if (wait_expired(a.hdr, t0, a.watchdog_ticks)) return false;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
            }
            if (te > m && has_below) pad_bottom(t, te);
            const char* xp = nullptr;
            if constexpr (D > 0) {
                if ((t % kTeamX) == 0) {
                    fold();
                    // (past the last column the depth stays)
                    if (t < m) set_depth((double)f->norm[(t / kTeamX) % kTeamQ] * dymax2);
                }
                if (kAhead && t == 0) cn = dot(tg.coef + (size_t)((tg.rb - lane) % tg.rb) * CB);
                xp = tg.coef + (size_t)slot * CB;
                slot += SUB;
                slot -= slot >= tg.rb ? tg.rb : 0;
            } else {
                fold();
                double cm = 0.0;
                char* dst = cring + lane * 8;
#pragma unroll
                for (int k = 0; k < SUB; ++k) {
                    const int col = t + k - lane;
                    const double c = (lane_ok && col >= 0 && col < m) ? cbuf[k] : 0.0;
                    *(double*)(dst + (size_t)k * kWave * 8) = c;
                    cm = fmax(cm, fabs(c));
                }
                const double cmax = wave_max_nn(cm);
                set_depth(cmax * cmax);
                xp = dst;
                if (te < T) {
                    // the next block's coefficients, in flight over this one
#pragma unroll
                    for (int k = 0; k < SUB; ++k)
                        cbuf[k] = csrc[(int64_t)min(te + k, T - 1) * kWave];
                }
            }
            if (q != qrun) {
                count(trun, t, qrun);
                trun = t;
                qrun = q;
            }
            run_depth<0>(t, te, xp);
            t = te;
            lds_publish(&f->done[w], t);
        }
        count(trun, T, qrun);
        fold();
        *out_est = wave_sum(etot) * inv_factorial<P>();
        return true;
    }
};

// Waves per SIMD the team kernel is compiled for, and the most compute waves of
// a team: one per SIMD (the chain runs at a lone wave's issue rate; a fifth
// compute wave shares a SIMD and slowed a 4096-point pair at order 6 from 3.04
// to 4.42 ms), the service wave beside one of them; three where the kernel
// takes a SIMD's whole register file.
template <int P, int D>
constexpr int team_eu = P <= 6 && D <= 8 ? 3 : (P <= 10 && D <= 16 ? 2 : 1);
template <int P, int D>
constexpr int team_max_waves = team_eu<P, D> > 1 ? 4 : 3;

template <int P, int D>
__global__ void __launch_bounds__(kWave*(team_max_waves<P, D> + 1))
    __attribute__((amdgpu_waves_per_eu(team_eu<P, D>))) team_kernel(FwdArgs a) {
    extern __shared__ double team_smem[];
    char* smem = (char*)team_smem;
    const int lane = lane_id();
    const int w = uniform((int)(threadIdx.x >> 6));
    TeamGeo tg;
    tg.W = a.team;
    tg.f = (TeamFlags*)smem;
    tg.edges = smem + 256;
    tg.coef = tg.edges + (size_t)(tg.W + 1) * team_ec<P> * P * 8;
    tg.rb = team_ring_cols(team_sub<P>, tg.W);
    Acc acc;
    for (;;) {
        __syncthreads();  // every wave is done with the previous ticket
        if (threadIdx.x == 0) {
            int t = (int)atomicAdd(&a.hdr->ticket, 1u);
            if ((int64_t)t >= a.ntickets || (load_status(a.hdr) & SIGK_ERR_WATCHDOG)) t = -1;
            tg.f->ticket = t;
        }
        if (threadIdx.x < 8) tg.f->done[threadIdx.x] = 0;
        if (threadIdx.x == 8) tg.f->x = 0;
        if (threadIdx.x == 9) tg.f->bot = 0;
        if (threadIdx.x == 10) tg.f->out = 0;
        __syncthreads();
        const int t = uniform(tg.f->ticket);
        if (t < 0) break;
        const int pair = (int)((int64_t)t % a.npairs);
        const Geo g = resolve(a, pair, P, 0);
        tg.s0 = (int)((int64_t)t / a.npairs) * tg.W;
        tg.nw = min(tg.W, a.strips - tg.s0);
        const bool below = tg.s0 > 0, above = tg.s0 + tg.nw < a.strips;
        constexpr int EB = team_ec<P> * P * 8;
        if constexpr (D > 0) {
            // zero increments in the 64 columns before the first
            for (int e = (int)threadIdx.x; e < kWave * team_colb<D> / 8; e += (int)blockDim.x)
                ((double*)(tg.coef + (size_t)(tg.rb - kWave) * team_colb<D>))[e] = 0.0;
        }
        if (!below) {
            // bottom row of the grid: K = 1 on the axis
            for (int e = (int)threadIdx.x; e < EB / 8; e += (int)blockDim.x)
                ((double*)tg.edges)[e] = (e % P) == 0 ? 1.0 : 0.0;
        }
        __syncthreads();
        if (w == tg.W) {
            TeamService<P, D> S{a, g, tg};
            S.run(a.frontier + g.front, a.frontier + g.front, a.progress + g.prog, below, above);
        } else if (w < tg.nw) {
            TeamWave<P, D> S(a, g, tg, acc);
            S.s = tg.s0 + w;
            S.w = w;
            S.has_below = w > 0 || below;
            S.has_above = w + 1 < tg.nw || above;
            S.Ein = (const double*)(tg.edges + (size_t)w * EB);
            S.Eout = (double*)(tg.edges + (size_t)(w + 1) * EB);
            double est = 0.0;
            if (S.sweep(&est)) {
                if (!isfinite(est)) acc.status |= SIGK_WARN_NONFINITE;
                if (lane == 0 && a.trunc_est) atomicAdd(&a.trunc_est[pair], est);
                if (!S.has_above) {
                    // the last row's lane holds the top edge of the corner cell
                    const bool mine = lane == S.nrows - 1;
                    double k = 0.0, fct = 1.0;
#pragma unroll
                    for (int i = 0; i < P; ++i) {
                        k = fma(S.Ac[i], fct, k);
                        fct = fct / (double)(i + 1);
                    }
                    if (ballot(mine && !isfinite(k))) acc.status |= SIGK_WARN_NONFINITE;
                    if (mine && a.out) {
                        a.out[g.o1] = k;
                        if (g.o2 >= 0) a.out[g.o2] = k;
                    }
                }
            }
        }
    }
    finish_forward(a, acc, w == 0);
}

}  // namespace sigk
