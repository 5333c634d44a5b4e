// sigk_bwd.hip -- gradient of kernel values with respect to the paths.
//
// Persistent kernels per (P, D) variant:
//   ckpt_kernel: the forward sweep of every strip, keeping (a) the frontier row
//                each strip reads (one snapshot per strip instead of the single
//                in-place row), (b) the wave state (left edges and in-flight top
//                edges of all 64 lanes) every kCkptEvery steps and (c) the
//                Neumann depth of every chunk.
//   bwd_kernel:  the adjoint sweep, strips in reverse topological order (top
//                strip of each pair first).  Per segment of kCkptEvery steps,
//                taken last to first: restore the wave state, recompute the
//                segment forward while storing each step's bottom-edge inputs
//                in a per-workgroup scratch, then run the adjoint cell map over
//                the segment in reverse step order, recovering each cell's left
//                edge from its right edge (the left-edge update is
//                triangular).  dL/dc of every cell is chained into
//                dL/d(increment) of both paths: the x side through an LDS ring
//                indexed by column (each column is complete once lane 0 has
//                passed it), the y side in registers of the row's lane.
//   bwd_two_kernel: the adjoint sweep with a second wave per strip for the
//                recompute, for launches of few strips.
// All also run the blocks of a long pair (block checkpointing, see BlockGeo):
// a block is a small pair whose bottom and left edges come from lines kept by
// a first sweep and whose top and right edge cotangents come from the blocks
// processed before it.
#include "sigk_adjoint.h"
#include "sigk_stop.h"

#ifndef SIGK_P
#define SIGK_P 8
#endif
#ifndef SIGK_D
#define SIGK_D 8
#endif

namespace sigk {

// Frontier chunk of the checkpointing forward sweep (which also sets the
// granularity of the Neumann depths the adjoint reads back): 64 columns at orders
// 10-20 with D <= 16, as in the plain forward sweep (this one runs a wave per SIMD
// there); 32 elsewhere.
template <int P, int D>
constexpr int ckpt_chunk = (P >= 10 && P <= 20 && D <= 16) ? 64 : 32;

template <int P, int D>
constexpr int ckpt_ring = ckpt_chunk<P, D> == 64 ? chunk64_ring(P, D) : ring_cols(P);
// Columns per Neumann depth it records.
template <int P, int D>
constexpr int ckpt_depth_cols = inc_chunk<ckpt_chunk<P, D>, ckpt_ring<P, D>>;

// Modes: kModeTable, the checkpointing sweep of a batch (snap: per-strip
// frontier rows); kModeBlock, the checkpointing sweep of the blocks of one
// anti-diagonal (snap: per-slot frontier rows; strip 0 reads its bottom line,
// column 0 its left line).
// (three waves per SIMD at orders 4-5 with d <= 8: 168 registers, 7% faster
// at order 5; at order 6 that limit would spill)
template <int P, int D>
__global__ void __launch_bounds__(kWave)
    __attribute__((amdgpu_waves_per_eu(P <= 5 && D <= 8 ? 3 : 1))) ckpt_kernel(FwdArgs a,
                                                                              double* snap) {
    constexpr int CH = ckpt_chunk<P, D>, RB = ckpt_ring<P, D>;
    __shared__ LdsStrip<P, D, CH, RB> L;
    Acc acc;
    const int lane = lane_id();
    for (;;) {
        unsigned t = 0;
        if (lane == 0) t = atomicAdd(&a.hdr->ticket, 1u);
        t = (unsigned)uniform((int)t);
        if ((int64_t)t >= a.ntickets) break;
        if (uniform((int)(load_status(a.hdr) & SIGK_ERR_WATCHDOG))) break;
        int pair, strip;
        Geo g;
        BlockRef r;
        r.bot = nullptr;
        r.left = nullptr;
        if (a.mode == kModeTable) {
            pair = a.tickets[t].pair;
            strip = a.tickets[t].strip;
            if (pair < 0) break;  // unused slots close a table built on the device
            g = resolve(a, pair, P, 0);
            g.front = a.desc[pair].snap_off;
        } else {
            pair = (int)(t % (unsigned)a.blk.nb);
            strip = (int)(t / (unsigned)a.blk.nb);
            g = resolve_block(a, pair, P, r);
            if (strip * kWave >= g.n) continue;  // the top block row has fewer strips
        }
        StripCtx<P, D, CH, RB, false, true> S(a, g, L, acc, strip);
        S.pair = pair;
        S.prog = a.progress + g.prog;
        const int64_t row = (int64_t)g.m * P;
        S.Fin = (strip == 0 && r.bot) ? r.bot : snap + g.front + (int64_t)strip * row;
        S.Fout = snap + g.front + (int64_t)(strip + 1) * row;
        double* ck = a.ckpt + g.ckpt + (int64_t)strip * ckpt_strip_doubles(g.m, P);
        S.ck = ck;
        S.ckq = ck + ckpt_states(g.m) * 2 * P * kWave;
        S.ck_every = kCkptEvery;
        S.left = r.left;
        S.below_line = r.bot != nullptr;
        if (!S.sweep()) break;
    }
    if (lane == 0) {
        atomicAdd(&a.hdr->cells, acc.cells);
        atomicAdd(&a.hdr->flops, acc.flops);
        if (acc.status) atomicOr(&a.hdr->status, acc.status);
    }
}

// The first sweep of a long pair's gradient (kModeLines): the plain forward
// sweep of the whole pair, with the plain forward kernel's chunks and
// occupancy, writing k(x, y) and keeping the block-boundary lines: a strip
// that ends a block row writes its top edges to that row's line instead of
// the in-place frontier row (the next strip reads them there), and every
// lane stores its right edge at the last column of each block column.
template <int P, int D>
__global__ void __launch_bounds__(kWave)
    __attribute__((amdgpu_waves_per_eu(P <= 6 && D <= 8 ? 3 : 1))) lines_kernel(FwdArgs a) {
    constexpr int CH = fwd_chunk_cols(P, D), RB = fwd_ring_cols(P, D);
    __shared__ LdsStrip<P, D, CH, RB> L;
    Acc acc;
    const int lane = lane_id();
    for (;;) {
        unsigned t = 0;
        if (lane == 0) t = atomicAdd(&a.hdr->ticket, 1u);
        t = (unsigned)uniform((int)t);
        if ((int64_t)t >= a.ntickets) break;
        if (uniform((int)(load_status(a.hdr) & SIGK_ERR_WATCHDOG))) break;
        const int strip = (int)t;
        Geo g = resolve_lines(a);
        StripCtx<P, D, CH, RB, false, true> S(a, g, L, acc, strip);
        S.pair = 0;
        S.prog = a.progress;
        const int64_t row = (int64_t)g.m * P;
        const int kb = a.blk.kb;
        S.Fin = (strip > 0 && strip % kb == 0) ? a.blk.hline + (int64_t)(strip / kb - 1) * row
                                               : a.frontier;
        S.Fout = ((strip + 1) % kb == 0 && (int64_t)(strip + 1) * kWave < g.n)
                     ? a.blk.hline + (int64_t)((strip + 1) / kb - 1) * row
                     : a.frontier;
        S.ck = nullptr;
        S.ckq = nullptr;
        S.ck_every = 1;
        S.vl = a.blk.nj > 1 ? a.blk.vline : nullptr;
        if (!S.sweep()) break;
    }
    if (lane == 0) {
        atomicAdd(&a.hdr->cells, acc.cells);
        atomicAdd(&a.hdr->flops, acc.flops);
        if (acc.status) atomicOr(&a.hdr->status, acc.status);
    }
}

// Orders a wave's LDS accesses (its lanes exchange data through LDS); the
// adjoint's waves never need the workgroup barrier for that.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

// A workgroup's segment scratch as a buffer resource: rows of 64 doubles,
// one per lane.  The lane's column goes in the vector offset and the row
// (step and coefficient) in the scalar offset, so stepping through the rows
// costs no vector instructions.  Every access is range-checked against the
// buffer's size by the hardware.
struct SegScratch {
    using u32x2 = unsigned int __attribute__((__vector_size__(8)));
    __amdgpu_buffer_rsrc_t r;
    __device__ void init(double* p, int rows) {
        const uint64_t a = (uint64_t)p;
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
        r = __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0,
                                              rows * kWave * 8, 0x00020000);
    }
    __device__ __forceinline__ void store(int row, double v) const {
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, lane_id() * 8,
                                              row * (kWave * 8), 0);
    }
    __device__ __forceinline__ double load(int row) const {
        return __builtin_bit_cast(
            double, __builtin_amdgcn_raw_buffer_load_b64(r, lane_id() * 8, row * (kWave * 8), 0));
    }
};

template <int P, int D>
struct LdsBwd {
    // Columns per cotangent-frontier chunk and of the increment rings.  At
    // orders 10-12 with D = 8 the adjoint exchanges 64-column chunks (a
    // 128-column ring; the buffers then fill LDS exactly at four waves per
    // CU, the register-bound occupancy): 2% faster on the MMD^2 workload.
    // Per-chunk Neumann depths are still read at the checkpointing sweep's
    // chunk width (depth_at).
    static constexpr int ACH = (P >= 10 && P <= 12 && D <= 8) ? 64 : 32;
    // (96 columns hold a 32-column chunk and the 63 before it; at orders 4-5
    // with d <= 8 the smaller rings let an eighth wave per CU fit its LDS:
    // 4.5% faster there than with 128)
    static constexpr int ARB = ACH == 64 ? 128 : 96;
    static_assert(ARB >= ACH + kWave - 1,
                  "the rings must hold a chunk and the 63 columns before it");
    // (the edge rows first: one address register with the instructions'
    // immediate offsets reaches a whole row)
    double bin[ACH * P];    // primal bottom edges (lane 0) of a chunk
    double lin[2 * ACH * P];  // top-edge cotangents (top lane), 2 chunks
    double lout[ACH * P];   // bottom-edge cotangents (lane 0), 1 chunk
    // increments of x and dL/d(dx) being accumulated, by ring slot,
    // interleaved per channel: [channel][dx, gx][slot].  A channel's rows lie
    // 2 ARB doubles apart, a multiple of 512 bytes, so one address register
    // and offsets in 512-byte units reach every channel's slot.
    double xg[D * 2 * ARB];
    static_assert((2 * ARB * 8) % 512 == 0 && (ACH * P * 4 * 8) % 512 == 0,
                  "channel rows on 512-byte boundaries");
    __device__ __forceinline__ double& dx(int ch, int slot) { return xg[2 * ch * ARB + slot]; }
    __device__ __forceinline__ double& gx(int ch, int slot) {
        return xg[(2 * ch + 1) * ARB + slot];
    }
    // the same by a RingPos byte offset
    __device__ __forceinline__ double& dx_at(int ch, const RingPos<ARB>& p) {
        return *(double*)((char*)&xg[2 * ch * ARB] + p.b);
    }
    __device__ __forceinline__ double& gx_at(int ch, const RingPos<ARB>& p) {
        return *(double*)((char*)&xg[(2 * ch + 1) * ARB] + p.b);
    }
};

template <int P, int D>
struct StripBwd {
    static constexpr int ACH = LdsBwd<P, D>::ACH;
    static constexpr int ARB = LdsBwd<P, D>::ARB;
    const BwdArgs& b;
    const FwdArgs& a;
    Geo& g;
    LdsBwd<P, D>& L;
    int s, nrows, m;
    bool lane_ok, has_below, has_above;
    double dy[D];
    double gy[D];
    Recip<P> R;  // scalar or rematerialised constants: registers are scarce here
    int dx_lo, lin_lo, bin_chunk;
    // kCkptEvery x P recomputed bottom-edge rows, then as many left-edge rows (a
    // smooth segment of the two-wave kernel: P rows of right edges after it);
    // two such buffers for the two-wave kernel
    SegScratch scr;
    unsigned long long* cells;  // per-workgroup tallies (cells, algorithmic flops)
    unsigned long long* flops;
    const double* ck;
    const double* ckq;
    const double* snap_in;   // primal frontier row read by lane 0 ([m][P])
    double* lam_row;         // adjoint frontier row of the pair ([m][P])
    int* lam_prog;           // adjoint progress of the pair's strips
    double seed_scale;       // grad_out of the pair (0: no seed in this grid)
    double* gxp;             // dL/d(dx) of the pair's columns ([m][d])
    double* gyp;             // dL/d(dy) of the pair's rows ([n][d])
    // block checkpointing (null / false for whole pairs): primal left edges at
    // column 0, a primal bottom line for strip 0 and a cotangent row from a
    // block above; the right-edge cotangents of the rows (read at the last
    // column when a block to the right exists, written at column 0 when one
    // to the left does)
    const double* left = nullptr;
    bool below_line = false;
    bool above_blk = false;
    double* lamv = nullptr;
    bool right_in = false;
    bool left_out = false;

    __device__ StripBwd(const BwdArgs& b_, Geo& g_, LdsBwd<P, D>& L_, int s_)
        : b(b_), a(b_.f), g(g_), L(L_), s(s_) {}

    // Increments of x in steps of kCkptEvery columns, descending, so that the
    // ring holds [t0-63, t0+kCkptEvery) for segment t0 (the recomputing wave of
    // the two-wave kernel works one segment lower: 96 columns in all), zero
    // outside the grid's columns: there the maps run with c = 0, which keeps
    // every right edge and every zero cotangent, and need no per-lane test.
    __device__ void load_dx_down_to(int lo_needed) {
        const int lane = lane_id();
        while (dx_lo > lo_needed) {
            const int c0 = dx_lo - kCkptEvery;
            const int col = c0 + lane;
            if (col < dx_lo && col < m) {
                const double* xp = g.x + (int64_t)max(col, 0) * a.d;
#pragma unroll
                for (int ch = 0; ch < D; ++ch)
                    L.dx(ch, ring_slot_of<ARB>(col)) =
                        ch < a.d && col >= 0 ? xp[a.d + ch] - xp[ch] : 0.0;
            }
            dx_lo = c0;
            wave_sync();
        }
    }

    __device__ bool load_lin_down_to(int lo_needed) {
        const int CH = ACH;
        const int lane = lane_id();
        while (lin_lo > lo_needed && lin_lo > 0) {
            const int c0 = lin_lo - CH;
            const int nc = min(CH, m - c0);
            if (!wait_flag(&lam_prog[s + 1], m - c0, a.hdr, a.watchdog_ticks)) return false;
            double* dst = &L.lin[((c0 / CH) & 1) * CH * P];
            constexpr int NB = (ACH * P + kWave - 1) / kWave;
            const CoherentSpan src(lam_row + (int64_t)c0 * P, nc * P);
            double v[NB];
#pragma unroll
            for (int k = 0; k < NB; ++k) v[k] = src.load(lane + k * kWave);
#pragma unroll
            for (int k = 0; k < NB; ++k)
                if (lane + k * kWave < nc * P) dst[lane + k * kWave] = v[k];
            lin_lo = c0;
            wave_sync();
        }
        return true;
    }

    // (steps past the last column read the last chunk's rows: any finite values)
    __device__ void load_bin(int chunk) {
        if (chunk == bin_chunk) return;
        const int CH = ACH;
        const int lane = lane_id();
        const int c0 = chunk * CH;
        const int nc = min(CH, m - c0);
        if (has_below) {
            const double* src = snap_in + (int64_t)c0 * P;
            // (0 past the last column: read by lanes past the end of their row)
            for (int e = lane; e < CH * P; e += kWave) L.bin[e] = e < nc * P ? src[e] : 0.0;
        } else {
            for (int e = lane; e < CH * P; e += kWave) L.bin[e] = (e % P) == 0 ? 1.0 : 0.0;
        }
        bin_chunk = chunk;
        wave_sync();
    }

    // columns [c0, c1) are final: publish the bottom-edge cotangents to the
    // strip below and add dL/d(dx) to the path's gradient scratch
    __device__ void flush_cols(int c0, int c1) {
        const int lane = lane_id();
        wave_sync();
        const int nc = c1 - c0;
        if (has_below) {
            double* dst = lam_row + (int64_t)c0 * P;
            for (int e = lane; e < nc * P; e += kWave) store_coherent(&dst[e], L.lout[e]);
            publish_coherent(&lam_prog[s], m - c0);
        }
        if (lane < nc) {
            const int col = c0 + lane;
            const int sl = ring_slot_of<ARB>(col);
            double* gp = gxp + (int64_t)col * a.d;
#pragma unroll
            for (int ch = 0; ch < D; ++ch) {
                if (ch < a.d) atomicAdd(&gp[ch], L.gx(ch, sl));
                L.gx(ch, sl) = 0.0;
            }
        }
        wave_sync();
    }

    // depth record of the chunk of step t: depth + kRoughFlag if rough
    __device__ __forceinline__ int depth_at(int t) const {
        const int k = min(t, m - 1) / ckpt_depth_cols<P, D>;
        return uniform((int)ckq[k]);
    }

    double lAprev[P];  // bottom-edge cotangents of the previous (later) step
    double lBst[P];    // left-edge cotangent carried along the row
    int topl;          // lane whose top-edge cotangent comes from outside the wave

    // Depth dispatch: one specialised segment loop per Neumann depth.  what:
    // 1 recompute, 2 adjoint, 3 both (buf: the scratch buffer's first row).
    template <int Q, int what>
    __device__ __forceinline__ void segment_at_depth(int q, bool rough, int t0, int t1, int buf) {
        if constexpr (Q >= 0 && Q < P - 1) {
            if (q > Q) {
                segment_at_depth<Q + 1, what>(q, rough, t0, t1, buf);
                return;
            }
        }
        if constexpr (what == 1) {
            double B[P];
            recompute<Q, true>(q, rough, t0, t1, buf, B);
        } else if constexpr (P == 12 && D == 32) {
            // (one copy of the recompute for both kinds of segment: here the
            // compiler keeps the loops' arrays in memory otherwise, 4 times
            // slower; elsewhere two copies are up to 4% faster)
            double B[P];
            if constexpr (what == 3) recompute<Q, false>(q, rough, t0, t1, buf, B);
            if (t0 >= kWave && t1 <= m - 1)
                adjoint<Q, true, what == 2>(q, rough, t0, t1, buf, B);
            else
                adjoint<Q, false, what == 2>(q, rough, t0, t1, buf, B);
        } else if (P <= 12 && t0 >= kWave && t1 <= m - 1) {
            half_or_both<Q, P <= 12, what>(q, rough, t0, t1, buf);
        } else {
            half_or_both<Q, false, what>(q, rough, t0, t1, buf);
        }
    }
    template <int Q, bool IN, int what>
    __device__ __forceinline__ void half_or_both(int q, bool rough, int t0, int t1, int buf) {
        double B[P];
        if constexpr (what == 3) recompute<Q, false>(q, rough, t0, t1, buf, B);
        adjoint<Q, IN, what == 2>(q, rough, t0, t1, buf, B);
    }

    // One segment [t0, t1) of kCkptEvery steps, recomputed forward from its
    // checkpoint, each step's bottom edges stored.  Q >= 0: depth fixed at
    // compile time (== q); Q < 0: q.  rough: the left edges are stored too
    // (second half of the buffer).  On return B holds the right edges after
    // the segment (HAND: left in the buffer for another wave).
    template <int Q, bool HAND>
    __device__ void recompute(int q, bool rough, int t0, int t1, int buf, double (&B)[P]) {
        const int lane = lane_id();
        const int CH = ACH;
        const int W = kCkptEvery;
        double Ac[P];
        {
            const double* src = ck + (int64_t)(t0 / W) * (2 * P * kWave);
#pragma unroll
            for (int i = 0; i < P; ++i) {
                B[i] = src[i * kWave + lane];
                Ac[i] = src[(P + i) * kWave + lane];
            }
        }
        RingPos<ARB> rp;
        rp.set(t0 - lane);
        for (int t = t0; t < t1; ++t) {
            double c0 = 0.0, c1 = 0.0;
#pragma unroll
            for (int ch = 0; ch < D; ch += 2) {
                c0 = fma(dy[ch], L.dx_at(ch, rp), c0);
                c1 = fma(dy[ch + 1], L.dx_at(ch + 1, rp), c1);
            }
            rp.next();
            const double c = c0 + c1;
            const int row0 = buf + (t - t0) * P;
            if (rough) {
#pragma unroll
                for (int i = 0; i < P; ++i) scr.store(kCkptEvery * P + row0 + i, B[i]);
            }
            double A[P], An[P], Bn[P];
            const double* bsrc = &L.bin[(t % CH) * P];
            if constexpr (Q >= 0 && P <= 12) {
                // the map in two halves, as in the forward sweep (the same
                // sums in the same order): the B-only half covers the latency
                // of the lane shift that delivers A
                SplitMap<P, Q, false> S;
                S.pre(B, c, Bn, R);
#pragma unroll
                for (int i = 0; i < P; ++i) A[i] = shift_up(Ac[i], bsrc[i]);
#pragma unroll
                for (int i = 0; i < P; ++i) scr.store(row0 + i, A[i]);
                S.post(A, An, Bn, R);
            } else {
#pragma unroll
                for (int i = 0; i < P; ++i) A[i] = shift_up(Ac[i], bsrc[i]);
#pragma unroll
                for (int i = 0; i < P; ++i) scr.store(row0 + i, A[i]);
                cell_map<P>(A, B, c, An, Bn, Q >= 0 ? Q : q, R);
            }
            // (past the end of the row c = 0: B keeps the row's last right edge)
#pragma unroll
            for (int i = 0; i < P; ++i) {
                B[i] = Bn[i];
                Ac[i] = An[i];
            }
        }
        if (HAND && !rough) {
#pragma unroll
            for (int i = 0; i < P; ++i) scr.store(buf + kCkptEvery * P + i, B[i]);
        }
    }

    // The adjoint over the segment, last step first; B walks back from the
    // right edges after the segment to each cell's left edge (rough: the left
    // edges are read back).  IN: every cell of the segment is inside the
    // strip's columns and none is in its first or last column (t0 >= 64,
    // t1 <= m - 1), so the per-lane tests for the row ends, the corner seed and
    // the block lines drop out.  HAND: recomputed by another wave, so the right
    // edges come from the buffer; each step's bottom edges are then loaded a
    // step ahead (a lone wave has nothing else to cover the load).
    template <int Q, bool IN, bool HAND>
    __device__ void adjoint(int q, bool rough, int t0, int t1, int buf, double (&B)[P]) {
        const int lane = lane_id();
        const int CH = ACH;
        const unsigned long long fl =
            (unsigned long long)(adjoint_flops(P, Q >= 0 ? Q : q, a.d) +
                                 cell_flops(P, Q >= 0 ? Q : q, a.d));
        double ahead[HAND ? P : 1];
        if constexpr (HAND) {
            if (!rough) {
#pragma unroll
                for (int i = 0; i < P; ++i) B[i] = scr.load(buf + kCkptEvery * P + i);
            }
#pragma unroll
            for (int i = 0; i < P; ++i) ahead[i] = scr.load(buf + (t1 - 1 - t0) * P + i);
        }
        RingPos<ARB> rp;
        rp.set(t1 - 1 - lane);
        for (int t = t1 - 1; t >= t0; --t) {
            const int col = t - lane;
            const bool act = lane_ok && (IN || (col >= 0 && col < m));
            {
                const unsigned cnt = (unsigned)__builtin_popcountll(ballot(act));
                *cells += cnt;
                *flops += cnt * fl;
            }
            const int row0 = buf + (t - t0) * P;
            double A[P];
#pragma unroll
            for (int i = 0; i < P; ++i) A[i] = HAND ? ahead[HAND ? i : 0] : scr.load(row0 + i);
            if (rough) {
#pragma unroll
                for (int i = 0; i < P; ++i) B[i] = scr.load(kCkptEvery * P + row0 + i);
            }
            if constexpr (HAND) {
                const int nrow = t > t0 ? row0 - P : row0;
#pragma unroll
                for (int i = 0; i < P; ++i) ahead[i] = scr.load(nrow + i);
            }
            double dxv[D];
            double c0 = 0.0, c1 = 0.0;
#pragma unroll
            for (int ch = 0; ch < D; ch += 2) {
                dxv[ch] = L.dx_at(ch, rp);
                dxv[ch + 1] = L.dx_at(ch + 1, rp);
                c0 = fma(dy[ch], dxv[ch], c0);
                c1 = fma(dy[ch + 1], dxv[ch + 1], c1);
            }
            const double c = c0 + c1;
            // cotangent of the top edge: from the lane above, the strip above
            // (top lane of a full strip) or the seed of the corner cell
            const int tcol = t - topl;  // column of the top lane at this step
            double lAo[P];
            if (has_above) {
                const double* lsrc = &L.lin[(((tcol >= 0 ? tcol : 0) / CH) & 1) * CH * P +
                                            ((tcol >= 0 ? tcol : 0) % CH) * P];
#pragma unroll
                for (int i = 0; i < P; ++i) lAo[i] = shift_down(lAprev[i], lsrc[i]);
            } else {
                const bool corner = !IN && col == m - 1;
                double f = seed_scale;
#pragma unroll
                for (int i = 0; i < P; ++i) {
                    const double topv = corner ? f : 0.0;
                    lAo[i] = shift_down(lAprev[i], topv);
                    if (nrows < kWave) lAo[i] = lane == topl ? topv : lAo[i];
                    f = f * R(i + 1);
                }
            }
            // (past the end of the row every cotangent stays 0: c = 0 there)
            if (!IN && right_in && col == m - 1 && lane_ok) {
                const double* lp = lamv + ((int64_t)s * kWave + lane) * P;
#pragma unroll
                for (int i = 0; i < P; ++i) lBst[i] = lp[i];
            }
            // column 0 on a left line: the left edge is recovered like any
            // other (it is the right edge of the block to the left)
            const bool axis = !IN && col == 0 && left == nullptr;
            double lA[P], lB[P];
            double gc;
            // (rough: B is the stored left edge)
            if constexpr (Q >= 0)
                gc = cell_adjoint_fixed<P, Q>(A, B, c, axis, !rough, lAo, lBst, lA, lB, R);
            else
                gc = cell_adjoint<P>(A, B, c, q, axis, !rough, lAo, lBst, lA, lB, R);
            if (!act) gc = 0.0;
            if (!IN && left_out && act && col == 0) {
                double* lp = lamv + ((int64_t)s * kWave + lane) * P;
#pragma unroll
                for (int i = 0; i < P; ++i) lp[i] = lB[i];
            }
#pragma unroll
            for (int ch = 0; ch < D; ++ch) gy[ch] = fma(gc, dxv[ch], gy[ch]);
            if (act) {
#pragma unroll
                for (int ch = 0; ch < D; ++ch) {
                    double& gv = L.gx_at(ch, rp);
                    gv = fma(gc, dy[ch], gv);
                }
                if (has_below && lane == 0) {
                    // lane 0's column is t (a uniform address)
#pragma unroll
                    for (int i = 0; i < P; ++i) L.lout[((unsigned)t % (unsigned)CH) * P + i] = lA[i];
                }
            }
            rp.prev();
#pragma unroll
            for (int i = 0; i < P; ++i) {
                lBst[i] = lB[i];
                lAprev[i] = lA[i];
            }
        }
    }

    // Before the segments: the strip's rows and an empty ring.
    __device__ void begin() {
        const int lane = lane_id();
        m = g.m;
        const int row0 = s * kWave;
        nrows = min(kWave, g.n - row0);
        lane_ok = lane < nrows;
        has_below = s > 0 || below_line;
        has_above = row0 + kWave < g.n || above_blk;
        R.init();
        const int l = row0 + lane;
#pragma unroll
        for (int ch = 0; ch < D; ++ch) {
            dy[ch] = (ch < a.d && lane_ok)
                         ? g.y[(int64_t)(l + 1) * a.d + ch] - g.y[(int64_t)l * a.d + ch]
                         : 0.0;
            gy[ch] = 0.0;
        }
        for (int e = (int)threadIdx.x; e < 2 * D * ARB; e += (int)blockDim.x) L.xg[e] = 0.0;
        dx_lo = kCkptEvery * ((m + kCkptEvery - 1) / kCkptEvery);
        lin_lo = ACH * ((m + ACH - 1) / ACH);
        bin_chunk = -1;
#pragma unroll
        for (int i = 0; i < P; ++i) {
            lAprev[i] = 0.0;
            lBst[i] = 0.0;
        }
        topl = has_above ? kWave - 1 : nrows - 1;
    }

    // After them: dL/d(dy_l) of this lane's row.
    __device__ void end() {
        if (lane_ok) {
            double* gp = gyp + (int64_t)(s * kWave + lane_id()) * a.d;
#pragma unroll
            for (int ch = 0; ch < D; ++ch)
                if (ch < a.d) atomicAdd(&gp[ch], gy[ch]);
        }
    }

    // One wave does both halves of every segment.
    __device__ bool sweep() {
        begin();
        wave_sync();
        const int T = m + nrows - 1;
        for (int t0 = ((T - 1) / kCkptEvery) * kCkptEvery; t0 >= 0; t0 -= kCkptEvery) {
            const int t1 = min(t0 + kCkptEvery, T);
            const int rec = depth_at(t0);
            const int q = rec % kRoughFlag;
            const bool rough = rec >= kRoughFlag;
            load_dx_down_to(t0 - (kWave - 1));
            if (has_above && !load_lin_down_to(max(t0 - (kWave - 1), 0))) return false;
            load_bin(min(t0, m - 1) / ACH);
            segment_at_depth<(P <= 12 ? 0 : -1), 3>(q, rough, t0, t1, 0);
            if (t0 < m && (t0 % ACH) == 0) flush_cols(t0, min(t0 + ACH, m));
        }
        end();
        wave_sync();
        return true;
    }

    // Two waves of one workgroup: wave 1 recomputes segment k while wave 0 runs
    // the adjoint of segment k + 1, one barrier per segment.  (Both waves leave
    // after the same barrier: sigk_stop.h.)
    __device__ bool sweep_two(int wave, StopFlags& stop) {
        begin();
        __syncthreads();
        const int T = m + nrows - 1;
        const int nseg = (T + kCkptEvery - 1) / kCkptEvery;
        for (int k = nseg - 1; k >= -1; --k) {
            const int mine = wave == 1 ? k : k + 1;
            if (mine >= 0 && mine < nseg) {
                const int t0 = mine * kCkptEvery, t1 = min(t0 + kCkptEvery, T);
                const int rec = depth_at(t0);
                const int q = rec % kRoughFlag;
                const bool rough = rec >= kRoughFlag;
                const int buf = (mine & 1) * 2 * kCkptEvery * P;
                if (wave == 1) {
                    load_dx_down_to(t0 - (kWave - 1));
                    load_bin(min(t0, m - 1) / ACH);
                    segment_at_depth<(P <= 12 ? 0 : -1), 1>(q, rough, t0, t1, buf);
                    __builtin_amdgcn_s_waitcnt(0);  // the buffer is written
                } else if (has_above && !load_lin_down_to(max(t0 - (kWave - 1), 0))) {
                    if (lane_id() == 0) stop.raise(k);
                } else {
                    segment_at_depth<(P <= 12 ? 0 : -1), 2>(q, rough, t0, t1, buf);
                    if (t0 < m && (t0 % ACH) == 0) flush_cols(t0, min(t0 + ACH, m));
                }
            }
            __syncthreads();
            if (uniform(stop.test(k))) return false;
        }
        if (wave == 0) end();
        return true;
    }
};

// Points S at strip `strip` of pair (or block slot) `pair`.
template <int P, int D>
__device__ __forceinline__ void place_strip(StripBwd<P, D>& S, const BwdArgs& b, const Geo& g,
                                            const BlockRef& r, int pair, int strip) {
    const FwdArgs& a = b.f;
    S.ck = b.ckpt + g.ckpt + (int64_t)strip * ckpt_strip_doubles(g.m, P);
    S.ckq = S.ck + ckpt_states(g.m) * 2 * P * kWave;
    if (a.mode == kModeTable) {
        const PairDesc& pd = a.desc[pair];
        S.snap_in = b.snap + pd.snap_off + (int64_t)strip * g.m * P;
        S.lam_row = b.lam_front + pd.front_off;
        S.lam_prog = b.lam_prog + pd.prog_off;
        S.seed_scale = b.grad_out[pair];
        S.gxp = b.gdx + pd.x_off;
        S.gyp = b.gdx + pd.y_off;
    } else {
        const BlockGeo& k = a.blk;
        S.snap_in = (strip == 0 && r.bot) ? r.bot
                                          : b.snap + g.front + (int64_t)strip * g.m * P;
        S.lam_row = b.lam_front + (int64_t)r.J * k.cb * P;
        S.lam_prog = b.lam_prog + g.prog;
        // the grid's corner cell belongs to the top-right block
        S.seed_scale = (!r.above && !r.right) ? b.grad_out[0] : 0.0;
        S.gxp = b.gdx + (int64_t)r.J * k.cb * a.d;
        S.gyp = b.gdx + k.y_gdx + (int64_t)r.I * k.rb * a.d;
        S.left = r.left;
        S.below_line = r.bot != nullptr;
        S.above_blk = r.above;
        S.lamv = b.lam_v + (int64_t)r.I * k.rb * P;
        S.right_in = r.right;
        S.left_out = r.J > 0;
    }
}

// Pair, strip and geometry of ticket t; 1: run it, 0: skip it, -1: no more.
template <int P>
__device__ __forceinline__ int take_ticket(const BwdArgs& b, unsigned t, int& pair, int& strip,
                                           Geo& g, BlockRef& r) {
    const FwdArgs& a = b.f;
    if (a.mode == kModeTable) {
        pair = b.tickets[t].pair;
        strip = b.tickets[t].strip;
        if (pair < 0) return -1;  // unused slots close a table built on the device
        g = resolve(a, pair, P, 0);
        return 1;
    }
    // kModeBlock: the blocks of one anti-diagonal, strips top-down
    pair = (int)(t % (unsigned)a.blk.nb);
    strip = a.blk.kb - 1 - (int)(t / (unsigned)a.blk.nb);
    g = resolve_block(a, pair, P, r);
    return strip * kWave >= g.n ? 0 : 1;  // the top block row has fewer strips
}

// (two waves per SIMD at orders up to 6 with d <= 8: the scheduler otherwise
// takes a few registers more than 256 at order 6, 17% slower)
template <int P, int D>
__global__ void __launch_bounds__(kWave)
    __attribute__((amdgpu_waves_per_eu(P <= 6 && D <= 8 ? 2 : 1))) bwd_kernel(BwdArgs b) {
    __shared__ LdsBwd<P, D> L;
    const FwdArgs& a = b.f;
    const int lane = lane_id();
    double* scratch = b.scratch + (int64_t)blockIdx.x * (2 * kCkptEvery * P * kWave);
    unsigned long long cells = 0, flops = 0;
    for (;;) {
        unsigned t = 0;
        if (lane == 0) t = atomicAdd(&a.hdr->ticket2, 1u);
        t = (unsigned)uniform((int)t);
        if ((int64_t)t >= b.ntickets) break;
        if (uniform((int)(load_status(a.hdr) & SIGK_ERR_WATCHDOG))) break;
        int pair, strip;
        Geo g;
        BlockRef r;
        const int todo = take_ticket<P>(b, t, pair, strip, g, r);
        if (todo < 0) break;
        if (todo == 0) continue;
        StripBwd<P, D> S(b, g, L, strip);
        S.scr.init(scratch, 2 * kCkptEvery * P);
        S.cells = &cells;
        S.flops = &flops;
        place_strip<P, D>(S, b, g, r, pair, strip);
        if (!S.sweep()) break;
    }
    if (lane == 0) {
        atomicAdd(&a.hdr->bwd_cells, cells);
        atomicAdd(&a.hdr->bwd_flops, flops);
    }
}

// The same with two waves per strip (sweep_two), for launches of so few strips
// that every wave has a SIMD to itself: the chain then runs at the adjoint's
// instructions per step and not at those of recompute and adjoint together
// (order 10: about 900 and 380).  Gram matrix of 16 paths of 100 points with its
// gradient, order 10: 1179 -> 1001 us; 20,001-point pair, order 5: 81.5 -> 63.0
// ms.  With more strips than that the
// recomputing waves would take the place of working ones.
template <int P, int D>
__global__ void __launch_bounds__(2 * kWave) bwd_two_kernel(BwdArgs b) {
    __shared__ LdsBwd<P, D> L;
    __shared__ StopFlags stop;
    __shared__ int ticket;
    const FwdArgs& a = b.f;
    const int lane = lane_id();
    const int wave = uniform((int)(threadIdx.x >> 6));
    double* scratch = b.scratch + (int64_t)blockIdx.x * (4 * kCkptEvery * P * kWave);
    unsigned long long cells = 0, flops = 0;
    if (threadIdx.x == 0) stop.clear();
    for (;;) {
        __syncthreads();  // both waves are done with the previous strip
        if (threadIdx.x == 0) {
            int t = (int)atomicAdd(&a.hdr->ticket2, 1u);
            if ((int64_t)t >= b.ntickets || (load_status(a.hdr) & SIGK_ERR_WATCHDOG)) t = -1;
            ticket = t;
        }
        __syncthreads();
        const int t = uniform(ticket);
        if (t < 0) break;
        int pair, strip;
        Geo g;
        BlockRef r;
        const int todo = take_ticket<P>(b, (unsigned)t, pair, strip, g, r);
        if (todo < 0) break;
        if (todo == 0) continue;
        StripBwd<P, D> S(b, g, L, strip);
        S.scr.init(scratch, 4 * kCkptEvery * P);
        S.cells = &cells;
        S.flops = &flops;
        place_strip<P, D>(S, b, g, r, pair, strip);
        if (!S.sweep_two(wave, stop)) break;
    }
    if (threadIdx.x == 0) {
        atomicAdd(&a.hdr->bwd_cells, cells);
        atomicAdd(&a.hdr->bwd_flops, flops);
    }
}

#define SIGK_CAT3(a, b, c) a##b##_##c
#define SIGK_NAME(pre, P, D) SIGK_CAT3(pre, P, D)

hipError_t SIGK_NAME(launch_ckpt_, SIGK_P, SIGK_D)(const FwdArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((ckpt_kernel<SIGK_P, SIGK_D>), dim3(grid), dim3(kWave), 0, s, a,
                       a.frontier);
    return hipGetLastError();
}

hipError_t SIGK_NAME(launch_lines_, SIGK_P, SIGK_D)(const FwdArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL((lines_kernel<SIGK_P, SIGK_D>), dim3(grid), dim3(kWave), 0, s, a);
    return hipGetLastError();
}

int SIGK_NAME(occupancy_lines_, SIGK_P, SIGK_D)() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, lines_kernel<SIGK_P, SIGK_D>, kWave,
                                                     0) != hipSuccess)
        return 0;
    return nb;
}

hipError_t SIGK_NAME(launch_bwd_, SIGK_P, SIGK_D)(const BwdArgs& b, int grid, hipStream_t s) {
    hipLaunchKernelGGL((bwd_kernel<SIGK_P, SIGK_D>), dim3(grid), dim3(kWave), 0, s, b);
    return hipGetLastError();
}

template <int P, int D>
hipError_t launch_two(const BwdArgs& b, int grid, hipStream_t s) {
    if constexpr (bwd_two_compiled(P, D)) {
        hipLaunchKernelGGL((bwd_two_kernel<P, D>), dim3(grid), dim3(2 * kWave), 0, s, b);
        return hipGetLastError();
    } else {
        return hipErrorNotSupported;
    }
}
hipError_t SIGK_NAME(launch_bwd_two_, SIGK_P, SIGK_D)(const BwdArgs& b, int grid, hipStream_t s) {
    return launch_two<SIGK_P, SIGK_D>(b, grid, s);
}

int SIGK_NAME(occupancy_ckpt_, SIGK_P, SIGK_D)() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, ckpt_kernel<SIGK_P, SIGK_D>, kWave, 0) !=
        hipSuccess)
        return 0;
    return nb;
}

int SIGK_NAME(occupancy_bwd_, SIGK_P, SIGK_D)() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, bwd_kernel<SIGK_P, SIGK_D>, kWave, 0) !=
        hipSuccess)
        return 0;
    return nb;
}

}  // namespace sigk
