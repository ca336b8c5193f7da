// A solve as ONE cooperative launch, for instances whose kernel fits in the
// LDS of the whole GPU (about 40 MB on 256 CUs: 20000 x 400 needs 32 MB in FP32)
// or in device memory (the streamed form below). Each workgroup (one per CU) owns a contiguous
// block of rows and holds their stabilised Gibbs kernel in LDS: with reference
// potentials G, E_ij = exp((G_j - C_ij) / eps - m_i) in FP32 (arguments in FP64,
// from the matrix or regenerated from positions; m_i the row's largest). It
// then runs Sinkhorn iterations (Sec. III-B) in the scaling form on that kernel
// until the device-side stop rule fires. Iteration k:
//
//   1. row update of the workgroup's rows: S_i = sum_j E_ij v_j (the row scaling
//      is a_i / S_i), the row residual of the previous iterate, a_i |S_i^k /
//      S_i^(k-1) - 1|, and the column partials sum_i E_ij a_i / S_i (FP32
//      products, FP64 sums across lanes, waves and workgroups), published to
//      an exchange buffer;
//   2. workgroup w owns the blocks of 8 consecutive columns w, w + nb, ...:
//      it collects their partials from every workgroup, sums them in a fixed
//      order and publishes v_j = b_j / sum; the last workgroup also sums the
//      residuals and publishes the stop decision;
//   3. every workgroup collects the new v and the decision.
//
// A cell costs two multiply-adds per iteration and no exponential; those run
// only when a reference is taken (C is then read again):
//   - at the first iteration, and again when a scaling leaves [2^-40, 2^40];
//   - once the residual is below 1e-5, for targets below the FP32 noise. From
//     there on the iteration adds to the FP64 sums R_i of the reference, and
//     likewise to those of its columns, only the change against it, S_i = R_i +
//     sum_j E_ij (v_j - 1), so its FP32 rounding is 2^-24 of |v - 1| instead of
//     2^-24 of 1, and the phase runs on to tol where FP64 sweeps of the whole
//     cost were needed before;
//   - in the FP64 iterations (polish_iters) that end such a solve.
//
// The noise: marginal violation at the fixed point of the plain sums, emulated
// on the CPU, against that of sweeps that form every exponential anew in FP32
// from its FP64 argument: 1.3 - 2.1e-8 and 2.5 - 3.0e-8 on C-RAN layouts, 0.9 -
// 1.2e-8 and 2.1 - 2.4e-8 with column offsets of 20 - 27 eps. (References in FP32
// exponentials: 1.3 - 2.1e-8, but 2.7 - 9.2e-8 with the offsets.)
//
// What bounds it: the exchange. With the cost in LDS and an exponential per cell
// the row update alone took 4.8 us of the 9.6 us per iteration at 20000 x 400;
// now an iteration takes 5.8 us, 1.7 of them the row update. The whole solve
// with its plan went 590 -> 436 us, and the distance cost at that size (about
// 1250 iterations, 200 of them FP64 sweeps before) 16.3 -> 7.6 ms.
//
// Only O(I + J) scalings and O(nb J) partials move per iteration; the I x J cost
// is read two to four times per launch instead of once per iteration.
//
// Exchange without fences or barriers. On this GPU the L2 of an XCD is not
// coherent with the other XCDs' L2s, and an agent-scope release writes a
// whole L2 back; so every exchanged value is stored and loaded with
// agent-scope relaxed atomics (stores that write through the L2, loads served
// at the device's coherence point), and a reader simply polls a slot until it
// holds the value of the iteration it waits for. Every exchanged double
// carries its iteration number modulo 4 in the two lowest mantissa bits (a
// relative change below 2^-50, far under the FP32 phase's own rounding), so
// slots are never emptied: buffers alternate by iteration parity, a slot's
// previous content is from two iterations earlier (a different tag), and no
// producer can get two iterations ahead of a reader (it needs every
// workgroup's contribution of the iteration in between). The exchange is laid
// out for the memory system: a producer's column partials are one contiguous
// row (whole cache lines), the owner of eight consecutive columns reads whole
// lines, and the new v and the stop decision are written in several replicas
// so that the 256 polling workgroups do not all wait on the same lines.
// Every poll is bounded: a workgroup that waits too long sets an abort word
// that releases every other poller, and the launch ends with its control
// block marked.
#pragma once

#include "kernels.h"

namespace otk {

// ----------------------------------------------------------- exchange words --
__device__ __forceinline__ void put_agent(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double get_agent(const double* p) {
    return __hip_atomic_load(const_cast<double*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void put_agent(uint64_t* p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t get_agent(const uint64_t* p) {
    return __hip_atomic_load(const_cast<uint64_t*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Iteration tags in the two lowest mantissa bits of an exchanged double.
__device__ __forceinline__ double tag_value(double v, int k) {
    return __longlong_as_double((__double_as_longlong(v) & ~3ll) | (long long)(k & 3));
}
__device__ __forceinline__ bool has_tag(double v, int k) { return (__double_as_longlong(v) & 3) == (long long)(k & 3); }

constexpr int kColBlock = 8;        // columns per owner block: one 64-byte line of doubles
constexpr int kReplicas = 8;        // copies of the new v and of the decision word
constexpr int kMaxCoopGroups = 256; // workgroups of a cooperative launch (an owner polls 4 per thread)

// Layout of the exchange block (offsets in doubles, each part 64-byte aligned):
//   part  [2][nb][Jp]      column partials by iteration parity; a producer's
//                          row is contiguous, Jp = J rounded up to kColBlock
//   rpart [2][nb]          row-residual partials by parity (padded to a line)
//   gx    [2][kReplicas][Gs]  new v by parity, Gs = Jp rounded up to 512 (4 KiB
//                          between replicas)
//   dec   [2][kReplicas][8]   (iteration << 3) | decision code, as uint64, one line per replica
//   abort [8]              uint64, nonzero once a poll gave up
//   fin   [7 x kMaxCoopGroups]  scalars of the final check: five per workgroup,
//                          two per column block, tagged 1 once written
struct XchLayout {
    int Jp, Gs;
    size_t part, rpart, gx, dec, abort_, fin, total;
};
__host__ __device__ inline XchLayout persist_xch_layout(int nb, int J) {
    XchLayout L;
    L.Jp = (J + kColBlock - 1) / kColBlock * kColBlock;
    L.Gs = (L.Jp + 511) / 512 * 512;
    L.part = 0;
    L.rpart = L.part + (size_t)2 * nb * L.Jp;
    L.gx = L.rpart + ((size_t)2 * nb + 7) / 8 * 8;
    L.dec = L.gx + (size_t)2 * kReplicas * L.Gs;
    L.abort_ = L.dec + (size_t)2 * kReplicas * 8;
    L.fin = L.abort_ + 8;
    L.total = L.fin + 7 * kMaxCoopGroups;
    return L;
}
__host__ __device__ inline size_t persist_exchange_doubles(int nb, int J) { return persist_xch_layout(nb, J).total; }

// Pause between two polls: short while the other side is about to answer,
// longer in a wait that lasts (a workgroup that an earlier instance of its
// batch still holds), so that the polls leave the memory system alone.
__device__ __forceinline__ void poll_pause(int spin) {
    if (spin < 64) __builtin_amdgcn_s_sleep(1);
    else __builtin_amdgcn_s_sleep(16);
}

// Polls U tagged slots per lane of one wave (slot u of lane l at
// base[(u 64 + l) stride] for u 64 + l < n) until each holds tag k; absent
// slots read 0. Returns false if the wait gave up (bound reached or abort set).
template <int U>
__device__ bool poll_tagged(const double* base, int64_t stride, int n, int k, double (&x)[U], uint64_t* abort_word,
                            int max_spin) {
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int p = u * kWave + lane;
        x[u] = p < n ? get_agent(base + (int64_t)p * stride) : tag_value(0.0, k);
    }
    int spin = 0;
    for (;;) {
        bool pend = false;
#pragma unroll
        for (int u = 0; u < U; ++u) pend |= !has_tag(x[u], k);
        if (!__any(pend)) return true;
        if ((++spin & 31) == 0 && (get_agent(abort_word) != 0 || spin > max_spin)) {
            put_agent(abort_word, (uint64_t)1);
            return false;
        }
        poll_pause(spin);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = u * kWave + lane;
            if (!has_tag(x[u], k)) x[u] = get_agent(base + (int64_t)p * stride);
        }
    }
}

// ------------------------------------------------------- persistent solve --
struct PersistArgs {
    int64_t I;
    int J;
    int Jp;   // row stride of the kernel tile (in LDS ncl * LPR, in device memory J rounded up
              // to 4; the padding holds 0)
    int ncl;  // cells per lane of a row: column q LPR + sub for q < ncl (<= CPL)
    int rpw;  // rows per workgroup: a whole number of wave steps
    int max_spin;
    int hold_iter;  // > 0: at iteration k0 + hold_iter of the launch no new v is published, so
                    // every wait after it ends by giving up (exercises that path); else 0
    double stall_below;
    const double* a;
    const double* b;
    double* f[2];  // iterate k lives in f[k & 1], g[k & 1]
    double* g[2];
    double* xch;   // exchange block (persist_exchange_doubles)
    Ctl* ctl;
    const SolveParams* prm;
    float* tile;   // the stored kernel in device memory, I x Jp (streamed form only)
    int validate;  // the first reference also checks the matrix (OT_EINVAL on a bad entry)
    void* plan_out;  // I x J plan the final check writes, or null
    int plan_f64;
    double* loads;   // J: RRH loads the final check sums, or null
    int batch;       // an instance of a batch: its control block carries a phase (kPh...)
    int polish;      // FP64 iterations after the stop rule
    int cap;         // iterations of this launch, a multiple of 4 (an instance of a batch that reaches it
                     // leaves with its iterate and goes on in sweeps or in another launch)
};

// Static LDS of the cooperative phase.
struct PersistShared {
    Ctl cs;  // decision workgroup: the control block for the whole launch
    double e2tab[64];
    double wres[8];
    double wst[8][7];           // the final check's scalars
    double ored[8][kColBlock];  // per-wave column sums of an owned block
    uint32_t dec;
    int flag[2];  // by iteration parity: 1 a wait gave up, 2 v not finite, 4 v out of the reference's range
};

// Column blocks each workgroup owns at most (workgroup w owns w, w + nb, ...).
__host__ __device__ inline int persist_owned_blocks(int nb, int J) {
    const int nblk = (J + kColBlock - 1) / kColBlock;
    return (nblk + nb - 1) / nb;
}
// Dynamic LDS of k_persist in bytes (the layout the kernel carves): the
// tile of rpw rows of stride Jp (Jp = 0: the tile is in device memory), a slack
// of (CPL - ncl) LPR floats after it, then the column vectors
// (G, v), the row vectors (a, m, R, S), b and the reference column sums of
// the owned columns, x and the fold buffer of the column partials (FP32 partials of all waves at
// once up to 512 columns, of half of them for wider rows), both of width
// CPL LPR, so that a lane handles all its cells alike. An FP64 kernel (elem 8)
// has the tile and x in FP64 and keeps the v of the iterate before.
__host__ __device__ inline size_t persist_lds_bytes(int rpw, int J, int Jp, int waves, int width, int slack, int nb,
                                                   int elem = 4) {
    const size_t Jr2 = (size_t)((J + 1) & ~1);
    return ((size_t)rpw * Jp + (size_t)slack) * elem + (elem == 8 ? 3 : 2) * Jr2 * 8 + 4 * (size_t)rpw * 8 +
           2 * (size_t)kColBlock * persist_owned_blocks(nb, J) * 8 + (size_t)width * elem +
           (size_t)(J > 512 ? waves / 2 : waves) * width * 4;
}

// Kinds of iteration of the cooperative phase (the same in every workgroup):
// a reference taken for plain sums, plain sums, one taken for delta sums,
// delta sums.
enum : int { kItRef = 0, kItPlain = 1, kItRefDelta = 2, kItDelta = 3 };
// Decision codes: bit 0 stop, bit 1 take a reference for delta sums next (in
// FP64: the iterate before is the returned one), bit 2 leave without the check.
constexpr int kDecStop = 1, kDecRefDelta = 2, kDecPrev = 2, kDecSkip = 4;
// Delta sums begin once the residual is below this: the scalings
// then stay within about 1e-5 / (1 - rate) of 1, so the FP32 delta sums resolve
// residuals down to about 1e-12, far below the FP32 noise (2e-8) of the plain
// sums; an earlier switch would buy nothing, a later one comes too close to
// that noise.
constexpr double kDeltaBelow = 1e-5;
// A reference for plain sums is renewed when a scaling leaves [2^-40, 2^40]: an entry
// flushed to zero in FP32 (below 2^-126 of its row's largest) then stands for
// less than 2^-46 of its row's sum, and so for 2^-46 a_i of its column's, which all
// of them together move by less than 2^-46 of the mass.
constexpr double kScaleMax = 0x1p40;
// The final check sums RRH loads up to this many cells per lane (416 columns):
// the second set of FP64 column sums takes wider rows past the registers.
constexpr int kLoadsCpl = 13;
// The delta sums keep |v - 1| below this (else the reference is renewed).
constexpr double kDeltaMax = 0.125;

// The stop rule of the cooperative phase, run by one lane: like the fast mode
// of bookkeep, except that a solve whose target lies below the FP32 noise
// (stall_below) goes on past it: the plain sums are left for delta sums
// (returned as kDecRefDelta), whose residuals are good to about
// 1e-6 of the residual r_ref at which the reference was taken and are therefore
// compared with tol itself. Long delta phases (a slowly converging instance
// whose scalings drift far from the reference) renew the reference.
//
// The solve then ends, as one in sweeps does, with `polish` FP64 iterations,
// unless its residual met a target above the noise: iterations that take a
// reference, whose exponentials and sums are FP64 throughout (one costs 25 us at
// 20000 x 400, 5 % of a solve). polish_left counts those still to come.
__device__ __forceinline__ int bookkeep_coop(Ctl* c, double rsum, int kind, double stall_below, int polish,
                                             double& r_ref, int& k_ref) {
    const int k = c->iter + 1;
    const double r = c->has_prev ? rsum / c->mass : pinf64();
    const bool bad = c->numeric_bad || (c->has_prev && !isfinite(r));
    c->r_last = r;
    c->iter = k;
    c->has_prev = 1;
    c->last_fp64 = c->polish_left > 0 ? 1 : 0;
    int code = 0;
    if (c->polish_left > 0) {
        c->fp64_iters += 1;
        code = --c->polish_left > 0 ? kDecRefDelta : kDecStop;
    } else {
        const double target = c->tol_fast > 0.0 ? c->tol_fast : c->tol;
        const bool fine = kind == kItRefDelta || kind == kItDelta;  // residuals of delta sums
        double mn = pinf64();
        int nfin = 0;
        for (int q = 0; q < 4; ++q)
            if (isfinite(c->r_hist[q])) { mn = fmin(mn, c->r_hist[q]); ++nfin; }
        const double noise = fine ? 1e-6 * r_ref : target >= stall_below ? stall_below : 0.0;
        const bool stall = (nfin >= 1) && isfinite(r) && (r < noise) && (r > 0.95 * mn);
        for (int q = 3; q > 0; --q) c->r_hist[q] = c->r_hist[q - 1];
        c->r_hist[0] = r;
        const bool met = r < target && (fine || target >= stall_below);
        const bool at_check = c->check_every <= 1 || k % c->check_every == 0;
        if (kind == kItRefDelta) k_ref = k;
        if (fine ? (k - k_ref >= 64 && r < 0.03 * r_ref && !met) : (target < stall_below && r < kDeltaBelow)) {
            r_ref = r;
            code = kDecRefDelta;
        }
        if (at_check && (met || stall)) {
            c->polish_left = r < target && target >= stall_below ? 0 : polish;
            code = c->polish_left > 0 ? kDecRefDelta : kDecStop;
        }
    }
    if (k >= c->max_iter) code = kDecStop;
    if (bad) {
        c->numeric_bad = 1;
        c->done = 1;
        c->result_iter = k;
        code = kDecStop;
    }
    if (code == kDecStop) c->stop = 1;
    return code;
}

// Lane layout: a row is handled by LPR lanes (16, 32 or 64) of CPL cells each: 16
// up to 64 columns, where 32 lanes left half of the 16-byte reads empty (an
// instance of a batch that fills its LDS with rows of 30 columns: 10.8 -> 7.0 us
// per iteration). The
// iterations read it 16 bytes per lane (lane `sub` owns columns (c LPR + sub) 4
// to + 3 of load c), the up to three cells past the last whole load word by
// word (columns q LPR + sub). Every cell is processed without a branch: cells
// past J read on into the next row of the tile, or into a zero slack after it,
// and get x = 0. A wave advances R = 64 / LPR rows per step and takes U steps
// together. References are taken with columns q LPR + sub, as the cost is read.
//
// GM: the streamed form, for instances whose kernel does not fit in LDS. The
// tile is in device memory and every iteration reads it once, PD row steps
// ahead (64 - 128 KB in flight per CU). Bound by that read.
//
// One workgroup's part of the phase: workgroup blk of the nb that solve the
// instance together.
//
// F64: the phase of a solve in FP64. The kernel, v and every product are FP64, the
// references take FP64 exponentials, and the stop rule is that of the
// FP64 sweeps: the iterate before the one just computed is returned once its
// residual is below tol. Bound by the exchange, too: a solve of 2999 x 197 with
// 72 iterations takes 351 us, with a sweep and a fold launch per iteration
// (7.2 + 4.3 us) it took 1038.
template <class Src, int CPL, int LPR, int WAVES, bool GM, bool LEAN = false, bool F64 = false>
__device__ __forceinline__ void persist_run(const PersistArgs& A, const Src& src, const int nb, const int blk,
                                            PersistShared& ps) {
    extern __shared__ __align__(16) float4 sm4[];  // (its 16-byte reads have to be aligned)
    double* sm = reinterpret_cast<double*>(sm4);
    constexpr int R = kWave / LPR;
    constexpr int T = WAVES * kWave;
    using Real = std::conditional_t<F64, double, float>;
    static_assert(!F64 || (!GM && !LEAN), "the FP64 kernel is held in LDS, by a solve of its own");
    constexpr int U = F64 ? (CPL <= 4 ? 5 : CPL <= 8 ? 3 : 2) : CPL <= 4 ? 8 : CPL <= 16 ? (LEAN && CPL > 8 ? 4 : 5) : 1;  // row steps at a time (their sums' chains overlap)
    static_assert(WAVES >= 4 && WAVES <= 8, "at least one wave per publishing column block, wres and ored sized for 8");
    int J = A.J, Jp = A.Jp, ncl = A.ncl;
    const int rpw = A.rpw;
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));  // (nothing derived from it is kept across a batch's instances)
    int lane = tid & (kWave - 1), w = tid / kWave;
    int sub = lane % LPR, rg = lane / LPR;
    const int64_t r0 = (int64_t)blk * rpw;
    const int nrows = (int)max((int64_t)0, min((int64_t)rpw, A.I - r0));
    constexpr int WD = CPL * LPR;  // width of x and of the fold buffer
    const int Jr2 = (J + 1) & ~1;
    const int slack = GM ? 0 : (CPL - ncl) * LPR;  // (a multiple of 16 floats: what follows stays 8-byte aligned)
    Real* tile = reinterpret_cast<Real*>(sm);
    if constexpr (GM) tile = A.tile + r0 * Jp;
    double* gl = GM ? sm : reinterpret_cast<double*>(tile + (size_t)rpw * Jp + slack);  // G_j of the reference
    double* vl = gl + Jr2;    // v_j = exp((g_j - G_j) / eps)
    double* al = vl + Jr2;    // a_i
    double* ml = al + rpw;    // m_i: the shift of row i's stored kernel entries (log2)
    double* Rl = ml + rpw;    // R_i = sum_j E_ij of the FP64 entries
    double* Sl = Rl + rpw;    // S_i = sum_j E_ij v_j of the last row update
    const int nown = persist_owned_blocks(nb, J);
    double* bl = Sl + rpw;    // b_j of the owned columns (8 per owned block), times asc
    double* cl = bl + (size_t)kColBlock * nown;  // their column sums at the reference (delta sums)
    double* vp = cl + (size_t)kColBlock * nown;  // FP64: v_j of the iterate before
    Real* xl = reinterpret_cast<Real*>(vp + (F64 ? Jr2 : 0));  // v_j, or v_j - 1 for delta sums
    float* red = reinterpret_cast<float*>(xl + WD);
    Ctl& cs = ps.cs;
    auto& e2tab = ps.e2tab;
    auto& wres = ps.wres;
    auto& wst = ps.wst;
    auto& ored = ps.ored;
    auto& s_dec = ps.dec;
    auto& s_flag = ps.flag;

    const XchLayout X = persist_xch_layout(nb, J);
    double* part = A.xch + X.part;
    double* rpart = A.xch + X.rpart;
    double* gx = A.xch + X.gx;
    uint64_t* dec = reinterpret_cast<uint64_t*>(A.xch + X.dec);
    uint64_t* abort_word = reinterpret_cast<uint64_t*>(A.xch + X.abort_);
    const int rep = blk % kReplicas;  // the replica of v and of the decision this workgroup reads

    Ctl* ctl = A.ctl;
    if (ctl->stop | ctl->done) return;  // the same words for every workgroup
    const int k0 = ctl->iter;
    int has_prev = ctl->has_prev;
    const double kk = A.prm->kk, eps = A.prm->eps, inv_eps = 1.0 / A.prm->eps;
    // The row scalings a_i / S_i are FP32 values: marginals of any total mass are
    // brought to one of [1, 2) by a power of two, which the column update takes
    // out again (S_i may drift over 2^40 between references; at a mass of 1e-30
    // the scalings would be flushed to zero).
    const double asc = F64 ? 1.0 : readlane_d(ldexp(1.0, -min(max(ilogb(ctl->mass), -1000), 1000)), 0);

    exp2_tab_fill(e2tab);
    for (int lr = tid; lr < rpw; lr += T) {
        al[lr] = lr < nrows ? A.a[r0 + lr] : 0.0;
        ml[lr] = 0.0;
        Rl[lr] = Sl[lr] = 1.0;
    }
    const double* g_in = (k0 & 1) ? A.g[1] : A.g[0];
    for (int j = tid; j < J; j += T) {
        gl[j] = g_in[j];
        vl[j] = 1.0;
    }
    for (int e = tid; e < kColBlock * nown; e += T) {
        const int j = (blk + (e / kColBlock) * nb) * kColBlock + e % kColBlock;
        bl[e] = j < J ? A.b[j] * asc : 1.0;
        cl[e] = 0.0;
    }
    for (int e = tid; e < slack; e += T) tile[(size_t)rpw * Jp + e] = 0;
    // column of cell q of this lane: as the references are taken, and as the
    // iterations read the tile
    auto col_ref = [&](int q) { return q * LPR + sub; };
    constexpr int NV = F64 ? 0 : CPL / 4;  // 16-byte loads of a lane and row step
    auto col_it = [&](int q) { return q < 4 * NV ? ((q / 4) * LPR + sub) * 4 + q % 4 : q * LPR + sub; };
    for (int j = tid; j < WD; j += T) xl[j] = 0;
    if (tid < 2) s_flag[tid] = 0;
    // the decision workgroup (the last one: with fewer column blocks than
    // workgroups it owns none) sums the residuals and takes the stop decision
    const int dblk = nb - 1;
    if (blk == dblk && tid == 0) cs = *ctl;
    double r_ref = ctl->r_last;  // (the deciding lane's)
    int k_ref = k0;

    const int steps = rpw / (WAVES * R);
    [[maybe_unused]] volatile int bad_before = 0;
    double res = 0.0;  // this lane's part of the row residual of the previous iterate
    int k = k0, kind = kItRef;
    // (an instance that a launch before this one left in delta sums or in its polish)
    if constexpr (!F64)
        if (k0 > 0 && (ctl->polish_left > 0 || (ctl->r_last < kDeltaBelow && ctl->tol_fast < A.stall_below)))
            kind = kItRefDelta;

    // Row update of an iteration that takes a new reference G = g: the kernel
    // entries E_ij = 2^(t_ij - m_i), t_ij = (G_j - C_ij) kk, m_i about the row maximum,
    // as FP64 exponentials (table-driven), stored in FP32; S_i = R_i and the
    // column partials sum_i E_ij a_i / S_i are sums of the FP64 entries. (As FP32
    // exponentials an entry that a scaling later raises to a column's largest
    // carried the rounding of an argument of up to 126.)
    auto take_reference = [&](double (&ac)[CPL]) {
        constexpr bool kAhead = Src::kCheap && CPL <= 16;  // a row's loads one step ahead, where the registers allow it
        double* stage = reinterpret_cast<double*>(red);
        src.stage(stage, J);
        for (int j = tid; j < J; j += T) {
            gl[j] += eps * log(vl[j]);
            vl[j] = 1.0;
        }
        // the previous row sums as logarithms (log2 sum_j exp((g_j - C_ij) / eps)),
        // at the launch's start from f
        for (int lr = tid; lr < nrows; lr += T)
            Rl[lr] = k == k0 + 1 ? (has_prev ? (log(al[lr]) - ((k0 & 1) ? A.f[1] : A.f[0])[r0 + lr] * inv_eps) * kLog2e : 0.0)
                                 : ml[lr] + log2(Sl[lr]);
        if constexpr (F64) {  // (kept in case iterate k - 1 is the returned one)
            double* fo = ((k - 1) & 1) ? A.f[1] : A.f[0];
            for (int lr = tid; lr < nrows && k > k0 + 1; lr += T) fo[r0 + lr] = eps * (log(al[lr]) - kLn2 * Rl[lr]);
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < CPL; ++q) ac[q] = 0;
        typename Src::template Raw<1> nraw[kAhead ? CPL : 1];
        [[maybe_unused]] auto fetch = [&](int st, auto& to) {
            const int lr = (st * WAVES + w) * R + rg;
            auto row = src.row(r0 + (lr < nrows ? lr : 0));
#pragma unroll
            for (int q = 0; q < CPL; ++q)
                if (q < ncl) to[q] = src.template load<1>(row, q * LPR + sub, J);
        };
        if constexpr (kAhead) fetch(0, nraw);
        [[maybe_unused]] bool bad_cost = false;
        for (int st = 0; st < steps; ++st) {
            const int lr = (st * WAVES + w) * R + rg;
            const bool vrow = lr < nrows;
            const int64_t i = r0 + (vrow ? lr : 0);
            double t[CPL];
            float mx = -__builtin_huge_valf();
            auto row = src.row(i);
            auto arg = [&](int q, const typename Src::template Raw<1>& raw) {
                t[q] = -pinf64();
                const int j = q * LPR + sub;
                if (q < ncl && j < J && vrow) {
                    const double c = src.template cost<true, 1>(row, raw, 0, i, j, stage);
                    if constexpr (Src::kTag <= 2) bad_cost |= !isfinite(c);
                    else if constexpr (Src::kTag <= 4) bad_cost |= !(c > 0.0 && isfinite(c));  // (R > 0 and finite)
                    t[q] = (gl[j] - c) * kk;
                }
                mx = fmaxf(mx, (float)t[q]);
            };
            if constexpr (kAhead) {
                typename Src::template Raw<1> raw[CPL];
#pragma unroll
                for (int q = 0; q < CPL; ++q) raw[q] = nraw[q];
                if (st + 1 < steps) fetch(st + 1, nraw);
#pragma unroll
                for (int q = 0; q < CPL; ++q) arg(q, raw[q]);
            } else {
                constexpr int G = CPL < 4 ? CPL : 4;  // cells at a time
#pragma unroll
                for (int q0 = 0; q0 < CPL; q0 += G) {
                    typename Src::template Raw<1> raw[G];
#pragma unroll
                    for (int u = 0; u < G; ++u)
                        if (q0 + u < CPL && q0 + u < ncl) raw[u] = src.template load<1>(row, (q0 + u) * LPR + sub, J);
#pragma unroll
                    for (int u = 0; u < G; ++u)
                        if (q0 + u < CPL) arg(q0 + u, raw[u]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            const double m = fmax((double)group_max<LPR>(mx), -1e300);
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
                t[q] = exp2_tab_neg(t[q] - m, e2tab);
                if constexpr (!kAhead)
                    if (q % 4 == 3) __builtin_amdgcn_sched_barrier(0);
            }
            double s = 0, s2 = 0;  // even and odd cells: two shorter add chains
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
                if (q & 1) s2 += t[q];
                else s += t[q];
            }
            const double S = group_sum<LPR>(s + s2);
            const double wq = vrow ? al[lr] * asc / S : 0.0;
            Real* trow = tile + (size_t)lr * Jp + sub;
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
                ac[q] = fma(t[q], wq, ac[q]);
                if (GM ? (vrow && q * LPR + sub < Jp) : q < ncl) trow[q * LPR] = (Real)t[q];
            }
            if (sub == 0 && vrow) {
                ml[lr] = m;
                Sl[lr] = S;
            }
        }
        // (the verdict is final once the value comes back, before this workgroup
        // publishes anything; in a batch a bad cost is a numeric failure)
        if ((A.validate || A.batch) && k == k0 + 1 && __any(bad_cost) && lane == 0)
            bad_before = __hip_atomic_fetch_or(A.batch ? &ctl->numeric_bad : &ctl->input_bad, A.batch ? 1 : 8,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();  // (the fold also reuses the staged source data's LDS)
        // |rowsum_i - a_i| of the previous iterate, from the change of the log-sum-exp
        res = 0.0;
        for (int lr = tid; lr < nrows; lr += T) {
            if (has_prev) res += al[lr] * fabs(expm1(kLn2 * (ml[lr] + log2(Sl[lr]) - Rl[lr])));
            Rl[lr] = Sl[lr];
        }
    };

    // Row update against the stored kernel: S_i = sum_j E_ij v_j, or from the
    // reference's FP64 sums S_i = R_i + sum_j E_ij (v_j - 1), whose FP32 rounding scales
    // with |v - 1|; the column partials sum_i E_ij a_i / S_i, or their change
    // against the reference, sum_i E_ij (a_i / S_i - a_i / R_i).
    auto rows = [&](auto delta, Real (&acc)[CPL]) {
        constexpr bool D = decltype(delta)::value;
        Real x[CPL];
#pragma unroll
        for (int q = 0; q < CPL; ++q) x[q] = xl[col_it(q)];  // (0 past J)
        res = 0.0;
        auto row_sum = [&](const Real (&ev)[CPL]) {
            Real s0 = 0, s1 = 0;
#pragma unroll
            for (int q = 0; q < CPL; ++q) {
                if (q & 1) s1 = fma(ev[q], x[q], s1);
                else s0 = fma(ev[q], x[q], s0);
            }
            return s0 + s1;
        };
        // the cells of one row step of this lane: 16 bytes at a time, then word by word
        auto load_row = [&](const Real* trow, Real (&ev)[CPL], bool whole) {
#pragma unroll
            for (int c = 0; c < NV; ++c) {
                float4 y = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                if (whole || (c * LPR + sub) * 4 < Jp) y = *reinterpret_cast<const float4*>(trow + (c * LPR + sub) * 4);
                ev[4 * c] = y.x; ev[4 * c + 1] = y.y; ev[4 * c + 2] = y.z; ev[4 * c + 3] = y.w;
            }
#pragma unroll
            for (int q = 4 * NV; q < CPL; ++q) ev[q] = trow[q * LPR + sub];
        };
        // N row steps at once, without a branch, so that the chains of their
        // sums overlap: row sums, column partials and residual terms (rows past
        // the range have a_i = 0 and a sum of 1)
        auto finish = [&](int st, const auto& ev) {
            constexpr int N = std::extent<std::remove_reference_t<decltype(ev)>>::value;
            double d[N], Sn[N];
            [[maybe_unused]] double Sp[N];
#pragma unroll
            for (int u = 0; u < N; ++u) d[u] = (double)row_sum(ev[u]);
            group_sums<LPR>(d);
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const int lr = ((st + u) * WAVES + w) * R + rg;
                const double ai = al[lr], Rr = D ? Rl[lr] : 0.0, So = Sl[lr];
                const double S = D ? Rr + d[u] : (lr < nrows ? d[u] : 1.0);
                Real wq;
                if constexpr (F64) {
                    wq = ai / S;
                    res += ai * (fabs(S - So) / So);
                    Sp[u] = So;
                } else {
                    wq = (float)(ai * asc) * __builtin_amdgcn_rcpf((float)S);
                    if constexpr (D) wq *= -(float)d[u] * __builtin_amdgcn_rcpf((float)Rr);
                    res += ai * (fabs(S - So) * (double)__builtin_amdgcn_rcpf((float)So));
                }
#pragma unroll
                for (int q = 0; q < CPL; ++q) acc[q] = fma(ev[u][q], wq, acc[q]);
                Sn[u] = S;
            }
            if (sub == 0) {
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    Sl[((st + u) * WAVES + w) * R + rg] = Sn[u];
                    if constexpr (F64) Rl[((st + u) * WAVES + w) * R + rg] = Sp[u];  // (of iterate k - 1)
                }
            }
        };
        if constexpr (GM) {
            constexpr int PD = 4;  // steps in flight
            float ev[PD][1][CPL];
            auto fetch = [&](int p, int st) {
                const int lr = (st * WAVES + w) * R + rg;
                load_row(tile + (size_t)(lr < nrows ? lr : 0) * Jp, ev[p][0], false);
            };
#pragma unroll
            for (int p = 0; p < PD; ++p) fetch(p, p);  // (steps past the last read row 0 of the block)
            for (int st = 0; st < steps; st += PD) {
#pragma unroll
                for (int p = 0; p < PD; ++p) {
                    if (st + p < steps) {  // uniform
                        finish(st + p, ev[p]);
                        if (st + p + PD < steps) fetch(p, st + p + PD);
                    }
                }
            }
        } else {
            auto step = [&](int st, auto nu) {
                constexpr int N = decltype(nu)::value;
                Real ev[N][CPL];
#pragma unroll
                for (int u = 0; u < N; ++u)
                    load_row(tile + (size_t)(((st + u) * WAVES + w) * R + rg) * Jp, ev[u], true);
                finish(st, ev);
            };
            int st = 0;
            for (; st + U <= steps; st += U) step(st, std::integral_constant<int, U>{});
            if constexpr (U > 2)
                for (; st + 2 <= steps; st += 2) step(st, std::integral_constant<int, 2>{});
            if constexpr (U > 1)
                for (; st < steps; ++st) step(st, std::integral_constant<int, 1>{});
        }
        if (sub != 0) res = 0.0;  // (every lane of a row holds its term)
    };

    // The workgroup's column partials: the row groups of a wave (lanes
    // sub + LPR r share columns), then the waves in FP64; calls out(c, sum)
    // for this thread's columns. The residual's wave sums go to wres.
    auto fold = [&](auto& ac, auto&& col, auto&& out) {
        using E = std::decay_t<decltype(ac[0])>;
        E* rb = reinterpret_cast<E*>(red);
        if constexpr (LPR <= 32) {
#pragma unroll
            for (int q = 0; q < CPL; ++q) ac[q] = xor32_sum(ac[q]);
        }
        if constexpr (LPR == 16) {
#pragma unroll
            for (int q = 0; q < CPL; ++q) ac[q] = xor16_sum(ac[q]);
        }
        const double rw = wave_sum(res);
        if (lane == 0) wres[w] = rw;
        constexpr int NW = WAVES * 4 / ((LPR == 64 ? 2 : 1) * (int)sizeof(E));  // waves per round
        constexpr int NC = (CPL * LPR + T - 1) / T;  // columns per thread
        double t[NC];
#pragma unroll
        for (int u = 0; u < NC; ++u) t[u] = 0.0;
#pragma unroll
        for (int w0 = 0; w0 < WAVES; w0 += NW) {
            if (w0 > 0) __syncthreads();  // the previous round's sums are taken
            if (w >= w0 && w < w0 + NW && rg == 0) {
#pragma unroll
                for (int q = 0; q < CPL; ++q) rb[(w - w0) * WD + col(q)] = ac[q];
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NC; ++u) {
                const int c = u * T + tid;
                if (c < J) {
#pragma unroll
                    for (int q = 0; q < NW; ++q) t[u] += (double)rb[q * WD + c];
                }
            }
        }
#pragma unroll
        for (int u = 0; u < NC; ++u) {
            const int c = u * T + tid;
            if (c < J) out(c, t[u]);
        }
    };

    // The partials of column block o tagged kt from every workgroup, summed in
    // a fixed order: thread t takes column t % 8 of producers t / 8 + (T / 8) u
    // (whole lines per wave). Leaves the waves' sums in ored, behind a barrier;
    // false (in every thread) if a wait gave up.
    auto collect = [&](int o, int kt) -> bool {
        constexpr int PB = T / kColBlock, NU = kMaxCoopGroups / PB;  // producers per round, rounds
        const double* pk = part + (size_t)(kt & 1) * nb * X.Jp;
        const int c = tid & (kColBlock - 1), pb = tid / kColBlock;
        const int j = o * kColBlock + c;
        const bool cv = j < J;
        double x[NU];
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int pr = pb + PB * u;
            x[u] = (cv && pr < nb) ? get_agent(pk + (size_t)pr * X.Jp + j) : tag_value(0.0, kt);
        }
        bool fail = false;
        int spin = 0;
        for (;;) {
            bool pend = false;
#pragma unroll
            for (int u = 0; u < NU; ++u) pend |= !has_tag(x[u], kt);
            if (!__any(pend)) break;
            if ((++spin & 31) == 0 && (get_agent(abort_word) != 0 || spin > A.max_spin)) {
                put_agent(abort_word, (uint64_t)1);
                fail = true;
                break;
            }
            poll_pause(spin);
#pragma unroll
            for (int u = 0; u < NU; ++u)
                if (!has_tag(x[u], kt)) x[u] = get_agent(pk + (size_t)(pb + PB * u) * X.Jp + j);
        }
        // (tag bits of the partials stay in the sum: a relative change below 2^-50)
        double s = x[0];
#pragma unroll
        for (int u = 1; u < NU; ++u) s += x[u];
        s += dpp_d<0x128>(s);  // lanes of one wave with the same column (producers
        s = xor16_sum(s);      // pb .. pb + 7 of this wave): lane l ^ 8, l ^ 16, l ^ 32
        s = xor32_sum(s);
        if (lane < kColBlock) ored[w][lane] = s;
        if (fail && lane == 0) atomicOr(&s_flag[kt & 1], 1);
        __syncthreads();
        return !(s_flag[kt & 1] & 1);
    };
    auto collected = [&](int cc) {
        double csum = 0.0;
#pragma unroll
        for (int q = 0; q < WAVES; ++q) csum += ored[q][cc];
        return csum;
    };

    __syncthreads();
    bool ok = true, bad = false, skip = false;
    [[maybe_unused]] bool prev = false;  // FP64: iterate k - 1 is the returned one
    for (;;) {
        ++k;
        const int P = k & 1;
        // (made opaque here: else the per-column masks and addresses of every
        // phase are computed once before the loop and kept, over a hundred
        // scalar and vector registers that then spill)
        asm volatile("" : "+v"(tid), "+v"(lane), "+v"(sub), "+v"(rg), "+s"(J), "+s"(Jp), "+s"(ncl));
        const bool fine = kind == kItRefDelta || kind == kItDelta;  // v - 1 is what the next delta sums need
        const bool hold = k - k0 == A.hold_iter;
        // v_j of this workgroup from the exchange (or, alone, from its own
        // sums), with the flags that choose the next iteration's kind
        int flag = 0;
        auto take_v = [&](int j, double v) {
            if constexpr (F64) vp[j] = vl[j];
            vl[j] = v;
            xl[j] = (Real)(fine ? v - 1.0 : v);
            if (!(v > 0.0) || !isfinite(v)) flag |= 2;
            if (fine ? !(fabs(v - 1.0) <= kDeltaMax) : !(v >= 1.0 / kScaleMax && v <= kScaleMax)) flag |= 4;
        };
        // column update v_j = b_j / sum_i E_ij a_i / S_i of owned column slot e
        auto col_v = [&](int e, double sum) {
            if (kind == kItDelta) sum += cl[e];
            return bl[e] / sum;
        };
        double* prow = part + ((size_t)P * nb + blk) * X.Jp;
        auto out = [&](int c, double t) {
            if (nb == 1) {
                take_v(c, col_v(c, t));
                if (kind == kItRefDelta) cl[c] = t;
            } else {
                put_agent(prow + c, tag_value(t, k));
            }
        };

        // ---- 1. row update and the workgroup's column partials
        if (kind == kItRef || kind == kItRefDelta) {
            double ac[CPL];
            take_reference(ac);
            fold(ac, col_ref, out);
        } else {
            Real ac[CPL];
#pragma unroll
            for (int q = 0; q < CPL; ++q) ac[q] = 0;
            if constexpr (F64) {
                rows(std::false_type{}, ac);
            } else {
                if (kind == kItDelta) rows(std::true_type{}, ac);
                else rows(std::false_type{}, ac);
            }
            fold(ac, col_it, out);
        }
        if (tid == T - 1 && nb > 1) {
            double r = 0.0;
#pragma unroll
            for (int q = 0; q < WAVES; ++q) r += wres[q];
            put_agent(rpart + (size_t)P * nb + blk, tag_value(r, k));
        }

        bool fail = false;
        if (blk == dblk && w == WAVES - 1) {  // residual of iterate k - 1 and the stop rule
            double x[4] = {0.0, 0.0, 0.0, 0.0};
            if (nb == 1) {
                if (lane < WAVES) x[0] = wres[lane];
                fail = hold;
            } else if (!poll_tagged(rpart + (size_t)P * nb, 1, nb, k, x, abort_word, A.max_spin)) {
                fail = true;
            }
            if (!fail) {
                double r = 0.0;
#pragma unroll
                for (int u = 0; u < 4; ++u) r += x[u];
                r = wave_sum(r);
                int code = 0;
                if constexpr (F64) {
                    if (lane == 0) {
                        bookkeep(&cs, r, kModeExact, 0.0);
                        code = cs.stop | cs.done ? kDecStop : 0;
                        if (cs.done && !cs.numeric_bad) code |= kDecPrev;
                    }
                } else if (lane == 0) {
                    code = bookkeep_coop(&cs, r, kind, A.stall_below, A.polish, r_ref, k_ref);
                }
                if (lane == 0 && k - k0 >= A.cap && !(code & kDecStop)) code = kDecStop | kDecSkip;
                // (every workgroup's verdict on its rows of the matrix preceded its
                // first partials)
                if (lane == 0 && k == k0 + 1 && (A.validate || A.batch)) {
                    cs.input_bad |= __hip_atomic_load(&ctl->input_bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    cs.numeric_bad |= __hip_atomic_load(&ctl->numeric_bad, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if (cs.input_bad | cs.numeric_bad) code = kDecStop | kDecSkip;
                }
                code = __shfl(code, 0, kWave);
                if (nb == 1) {
                    if (lane == 0) s_dec = (uint32_t)code;
                } else if (lane < kReplicas) {
                    put_agent(dec + ((size_t)P * kReplicas + lane) * 8, ((uint64_t)k << 3) | (uint64_t)code);
                }
            }
        }

        // ---- 2. column update of the owned blocks of kColBlock columns, v
        //      published in every replica
        for (int o = blk, oi = 0; nb > 1 && o * kColBlock < J; o += nb, ++oi) {
            if (oi > 0) __syncthreads();  // ored still holds the previous block
            if (!collect(o, k)) { fail = true; break; }
            if (tid < kColBlock * kReplicas) {
                const int cc = tid & (kColBlock - 1), r = tid >> 3;
                const int jj = o * kColBlock + cc;
                if (jj < J && !hold) {
                    const double csum = collected(cc);
                    const int e = oi * kColBlock + cc;
                    put_agent(gx + ((size_t)P * kReplicas + r) * X.Gs + jj, tag_value(col_v(e, csum), k));
                    if (kind == kItRefDelta && r == 0) cl[e] = csum;
                }
            }
        }

        // ---- 3. v and the decision, from this workgroup's replica: every wave
        //      polls 64 columns at a time (one load per lane in flight: short
        //      poll rounds), the last wave also the decision
        if (!fail && nb > 1) {
            const double* vx = gx + ((size_t)P * kReplicas + rep) * X.Gs;
            for (int j0 = w * kWave; j0 < J; j0 += WAVES * kWave) {
                double x[1];
                if (!poll_tagged(vx + j0, 1, min(J - j0, kWave), k, x, abort_word, A.max_spin)) {
                    fail = true;
                    break;
                }
                if (j0 + lane < J) take_v(j0 + lane, x[0]);
            }
        }
        if (w == WAVES - 1 && lane == 0 && !fail && nb > 1) {
            const uint64_t* dp = dec + ((size_t)P * kReplicas + rep) * 8;
            uint64_t d = get_agent(dp);
            int spin = 0;
            while ((d >> 3) != (uint64_t)k) {
                if ((++spin & 31) == 0 && (get_agent(abort_word) != 0 || spin > A.max_spin)) {
                    put_agent(abort_word, (uint64_t)1);
                    fail = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
                d = get_agent(dp);
            }
            s_dec = (uint32_t)(d & 7);
        }
        if (fail) flag |= 1;
        if (__any(flag)) {  // (rare; one LDS atomic per wave, not one per lane)
            const int f = (__any(flag & 1) ? 1 : 0) | (__any(flag & 2) ? 2 : 0) | (__any(flag & 4) ? 4 : 0);
            if (lane == 0) atomicOr(&s_flag[P], f);
        }
        __syncthreads();
        const int fl = __builtin_amdgcn_readfirstlane(s_flag[P]);
        const uint32_t code = __builtin_amdgcn_readfirstlane(s_dec);
        // (the other parity's flags were last read before this iteration's
        // barriers, and are next set after the next iteration's first)
        if (tid == 0) s_flag[P ^ 1] = 0;
        if (fl & 1) { ok = false; break; }
        has_prev = 1;
        if ((code & kDecStop) || (fl & 2)) {
            skip = (code & kDecSkip) != 0;
            bad = (fl & 2) != 0;
            prev = F64 && !bad && (code & kDecPrev);
            break;
        }
        if constexpr (F64) kind = (fl & 4) ? kItRef : kItPlain;
        else if (fine) kind = ((code & kDecRefDelta) || (fl & 4)) ? kItRefDelta : kItDelta;
        else kind = (code & kDecRefDelta) ? kItRefDelta : (fl & 4) ? kItRef : kItPlain;
    }

    if (ok && !bad) {
        // ---- the returned iterate k: f of the rows, g (workgroup 0)
        J = __builtin_amdgcn_readfirstlane(J);
        Jp = __builtin_amdgcn_readfirstlane(Jp);
        ncl = __builtin_amdgcn_readfirstlane(ncl);
        asm volatile("" : "+v"(tid), "+v"(lane), "+v"(sub), "+v"(rg), "+s"(J), "+s"(Jp), "+s"(ncl));
        src.stage(reinterpret_cast<double*>(red), J);
        const int kr = F64 && prev ? k - 1 : k;  // the returned iterate
        double* fo = (kr & 1) ? A.f[1] : A.f[0];
        for (int lr = tid; lr < nrows; lr += T) {
            double fi;
            if (F64 && prev && kind == kItRef) fi = fo[r0 + lr];  // (kept when the reference was taken)
            else fi = eps * (log(al[lr]) - kLn2 * (ml[lr] + log2(F64 && prev ? Rl[lr] : Sl[lr])));
            ml[lr] = fi;
            fo[r0 + lr] = fi;
        }
        double* go = (kr & 1) ? A.g[1] : A.g[0];
        for (int j = tid; j < J; j += T) {
            gl[j] += eps * log(F64 && prev ? vp[j] : vl[j]);
            if (blk == 0) go[j] = gl[j];
        }
        __syncthreads();
    }
    if (ok && !bad && !skip) {
        // ---- its exact check: FP64 sums over pi_ij = exp((f_i + g_j - C_ij) / eps) from
        //      the cost (read or regenerated once more), the plan and the RRH loads
        //      sum_i C_ij pi_ij where they are asked for. In this launch it costs
        //      one pass and two hops of the exchange; as launches of its own it
        //      took four more (combine, check, two folds).
        const double* stage = reinterpret_cast<const double*>(red);
        constexpr bool kLoads = !LEAN && CPL <= kLoadsCpl;
        const bool with_loads = kLoads && A.loads != nullptr;
        double ac[CPL], acl[kLoads ? CPL : 1];
#pragma unroll
        for (int q = 0; q < CPL; ++q) ac[q] = acl[kLoads ? q : 0] = 0.0;
        double rowres = 0.0, cost = 0.0, ent = 0.0, mass = 0.0, fa = 0.0;
        // (a row's loads one step ahead, as the references take them)
        constexpr bool kAhead = Src::kCheap && CPL * sizeof(typename Src::template Raw<1>) <= (LEAN ? 32 : 104);
        constexpr int G = Src::kTag == 5 ? 1 : LEAN && CPL > 8 ? 2 : LEAN || CPL > 13 ? (CPL < 4 ? CPL : 4) : CPL;  // cells at a time (their plan values held until stored)
        typename Src::template Raw<1> nraw[kAhead ? CPL : 1];
        [[maybe_unused]] auto fetch = [&](int st) {
            const int lr = (st * WAVES + w) * R + rg;
            auto row = src.row(r0 + (lr < nrows ? lr : 0));
#pragma unroll
            for (int q = 0; q < CPL; ++q)
                if (q < ncl) nraw[kAhead ? q : 0] = src.template load<1>(row, q * LPR + sub, J);
        };
        if constexpr (kAhead) fetch(0);
        for (int st = 0; st < steps; ++st) {
            const int lr = (st * WAVES + w) * R + rg;
            const bool vrow = lr < nrows;
            const int64_t i = r0 + (vrow ? lr : 0);
            auto row = src.row(i);
            const double fk = vrow ? ml[lr] * kk : 0.0;
            double rs = 0.0;
            // without a branch, so that the cells' exponentials overlap; a cell
            // outside the instance, or of infinite cost, adds zeros
            double pl[G];
            auto cell = [&](int q, const typename Src::template Raw<1>& raw) {
                const int j = q * LPR + sub;
                const bool in = q < ncl && j < J && vrow;
                pl[q % G] = 0.0;
                if (Src::kTag == 5 && !in) return;  // (the geometry functor has no registers for several cells)
                double c = 0.0;
                if (in) c = src.template cost<true, 1>(row, raw, 0, i, j, stage);
                // log2 pi_ij (rounded as in the plan kernel)
                const double t = in ? fmax(fk + fma(c, -kk, gl[j] * kk), -2000.0) : -2000.0;
                const double p = exp2_tab(t, e2tab);
                c = p > 0.0 ? c : 0.0;
                rs += p;
                cost = fma(c, p, cost);
                ent = fma(p, t * kLn2 - 1.0, ent);
                if constexpr (kLoads) acl[q] = fma(c, p, acl[q]);
                ac[q] += p;
                pl[q % G] = p;
            };
            auto store = [&](int q0) {
                if (!A.plan_out) return;
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const int q = q0 + u, j = q * LPR + sub;
                    if (q < CPL && q < ncl && j < J && vrow) {
                        if (A.plan_f64) reinterpret_cast<double*>(A.plan_out)[i * J + j] = pl[u];
                        else reinterpret_cast<float*>(A.plan_out)[i * J + j] = (float)pl[u];
                    }
                }
            };
            typename Src::template Raw<1> raw[kAhead ? CPL : G];
            if constexpr (kAhead) {
#pragma unroll
                for (int q = 0; q < CPL; ++q) raw[q] = nraw[q];
                if (st + 1 < steps) fetch(st + 1);
            }
#pragma unroll
            for (int q0 = 0; q0 < CPL; q0 += G) {
                if constexpr (!kAhead) {
#pragma unroll
                    for (int u = 0; u < G; ++u)
                        if (q0 + u < CPL && q0 + u < ncl) raw[u] = src.template load<1>(row, (q0 + u) * LPR + sub, J);
                }
#pragma unroll
                for (int u = 0; u < G; ++u)
                    if (q0 + u < CPL) cell(q0 + u, raw[kAhead ? (q0 + u < CPL ? q0 + u : 0) : u]);
                store(q0);
                if constexpr (G < CPL) __builtin_amdgcn_sched_barrier(0);
            }
            rs = group_sum<LPR>(rs);
            if (sub == 0 && vrow) {
                rowres += fabs(rs - al[lr]);
                mass += rs;
                fa += ml[lr] * al[lr];
            }
        }
        {
            const double v[5] = {wave_sum(rowres), wave_sum(cost), wave_sum(ent), wave_sum(mass), wave_sum(fa)};
            if (lane == 0)
                for (int q = 0; q < 5; ++q) wst[w][q] = v[q];
        }
        __syncthreads();  // (the fold reuses the staged source data's LDS)
        // partials tagged k + 1 (loads: k + 2; the last reader of either parity's
        // slots was done with them before iteration k's v arrived), scalars
        // and column owners' results
        const int k1 = k + 1;
        double* slots = A.xch + X.fin;
        constexpr int kOwnSlots = 5 * kMaxCoopGroups;
        auto publish = [&](double (&v)[CPL], int kt) {
            double* prow = part + ((size_t)(kt & 1) * nb + blk) * X.Jp;
            fold(v, col_ref, [&](int c, double t) { put_agent(prow + c, tag_value(t, kt)); });
        };
        publish(ac, k1);
        if (tid < 5) {
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < WAVES; ++q) t += wst[q][tid];
            put_agent(slots + blk * 5 + tid, tag_value(t, 1));
        }
        if constexpr (kLoads) {
            if (with_loads) {
                __syncthreads();  // the fold buffer is still read
                publish(acl, k1 + 1);
            }
        }
        for (int o = blk; ok && o * kColBlock < J; o += nb) {
            __syncthreads();
            ok = collect(o, k1);
            if (!ok) break;
            if (tid < kColBlock) {
                const int jj = o * kColBlock + tid;
                double cres = 0.0, gb = 0.0;
                if (jj < J) {
                    const double bj = A.b[jj];
                    cres = fabs(collected(tid) - bj);
                    gb = gl[jj] * bj;
                }
                cres += dpp_d<0xB1>(cres);  // the 8 columns of the block
                cres += dpp_d<0x4E>(cres);
                cres += dpp_d<0x141>(cres);
                gb += dpp_d<0xB1>(gb);
                gb += dpp_d<0x4E>(gb);
                gb += dpp_d<0x141>(gb);
                if (tid == 0) {
                    put_agent(slots + kOwnSlots + 2 * o, tag_value(cres, 1));
                    put_agent(slots + kOwnSlots + 2 * o + 1, tag_value(gb, 1));
                }
            }
            if (with_loads) {
                __syncthreads();
                ok = collect(o, k1 + 1);
                if (!ok) break;
                if (tid < kColBlock && o * kColBlock + tid < J) A.loads[o * kColBlock + tid] = collected(tid);
            }
        }
        if (blk == dblk && ok) {
            const int nblk = (J + kColBlock - 1) / kColBlock;
            double x[7];
            auto at = [&](int u, bool& live) {
                live = u < 5 ? tid < nb : tid < nblk;
                return u < 5 ? slots + tid * 5 + u : slots + kOwnSlots + 2 * tid + (u - 5);
            };
            static_assert(T >= kMaxCoopGroups, "one thread per workgroup and per column block");
#pragma unroll
            for (int u = 0; u < 7; ++u) {
                bool live;
                const double* p = at(u, live);
                x[u] = live ? get_agent(p) : tag_value(0.0, 1);
            }
            int spin = 0;
            bool fail = false;
            for (;;) {
                bool pend = false;
#pragma unroll
                for (int u = 0; u < 7; ++u) pend |= !has_tag(x[u], 1);
                if (!__any(pend)) break;
                if ((++spin & 31) == 0 && (get_agent(abort_word) != 0 || spin > A.max_spin)) {
                    put_agent(abort_word, (uint64_t)1);
                    fail = true;
                    break;
                }
                __builtin_amdgcn_s_sleep(1);
#pragma unroll
                for (int u = 0; u < 7; ++u) {
                    bool live;
                    const double* p = at(u, live);
                    if (!has_tag(x[u], 1)) x[u] = get_agent(p);
                }
            }
            __syncthreads();  // wst and the flags are reused
            if (fail && lane == 0) atomicOr(&s_flag[k1 & 1], 1);
#pragma unroll
            for (int u = 0; u < 7; ++u) {
                const double t = wave_sum(x[u]);
                if (lane == 0) wst[w][u] = t;
            }
            __syncthreads();
            ok = !(s_flag[k1 & 1] & 1);
            if (ok && tid == 0) {
                double t[7];
                for (int u = 0; u < 7; ++u) {
                    t[u] = 0.0;
                    for (int q = 0; q < WAVES; ++q) t[u] += wst[q][u];
                }
                cs.chk_row_res = t[0];
                cs.chk_col_res = t[5];
                cs.chk_violation = (t[0] + t[5]) / cs.mass;
                cs.chk_objective = t[1];
                cs.chk_reg_objective = t[1] + eps * t[2];
                cs.chk_mass = t[3];
                cs.chk_dual = t[4] + t[6] - eps * t[3];
            }
        }
    }
    if (blk == dblk && tid == 0) {
        if (bad || !ok) {
            cs.numeric_bad |= bad ? 1 : 0;
            cs.sync_fail = ok ? 0 : 1;
            cs.done = 1;
            cs.stop = 1;
            cs.result_iter = cs.iter;
        }
        if (F64 && prev && ok) {
            cs.iter = k - 1;
            cs.done = 0;
        }
        if (skip && (cs.input_bad | cs.numeric_bad)) {
            cs.done = cs.stop = 1;
            cs.result_iter = cs.iter;
        }
        if (A.batch) {
            // done, or further FP64 sweeps until an iterate meets tol; at the
            // launch's cap further iterations of the phase
            const bool fin = cs.done || (!skip && (cs.chk_violation < cs.tol || cs.iter >= cs.max_iter ||
                                                   !isfinite(cs.chk_violation)));
            cs.phase = fin ? kPhDone : skip ? kPhFast : kPhExact;
            cs.done = fin ? 1 : 0;
            cs.stop = 0;
            cs.result_iter = cs.check_iter = cs.iter;
        }
        *ctl = cs;
    }
}

template <class Src, int CPL, int LPR, int WAVES, bool GM, bool F64 = false>
__global__ __launch_bounds__(WAVES * kWave) void k_persist(PersistArgs A, Src src) {
    __shared__ PersistShared ps;
    persist_run<Src, CPL, LPR, WAVES, GM, false, F64>(A, src, (int)gridDim.x, (int)blockIdx.x, ps);
}

// ------------------------------------------------------------ solve set-up --
// Checks the marginals (positive and finite, equal masses), copies them into
// the solver's buffers, zeroes g for a cold start and writes the solve
// constants and the initial control block, so that a solve needs no host
// round trip before its first sweep. The masses are compensated sums
// (per-thread Neumaier sums in a fixed strided order, then two-sum merges in
// a fixed order across lanes, waves and workgroups). One workgroup does it all
// for up to kInitSingle devices; above, the devices are split over workgroups
// whose sums k_solve_init_fin merges: the compensated sums of one CU take
// 11 us at I = 5000, 17 at 20000 and 76 at 200000, split 17, 19 and 25 (both
// launches start cold).
constexpr int64_t kInitSingle = 32768;
constexpr int kInitGroups = 64;  // workgroups of the device sums at most
struct InitArgs {
    int64_t I;
    int J;
    int cold;
    const double* a_src;  // may equal a
    const double* b_src;  // may equal b
    double* a;
    double* b;
    double* g0;
    SolveParams* prm_out;
    Ctl* ctl_out;
    SolveParams prm;
    Ctl ctl;
    double* xch;  // exchange block zeroed by the workgroups past the first (nx doubles), or nullptr
    int64_t nx;
    int groups;    // workgroups of the device sums (1: no second launch)
    double* part;  // 3 per such workgroup: sum, its error, invalid entries
};

__device__ __forceinline__ void two_sum_add(double& s, double& c, double x) {
    const double t = s + x;
    c += (fabs(s) >= fabs(x)) ? (s - t) + x : (x - t) + s;
    s = t;
}

// A lane's compensated sum merged with its partner's, by DPP lane moves within
// 16 lanes and row swaps beyond (as a tree through LDS with ten
// barriers: 10.4 us at I = 100, now 8.2).
template <int CTRL>
__device__ __forceinline__ void two_sum_dpp(double& s, double& c) {
    const double s2 = dpp_d<CTRL>(s), c2 = dpp_d<CTRL>(c);
    two_sum_add(s, c, s2);
    c += c2;
}
__device__ __forceinline__ void two_sum_row16(double& s, double& c) {
    two_sum_dpp<0xB1>(s, c);
    two_sum_dpp<0x4E>(s, c);
    two_sum_dpp<0x141>(s, c);
    two_sum_dpp<0x140>(s, c);
}
// lanes 0, 16, 32, 48 hold their rows' sums; the same in every lane
__device__ __forceinline__ void two_sum_rows(double& s, double& c) {
    const double s0 = readlane_d(s, 0), c0 = readlane_d(c, 0);
    double t = s0, e = c0;
#pragma unroll
    for (int q = 1; q < 4; ++q) {
        two_sum_add(t, e, readlane_d(s, 16 * q));
        e += readlane_d(c, 16 * q);
    }
    s = t;
    c = e;
}

// Thread 0 of the workgroup gets the merged sum of all its threads (sums of b
// and flags likewise); ends behind a barrier.
__device__ __forceinline__ void init_merge(double (&sum)[2], double (&err)[2], int& bad) {
    __shared__ double ws[2][16], wc[2][16];  // per-wave sums and their errors
    __shared__ int s_bad;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (threadIdx.x == 0) s_bad = 0;
    __syncthreads();
    if (bad) atomicOr(&s_bad, bad);
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        two_sum_row16(sum[u], err[u]);
        two_sum_rows(sum[u], err[u]);
    }
    if (lane == 0)
        for (int u = 0; u < 2; ++u) { ws[u][w] = sum[u]; wc[u][w] = err[u]; }
    __syncthreads();
    bad = s_bad;
    if (w == 0) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const bool in = lane < (int)(blockDim.x / kWave);
            sum[u] = in ? ws[u][lane & 15] : 0.0;
            err[u] = in ? wc[u][lane & 15] : 0.0;
            two_sum_row16(sum[u], err[u]);
        }
    }
}

// The RRHs' marginal (one workgroup).
__device__ __forceinline__ void init_rrhs(const InitArgs& A, double& sum, double& err, int& bad) {
    for (int j = threadIdx.x; j < A.J; j += blockDim.x) {
        const double v = A.b_src[j];
        if (!(v > 0.0) || !isfinite(v)) bad |= 2;
        if (A.b != A.b_src) A.b[j] = v;
        two_sum_add(sum, err, v);
        if (A.cold) A.g0[j] = 0.0;
    }
}

// Thread 0: the solve constants and the control block.
__device__ __forceinline__ void init_ctl(const InitArgs& A, double ma, double mb, int flags) {
    if (fabs(ma - mb) > 1e-12 * ma) flags |= 4;
    *A.prm_out = A.prm;
    Ctl c = A.ctl;
    c.mass = ma;
    c.mass_b = mb;
    c.input_bad = flags;
    if (flags) {
        c.done = 1;
        c.stop = 1;
    }
    *A.ctl_out = c;
}

// Workgroups below A.groups sum the devices' marginal. Those past them zero the
// cooperative exchange block, for a cooperative launch that starts from
// iteration 0: a zero slot carries tag 0, which neither of the launch's first
// two iterations (1 and 2, one per buffer parity) waits for, and zero decision
// and abort words; so the launch needs no clearing pass of its own.
static __global__ __launch_bounds__(1024) void k_solve_init(InitArgs A) {
    if ((int)blockIdx.x >= A.groups) {
        const size_t stride = (size_t)(gridDim.x - A.groups) * blockDim.x;
        for (size_t q = (size_t)(blockIdx.x - A.groups) * blockDim.x + threadIdx.x; q < (size_t)A.nx; q += stride)
            A.xch[q] = 0.0;
        return;
    }
    double sum[2] = {0.0, 0.0}, err[2] = {0.0, 0.0};
    int bad = 0;
    constexpr int N = 8;  // loads in flight per thread, then their terms in index order
    const int64_t step = (int64_t)A.groups * blockDim.x;
    for (int64_t i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i0 < A.I; i0 += N * step) {
        double v[N];
#pragma unroll
        for (int u = 0; u < N; ++u) v[u] = i0 + u * step < A.I ? A.a_src[i0 + u * step] : 1.0;
#pragma unroll
        for (int u = 0; u < N; ++u) {
            const int64_t i = i0 + u * step;
            if (i < A.I) {
                if (!(v[u] > 0.0) || !isfinite(v[u])) bad |= 1;
                if (A.a != A.a_src) A.a[i] = v[u];
                two_sum_add(sum[0], err[0], v[u]);
            }
        }
    }
    if (A.groups == 1) init_rrhs(A, sum[1], err[1], bad);
    init_merge(sum, err, bad);
    if (threadIdx.x != 0) return;
    if (A.groups == 1) {
        init_ctl(A, sum[0] + err[0], sum[1] + err[1], bad);
    } else {
        double* p = A.part + 3 * blockIdx.x;
        p[0] = sum[0];
        p[1] = err[0];
        p[2] = (double)bad;
    }
}

// The second launch for more than kInitSingle devices: merges the workgroups'
// sums, sums the RRHs' marginal and writes the control block.
static __global__ __launch_bounds__(256) void k_solve_init_fin(InitArgs A) {
    double sum[2] = {0.0, 0.0}, err[2] = {0.0, 0.0};
    int bad = 0;
    if ((int)threadIdx.x < A.groups) {
        const double* p = A.part + 3 * threadIdx.x;
        sum[0] = p[0];
        err[0] = p[1];
        bad = (int)p[2];
    }
    init_rrhs(A, sum[1], err[1], bad);
    init_merge(sum, err, bad);
    if (threadIdx.x == 0) init_ctl(A, sum[0] + err[0], sum[1] + err[1], bad);
}

}  // namespace otk
