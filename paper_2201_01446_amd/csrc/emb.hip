// emb.hip -- fused environment matrix, tabulated embedding and R^T G
// contraction (forward), and its hand-written adjoint down to forces and the
// virial (backward), on gfx950.
//
// What is computed per atom i (paper Sec. 2.1, Eqs. 1-5; Sec. 3.2-3.4):
//   for every neighbor j with r = |r_ij| < rcut (the sel nearest at most):
//     s = w(r)/r, R_j = s (1, x/r, y/r, z/r)                      (Eq. 1)
//     G_j = f_theta(s): the M quintics of s's table interval      (Sec. 3.2)
//   T = desc_scale * sum_j R_j^T G_j   (4 x M), D = T<^T T (M< x M)  (Eq. 2)
// G is never stored (the kernel fusion of Sec. 3.3/3.4.1) and only the n_i
// real neighbors are visited (the redundancy removal of Sec. 3.4.2; with
// unnormalised R the padded rows would contribute exact zeros).
//
// Interval-moment form of the contraction.  In table interval theta the
// embedding is G_eta(s) = sum_e a[theta][eta][e] t^e with t = s - x_theta, so
// for the neighbors j whose s falls in theta
//   sum_j R_jk G_j,eta = sum_e a[theta][eta][e] M[theta][k][e],
//   M[theta][k][e] = sum_{j in theta} R_jk t_j^e      (4 x 6 moments).
// The neighbor list is sorted by distance and s decreases with r, so the
// neighbors of one interval form consecutive runs ("segments"; about 20 per
// atom in copper against about 178 neighbors).  The forward therefore forms
// 24 moments per neighbor and then 24 FMA per (segment, column), instead of
// 9 FMA per (neighbor, column).  The backward does the same on the other
// side: with dT = dE/dT (desc_scale applied),
//   dE/dR_jk  = sum_eta dT_k,eta G_j,eta = sum_e B[theta][k][e] t_j^e,
//   B[theta][k][e] = sum_eta dT_k,eta a[theta][eta][e],
//   dE/ds_j  += sum_k R_jk d/dt (sum_e B[theta][k][e] t^e) at t_j,
// so each segment costs 24 FMA per column once, and each neighbor two
// quintics per k.  Then g_ij = dE_i/dr_ij by the chain rule through Eq. 1:
// F_i = sum_j g_ij is written directly and W_i -= r_ij (x) g_ij; each g_ij is
// stored at its candidate slot, and a gather after the kernel subtracts from
// F_j the g_ij of every atom i that lists j (no atomics, a fixed order).
// Neighbors clamped to the table end form their own segment and get G' = 0.
// A run split because atoms moved since the list was sorted gives two
// segments of the same interval.  In the forward, such duplicates within a
// round of segments share one representative (the first of the round with
// that interval), which alone is contracted, with the sum of their moments.
// (The backward's B is computed by the segments' quads in parallel.  Rounds of
// 16 distinct intervals there, 20 to an atom of copper instead of 26 segments,
// gained 3 % in FP32 and lost 5 % in water and more in FP64, by their registers.)
//
// Work distribution (one 64-lane wavefront per atom, a block of its own:
// nothing is shared, and a block of four held its LDS until its slowest wave
// was done; neighbor data in LDS):
//   moments and B: quad q of the wave owns one segment per round; for the
//   moments lane l of the quad takes environment column k = l of every
//   neighbor of the segment, for B the four lanes split the 128 columns and
//   their partial sums meet in two DPP steps;
//   contraction into T: each lane owns columns eta = lane and lane + 64;
//   per-neighbor tail of the backward: each lane owns neighbors.

#include "dp_internal.h"
#include "emb_common.h"
#include "env.h"

#include <type_traits>

namespace dp {

namespace {

constexpr int kSegRound = 16;   // segments per round: one per quad of the wave

__device__ inline void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// f = sum_e a[e] t^e and its derivative.
template <typename real>
__device__ inline void horner2(const real *a, real t, real &f, real &fp)
{
    real p = a[5], q = a[5];
    p = fma(p, t, a[4]);
    q = fma(q, t, p);
    p = fma(p, t, a[3]);
    q = fma(q, t, p);
    p = fma(p, t, a[2]);
    q = fma(q, t, p);
    p = fma(p, t, a[1]);
    q = fma(q, t, p);
    f = fma(p, t, a[0]);
    fp = q;
}

__device__ inline float quad_sum(float v)
{
    v += dpp_f<0xB1>(v);   // quad_perm [1,0,3,2]
    v += dpp_f<0x4E>(v);   // quad_perm [2,3,0,1]
    return v;
}
__device__ inline double quad_sum(double v)
{
    v += dpp_d<0xB1>(v);
    v += dpp_d<0x4E>(v);
    return v;
}

// One DPP move of a float or a double.
template <int CTRL>
__device__ inline float dpp_any(float v) { return dpp_f<CTRL>(v); }
template <int CTRL>
__device__ inline double dpp_any(double v) { return dpp_d<CTRL>(v); }

// Representatives of the ns segments of a round starting at s0: lane u < ns
// returns the first segment v <= u of the round with the same table interval
// (the clamp bit aside); other lanes return themselves.
template <typename real>
__device__ inline int round_reps(const NbrLDS<real> &L, const int *seg, int s0, int ns, int lane)
{
    int thu = lane < ns ? (L.th[seg[s0 + lane]] & ~kOobBit) : -1;
    int rep = lane;
    // from the last to the first, so that the first match stays; past ns no
    // lane matches (-1) but those, which keep themselves below.  Lane reads:
    // as shuffles these were 32 dependent trips through the LDS a round (the
    // forward at 108,000 atoms 670 us against 600, FP32).
#pragma unroll
    for (int v = kSegRound - 2; v >= 0; v--) {
        const int thv = __builtin_amdgcn_readlane(thu, v);
        if (v < lane && thv == thu) rep = v;
    }
    return lane < ns ? rep : lane;
}

// Starts of the runs of equal interval in the neighbor list: seg[0..nseg-1],
// seg[nseg] = nn.  Returns nseg (uniform over the wave).  X > 0: a run longer
// than X is cut into pieces of X neighbors (and a last shorter one), which
// become segments of their own; nruns then receives the number of whole runs.
template <typename real, int X = 0>
__device__ __forceinline__ int find_segments(const NbrLDS<real> &L, int nn, int lane, int *seg, int *nruns = nullptr)
{
    int nseg = 0, runs = 0;
    int open = 0;   // start of the run that continues into the next chunk
    for (int base = 0; base < nn; base += 64) {
        int k = base + lane;
        bool head = k < nn && (k == 0 || L.th[k] != L.th[k - 1]);
        if (X > 0) {
            unsigned long long hm = __ballot(head);
            runs += __popcll(hm);
            unsigned long long upto = hm & ((2ull << lane) - 1ull);   // run heads at lanes <= lane
            int start = upto ? base + 63 - __builtin_clzll(upto) : open;
            head = head || (k < nn && (k - start) % X == 0);
            if (hm) open = base + 63 - __builtin_clzll(hm);
        }
        unsigned long long m = __ballot(head);
        if (head) seg[nseg + __popcll(m & ((1ull << lane) - 1ull))] = k;
        nseg += __popcll(m);
    }
    if (lane == 0) seg[nseg] = nn;
    if (nruns) *nruns = X > 0 ? runs : nseg;
    wave_sync();
    return nseg;
}

// Longest segment of the forward: its moments take one quad as many steps as
// the segment has neighbors, and a round waits for its longest segment, so
// long runs (a whole neighbor shell can share one table interval) are cut;
// the pieces share an interval, and the round's representatives merge them
// again before the contraction.
constexpr int kFwdMaxRun = 16;

constexpr int seg_bytes(int sel) { return ((sel + 1) * 4 + 15) / 16 * 16; }

// Per-wave LDS of the forward: neighbor arrays, the moments of one round of
// segments, segment starts; T (4 x M) for the descriptor at the end takes
// the slice's start once those are dead.
template <typename real>
constexpr int fwd_lds_bytes(int sel)
{
    constexpr int al = (int)sizeof(V4<real>);   // keeps every wave's slice aligned
    int b = nbr_lds_bytes<real>(sel, ENV_FWD) + kSegRound * 24 * (int)sizeof(real) + seg_bytes(sel);
    int t = 4 * kM * (int)sizeof(real);
    return ((b > t ? b : t) + al - 1) / al * al;
}

// Per-wave LDS of the backward: neighbor arrays, dT as (dT_0c, .., dT_3c)
// per column c, B of one round of segments, segment starts.
template <typename real>
constexpr int bwd_lds_bytes(int sel)
{
    constexpr int al = (int)sizeof(V4<real>);
    return (nbr_lds_bytes<real>(sel, ENV_BWD) + kM * (int)sizeof(V4<real>) + kSegRound * 24 * (int)sizeof(real) +
            seg_bytes(sel) + al - 1) / al * al;
}

// -------------------------------------------------------------- forward
// One round of the forward: the moments of the ns segments from s0 on, those of
// segments that share an interval added up in the first of them; returns which
// segments those are (bit u: segment s0 + u).
template <typename real>
__device__ __forceinline__ unsigned long long round_moments(const NbrLDS<real> &L, const int *seg, int s0, int ns, real *Ms, int lane)
{
    const int q = lane >> 2, ql = lane & 3;
    // moments of segment s0 + q: lane ql of the quad sums column k = ql
    // of R over the segment's neighbors, in list order
    if (q < ns) {
        real Mk[6] = {0, 0, 0, 0, 0, 0};
        int e1 = seg[s0 + q + 1];
        for (int k = seg[s0 + q]; k < e1; k++) {
            real t = L.t[k];
            real r = reinterpret_cast<const real *>(&L.R[k])[ql];
            real pw = 1;
#pragma unroll
            for (int e = 0; e < 6; e++) {
                Mk[e] = fma(r, pw, Mk[e]);
                pw *= t;
            }
        }
#pragma unroll
        for (int e = 0; e < 6; e++) Ms[q * 24 + ql * 6 + e] = Mk[e];
    }
    // segments of the round that share an interval: the representative
    // takes the others' moments (in segment order), and only it is contracted
    const int rep = round_reps(L, seg, s0, ns, lane);
    const unsigned long long reps = __ballot(lane < ns && rep == lane);
    if (reps != ((1ull << ns) - 1ull)) {
        wave_sync();
        real add[6] = {0, 0, 0, 0, 0, 0};
        for (unsigned long long rest = ((1ull << ns) - 1ull) & ~reps; rest; rest &= rest - 1) {
            const int u = __builtin_ctzll(rest);
            if (__builtin_amdgcn_readlane(rep, u) == q) {
#pragma unroll
                for (int e = 0; e < 6; e++) add[e] += Ms[u * 24 + ql * 6 + e];
            }
        }
        if (reps >> q & 1) {   // quad q holds a representative
#pragma unroll
            for (int e = 0; e < 6; e++) Ms[q * 24 + ql * 6 + e] += add[e];
        }
    }
    wave_sync();
    return reps;
}

// At 108,000 atoms 570 us (FP32) and 1,000 (FP64), 670 and 1,110 before the
// lane reads, the blocks of one wave and the coalesced table: the scan with
// the stores of records and T takes 40-45 %, the contraction 40 %; bound by
// the instructions of the wave (FP32) and by latency at the 3 waves a SIMD that
// its LDS allows (FP64).
template <typename real, typename TD>
__global__ void __launch_bounds__(64) k_emb_fwd(int natoms, EnvArgs A, const real *__restrict__ tab,
                                                 real sigma, real *__restrict__ T_out,
                                                 TD *__restrict__ D_out, int *__restrict__ nnei_out,
                                                 int *__restrict__ nseg_out)
{
    HIP_DYNAMIC_SHARED(uint4, smem_raw)   // 16-byte aligned
    char *base = reinterpret_cast<char *>(smem_raw);
    int lane = threadIdx.x;
    int i = xcd_item(blockIdx.x, gridDim.x);
    if (i >= natoms) return;
    NbrLDS<real> L = carve<real>(base, A.sel, ENV_FWD);
    char *p = base + nbr_lds_bytes<real>(A.sel, ENV_FWD);
    real *Tl = reinterpret_cast<real *>(base);   // 4 x M, after the rounds
    real *Ms = reinterpret_cast<real *>(p);   // kSegRound x 24
    p += kSegRound * 24 * sizeof(real);
    int *seg = reinterpret_cast<int *>(p);
    int n_in = 0, over = 0, oob = 0;
    const int nn = build_env<real, ENV_FWD>(i, A, L, lane, n_in, over, oob);
    wave_sync();
    int nruns = 0;
    int nseg = find_segments<real, kFwdMaxRun>(L, nn, lane, seg, &nruns);

    real T0[4] = {0, 0, 0, 0}, T1[4] = {0, 0, 0, 0};   // columns lane, lane + 64
    for (int s0 = 0; s0 < nseg; s0 += kSegRound) {
        int ns = min(kSegRound, nseg - s0);
        const unsigned long long reps = round_moments(L, seg, s0, ns, Ms, lane);
        // T[k][c] += sum_e a[theta][c][e] M[k][e], lanes over columns; the
        // coefficients of up to NG representatives are requested before any is used
        for (unsigned long long left = reps; left;) {
            constexpr int NG = 3;   // (four cost a wave a SIMD: 41,472 water atoms, FP32, 257 us against 245)
            int us[NG];
            int nu = 0;
#pragma unroll
            for (int u = 0; u < NG; u++) {
                us[u] = left ? __builtin_ctzll(left) : -1;
                if (left) {
                    left &= left - 1;
                    nu++;
                }
            }
            real a0[NG][6], a1[NG][6];
#pragma unroll
            for (int u = 0; u < NG; u++) {
                if (u < nu) {
                    int th = L.th[seg[s0 + us[u]]] & ~kOobBit;
                    coef_col(tab, th, lane, a0[u]);
                    coef_col(tab, th, lane + 64, a1[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < NG; u++) {
                if (u < nu) {
                    const real *m = Ms + us[u] * 24;
#pragma unroll
                    for (int k = 0; k < 4; k++)
#pragma unroll
                        for (int e = 0; e < 6; e++) {
                            real mv = m[k * 6 + e];
                            T0[k] = fma(mv, a0[u][e], T0[k]);
                            T1[k] = fma(mv, a1[u][e], T1[k]);
                        }
                }
            }
        }
        wave_sync();   // Ms is rewritten by the next round (and the arrays give way to T)
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        T0[k] *= sigma;
        T1[k] *= sigma;
        Tl[k * kM + lane] = T0[k];
        Tl[k * kM + lane + 64] = T1[k];
    }
    // T out by column: (T_0c, T_1c, T_2c, T_3c) for c < M, one vector store per column
    V4<real> *T4 = reinterpret_cast<V4<real> *>(T_out) + (long)i * kM;
    T4[lane] = V4<real>{T0[0], T0[1], T0[2], T0[3]};
    T4[lane + 64] = V4<real>{T1[0], T1[1], T1[2], T1[3]};
    wave_sync();
    // D[a][b] = sum_k T[k][a] T[k][b], a < M<: lane owns b = lane, lane + 64;
    // the row of the atom in the fitting net's operand (grouped by type).
    // No D_out: the first fitting layer forms D from T itself.
    const long drow = fit_row(A, i);
#pragma unroll 4
    for (int a = 0; a < (D_out ? kMlt : 0); a++) {
        real d0 = 0, d1 = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            real ta = Tl[k * kM + a];
            d0 = fma(ta, T0[k], d0);
            d1 = fma(ta, T1[k], d1);
        }
        store_op(D_out, drow, a * kM + lane, kDdim, (double)d0);
        store_op(D_out, drow, a * kM + lane + 64, kDdim, (double)d1);
    }
    // counters last: nothing in this kernel waits for these atomics
    if (nnei_out && lane == 0) nnei_out[i] = nn;
    if (nseg_out && lane == 0) nseg_out[i] = nruns;
    record_flags<real>(A, lane, n_in, over, oob);
}

// ------------------------------------------------------------- backward
// B[k][e] = sum_c dT[k][c] a[theta][c][e] for the ns segments of a round
// starting at s0, 2^lg lanes per segment (lg = 2 in a full round; the last
// round's segments get more): segment s0 + (lane >> lg), its lanes taking
// columns c = 2^lg m + (lane mod 2^lg), then summed over the group, whose
// first lane stores B at Bs[(lane >> lg) * 24].  FULL: lg = 2 known at
// compile time.
template <typename real, bool FULL>
__device__ __forceinline__ void round_B(const NbrLDS<real> &L, const int *seg, int s0, int ns, int lg,
                               const real *__restrict__ tab, const V4<real> *dTl, real *Bs, int lane)
{
    if (FULL) lg = 2;
    const int G = 1 << lg, q = lane >> lg, ql = lane & (G - 1);
    real B[4][6];
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
        for (int e = 0; e < 6; e++) B[k][e] = 0;
    if (q < ns) {
        int th = L.th[seg[s0 + q]] & ~kOobBit;
        // full rounds: in FP64 every coefficient load of the segment in flight
        // at once, in FP32 four (measured fastest for each); wider groups: two
        constexpr int kLoadsInFlight = !FULL ? 2 : sizeof(real) == 8 ? kM / 4 : 4;
#pragma unroll kLoadsInFlight
        for (int m = 0; m < (kM >> lg); m++) {
            int c = (m << lg) + ql;
            V4<real> d = dTl[c];
            real a[6];
            coef_col(tab, th, c, a);
#pragma unroll
            for (int e = 0; e < 6; e++) {
                B[0][e] = fma(d.x, a[e], B[0][e]);
                B[1][e] = fma(d.y, a[e], B[1][e]);
                B[2][e] = fma(d.z, a[e], B[2][e]);
                B[3][e] = fma(d.w, a[e], B[3][e]);
            }
        }
    }
#pragma unroll
    for (int k = 0; k < 4; k++)
#pragma unroll
        for (int e = 0; e < 6; e++) B[k][e] = quad_sum(B[k][e]);
    if (!FULL) {
        // the rest of the group (wave-uniform steps): within 8 and 16 lanes by
        // DPP mirrors, then across rows
        if (lg >= 3) {
#pragma unroll
            for (int k = 0; k < 4; k++)
#pragma unroll
                for (int e = 0; e < 6; e++) B[k][e] += dpp_any<0x141>(B[k][e]);
        }
        if (lg >= 4) {
#pragma unroll
            for (int k = 0; k < 4; k++)
#pragma unroll
                for (int e = 0; e < 6; e++) B[k][e] += dpp_any<0x140>(B[k][e]);
        }
        for (int off = 16; off < G; off <<= 1) {
#pragma unroll
            for (int k = 0; k < 4; k++)
#pragma unroll
                for (int e = 0; e < 6; e++) B[k][e] += __shfl_xor(B[k][e], off);
        }
    }
    if (q < ns && ql == 0) {
#pragma unroll
        for (int k = 0; k < 4; k++)
#pragma unroll
            for (int e = 0; e < 6; e++) Bs[q * 24 + k * 6 + e] = B[k][e];
    }
}

// dE/dT of one atom: load() starts its reads, finish() puts it, scaled, into
// the wave's LDS as (dT_0c, .., dT_3c) per column c.  The part dT2 of the
// columns c < M< that sums over all columns comes in nparts groups and is
// added here: 1, the whole; 8, groups of 16 columns; 32, groups of 4, four to
// one of 16.
template <typename real>
struct DTRegs {
    V4<real> d0, d1;
    real s;   // dT2[k = lane mod 4] of column lane / 4
    __device__ inline void load(int i, long n, int lane, const real *dT, const real *dTp, int nparts)
    {
        const V4<real> *D = reinterpret_cast<const V4<real> *>(dT) + (long)i * kM;
        d0 = D[lane];
        d1 = D[lane + 64];
        const real *p = dTp + (long)i * 64 + lane;
        if (nparts <= 8) {
            s = p[0];
            for (int w = 1; w < nparts; w++) s += p[(long)w * n * 64];
        } else {
            for (int w = 0; w < nparts; w += 4) {
                real t = p[(long)w * n * 64];
#pragma unroll
                for (int u = 1; u < 4; u++) t += p[(long)(w + u) * n * 64];
                s = w ? s + t : t;
            }
        }
    }
    __device__ inline void finish(int lane, real sigma, V4<real> *dTl)
    {
        const int c = (lane & 15) * 4;
        const real a0 = __shfl(s, c), a1 = __shfl(s, c + 1), a2 = __shfl(s, c + 2), a3 = __shfl(s, c + 3);
        if (lane < kMlt) d0 = V4<real>{d0.x + a0, d0.y + a1, d0.z + a2, d0.w + a3};
        dTl[lane] = V4<real>{sigma * d0.x, sigma * d0.y, sigma * d0.z, sigma * d0.w};
        dTl[lane + 64] = V4<real>{sigma * d1.x, sigma * d1.y, sigma * d1.z, sigma * d1.w};
    }
};

// B of a round: four lanes per segment in a full one; a round of at most 8, 4, 2
// or 1 segments (the last one) gives each 8, 16, 32 or 64 lanes, so its lanes
// still share the columns.
template <typename real>
__device__ __forceinline__ void round_B(const NbrLDS<real> &L, const int *seg, int s0, int ns, const real *__restrict__ tab,
                               const V4<real> *dTl, real *Bs, int lane)
{
    if (ns > 8) round_B<real, true>(L, seg, s0, ns, 2, tab, dTl, Bs, lane);
    else round_B<real, false>(L, seg, s0, ns, ns > 4 ? 3 : ns > 2 ? 4 : ns > 1 ? 5 : 6, tab, dTl, Bs, lane);
    wave_sync();
}

// f(k, segment of k relative to s0) for the neighbors k of a round, one per lane.
template <typename real, typename Fn>
__device__ __forceinline__ void each_neighbor(const NbrLDS<real> &L, const int *seg, int s0, int ns, int lane, Fn f)
{
    int kb = seg[s0], ke = seg[s0 + ns];
    int cur = -1;   // segment (relative to s0) of the last neighbor before this chunk
    for (int b0 = kb; b0 < ke; b0 += 64) {
        int k = b0 + lane;
        bool in = k < ke;
        bool head = in && (k == kb || L.th[k] != L.th[k - 1]);
        unsigned long long hm = __ballot(head);
        int sidx = cur + __popcll(hm & ((2ull << lane) - 1ull));   // heads up to and including k
        cur += __popcll(hm);
        if (in) f(k, sidx);
    }
}

// Neighbor k of atom i, b: B of its interval.  dE/dR_j and dE/ds_j, then the
// chain rule through Eq. 1: g = dE_i/dr_ij, to the neighbor's pair-gradient
// slot; d = r_ij.
template <typename real>
__device__ __forceinline__ void pair_grad(const EnvArgs &A, const NbrLDS<real> &L, int i, int k, const real *b, V4<real> &d,
                                 real &g0, real &g1, real &g2)
{
    int th = L.th[k];
    real t = L.t[k];
    d = L.Dv[k];
    int slot = L.j[k];
    real dR[4], Q[4];
#pragma unroll
    for (int kk = 0; kk < 4; kk++) horner2<real>(b + kk * 6, t, dR[kk], Q[kk]);
    real rinv, s, sp;
    env_geom<real>(A, d, rinv, s, sp);
    real h0 = d.x * rinv, h1 = d.y * rinv, h2 = d.z * rinv;
    // dE/ds through G: sum_k R_k dB_k/dt with R = s (1, h); no G' past the table end
    real dsG = (th & kOobBit) ? (real)0 : s * (Q[0] + Q[1] * h0 + Q[2] * h1 + Q[3] * h2);
    // R = s (1, h): dE/ds collects dR0 + dR.h; dE/dh = s dR[1..3]
    real dEds = dsG + dR[0] + dR[1] * h0 + dR[2] * h1 + dR[3] * h2;
    real u0 = s * dR[1], u1 = s * dR[2], u2 = s * dR[3];
    real udh = u0 * h0 + u1 * h1 + u2 * h2;
    real c0 = dEds * sp;
    g0 = c0 * h0 + (u0 - udh * h0) * rinv;
    g1 = c0 * h1 + (u1 - udh * h1) * rinv;
    g2 = c0 * h2 + (u2 - udh * h2) * rinv;
    // dE_i/dr_ij, gathered into F_j after the kernel (no atomics)
    put_pg<real>(A.pg, A.cap, i, slot, g0, g1, g2);
}

// The registers are those of 2 (FP64) and 4 waves a SIMD: with the 3 that it
// would choose in FP64 the compiler keeps fewer coefficient loads in flight
// (1,155 us against 1,010 at 108,000 atoms; 555 in FP32).
template <typename real>
__global__ void __launch_bounds__(64)
__attribute__((amdgpu_waves_per_eu(sizeof(real) == 8 ? 2 : 4, sizeof(real) == 8 ? 2 : 4)))
k_emb_bwd(int natoms, EnvArgs A, const real *__restrict__ tab, real sigma, const real *__restrict__ dT,
          const real *__restrict__ dTp, int nparts, double *__restrict__ force, double *__restrict__ w_atom)
{
    HIP_DYNAMIC_SHARED(uint4, smem_raw)   // 16-byte aligned
    char *base = reinterpret_cast<char *>(smem_raw);
    int lane = threadIdx.x;
    int i = xcd_item(blockIdx.x, gridDim.x);
    if (i >= natoms) return;
    NbrLDS<real> L = carve<real>(base, A.sel, ENV_BWD);
    char *p = base + nbr_lds_bytes<real>(A.sel, ENV_BWD);
    V4<real> *dTl = reinterpret_cast<V4<real> *>(p);   // per column
    p += kM * sizeof(V4<real>);
    real *Bs = reinterpret_cast<real *>(p);             // kSegRound x 24
    p += kSegRound * 24 * sizeof(real);
    int *seg = reinterpret_cast<int *>(p);
    // dE/dT into registers first: its loads stream from HBM while the
    // neighbor scan runs
    DTRegs<real> dt;
    dt.load(i, natoms, lane, dT, dTp, nparts);
    const int nn = load_env<real>(i, A, L, lane);
    wave_sync();

    dt.finish(lane, sigma, dTl);
    int nseg = find_segments(L, nn, lane, seg);   // its wave barrier also publishes dT

    real Fi0 = 0, Fi1 = 0, Fi2 = 0;
    real W[9];
#pragma unroll
    for (int r = 0; r < 9; r++) W[r] = 0;
    for (int s0 = 0; s0 < nseg; s0 += kSegRound) {
        int ns = min(kSegRound, nseg - s0);
        round_B(L, seg, s0, ns, tab, dTl, Bs, lane);
        each_neighbor(L, seg, s0, ns, lane, [&](int k, int sidx) __attribute__((always_inline)) {
            V4<real> d;
            real g0, g1, g2;
            pair_grad(A, L, i, k, Bs + sidx * 24, d, g0, g1, g2);
            Fi0 += g0;
            Fi1 += g1;
            Fi2 += g2;
            W[0] -= d.x * g0; W[1] -= d.x * g1; W[2] -= d.x * g2;
            W[3] -= d.y * g0; W[4] -= d.y * g1; W[5] -= d.y * g2;
            W[6] -= d.z * g0; W[7] -= d.z * g1; W[8] -= d.z * g2;
        });
        wave_sync();   // Bs is rewritten by the next round
    }
    for (int off = 32; off > 0; off >>= 1) {
        Fi0 += __shfl_xor(Fi0, off);
        Fi1 += __shfl_xor(Fi1, off);
        Fi2 += __shfl_xor(Fi2, off);
#pragma unroll
        for (int r = 0; r < 9; r++) W[r] += __shfl_xor(W[r], off);
    }
    if (lane == 0) {   // the gather then subtracts the neighbors' dE_j/dr_ji
        force[3 * i] = (double)Fi0;
        force[3 * i + 1] = (double)Fi1;
        force[3 * i + 2] = (double)Fi2;
    }
    if (lane < 9) {
        real v = W[0];
#pragma unroll
        for (int r = 1; r < 9; r++) v = lane == r ? W[r] : v;
        w_atom[(long)i * 9 + lane] = (double)v;
    }
}

// ------------------------------------------------- four waves to an atom
// For systems of fewer atoms than the chip has SIMDs a wave per atom leaves most
// of them idle and the step waits for one wave's chain of work.  Here a block of
// four waves takes an atom: they share the scan and the environment, each forms
// the moments (B) of every fourth round of segments, and the sums over segments
// are split by column and component of R (by component of force and virial),
// so that every sum has the order that it has in the kernels of one wave, and
// the same bits.  Forward and backward
// at 108 atoms, FP64: 24 and 23 us by one wave, 18 and 16 by four; forward at 500,
// FP32: 23 and 18.
constexpr int kWide = 4;

template <typename real>
constexpr int wide_lds_bytes(int sel, bool fwd)
{
    constexpr int al = (int)sizeof(V4<real>);
    int b = (nbr_lds_bytes<real>(sel, fwd ? ENV_FWD : ENV_BWD) + (fwd ? 0 : kM * al) +
             kWide * kSegRound * 24 * (int)sizeof(real) + kWide * seg_bytes(sel) + 31) / 32 * 32;
    return (b + (fwd ? 512 : 3 * sel * (int)sizeof(real)) + al - 1) / al * al;
}

template <typename real>
__global__ void __launch_bounds__(64 * kWide) k_emb_fwd_wide(int natoms, EnvArgs A, const real *__restrict__ tab,
                                                             real sigma, real *__restrict__ T_out,
                                                             int *__restrict__ nnei_out, int *__restrict__ nseg_out)
{
    HIP_DYNAMIC_SHARED(uint4, smem_raw)   // 16-byte aligned
    char *base = reinterpret_cast<char *>(smem_raw);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = xcd_item(blockIdx.x, gridDim.x);
    if (i >= natoms) return;   // the whole block
    NbrLDS<real> L = carve<real>(base, A.sel, ENV_FWD);
    char *p = base + nbr_lds_bytes<real>(A.sel, ENV_FWD);
    real *Ms = reinterpret_cast<real *>(p);   // kWide x kSegRound x 24
    p += kWide * kSegRound * 24 * sizeof(real);
    int *seg = reinterpret_cast<int *>(p + wave * seg_bytes(A.sel));
    // per round of a turn: its intervals (with their place in Ms) and their number
    int *list = reinterpret_cast<int *>(p + kWide * seg_bytes(A.sel));
    int *cnts = list + kWide * kSegRound;   // 2 x kWide of the scan, then kWide of the rounds
    int *num = cnts + 2 * kWide;
    int n_in = 0, over = 0, oob = 0;
    const int nn = build_env_wide<real, kWide>(i, A, L, cnts, n_in, over, oob);
    int nruns = 0;
    const int nseg = find_segments<real, kFwdMaxRun>(L, nn, lane, seg, &nruns);

    // sums: wave w has columns 64 (w mod 2) + lane, components 2 (w / 2) and the next
    const int c = (wave & 1) * 64 + lane, kk = (wave >> 1) * 2;
    real T0 = 0, T1 = 0;
    for (int t0 = 0; t0 < nseg; t0 += kSegRound * kWide) {
        const int s0 = t0 + wave * kSegRound, ns = max(0, min(kSegRound, nseg - s0));
        unsigned long long reps = 0;
        if (ns > 0) reps = round_moments(L, seg, s0, ns, Ms + wave * kSegRound * 24, lane);
        if (reps >> lane & 1)
            list[wave * kSegRound + __popcll(reps & ((1ull << lane) - 1ull))] =
                (L.th[seg[s0 + lane]] & ~kOobBit) << 6 | (wave * kSegRound + lane);
        if (lane == 0) num[wave] = __popcll(reps);
        __syncthreads();
        const int p1 = num[0], p2 = p1 + num[1], p3 = p2 + num[2], tot = p3 + num[3];
        auto entry = [&](int u) {
            const int r = (u >= p1) + (u >= p2) + (u >= p3);
            return __builtin_amdgcn_readfirstlane(list[r * kSegRound + u - (r == 0 ? 0 : r == 1 ? p1 : r == 2 ? p2 : p3)]);
        };
        constexpr int PD = 8;   // intervals whose coefficients are in flight
        real a[PD][6];
        int at[PD];
#pragma unroll
        for (int u = 0; u < PD; u++)
            if (u < tot) {
                const int x = entry(u);
                at[u] = x & 63;
                coef_col(tab, x >> 6, c, a[u]);
            }
        for (int u0 = 0; u0 < tot; u0 += PD) {
#pragma unroll
            for (int u = 0; u < PD; u++) {
                if (u0 + u < tot) {
                    const real *m = Ms + at[u] * 24 + kk * 6;
#pragma unroll
                    for (int e = 0; e < 6; e++) {
                        T0 = fma(m[e], a[u][e], T0);
                        T1 = fma(m[6 + e], a[u][e], T1);
                    }
                    if (u0 + u + PD < tot) {
                        const int x = entry(u0 + u + PD);
                        at[u] = x & 63;
                        coef_col(tab, x >> 6, c, a[u]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        __syncthreads();   // Ms and the list are rewritten by the next turn
    }
    real *o = T_out + ((long)i * kM + c) * 4 + kk;
    o[0] = T0 * sigma;
    o[1] = T1 * sigma;
    if (wave == 0) {
        if (nnei_out && lane == 0) nnei_out[i] = nn;
        if (nseg_out && lane == 0) nseg_out[i] = nruns;
        record_flags<real>(A, lane, n_in, over, oob);
    }
}

template <typename real>
__global__ void __launch_bounds__(64 * kWide) k_emb_bwd_wide(int natoms, EnvArgs A, const real *__restrict__ tab,
                                                             real sigma, const real *__restrict__ dT,
                                                             const real *__restrict__ dTp, int nparts,
                                                             double *__restrict__ force, double *__restrict__ w_atom)
{
    HIP_DYNAMIC_SHARED(uint4, smem_raw)   // 16-byte aligned
    char *base = reinterpret_cast<char *>(smem_raw);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int i = xcd_item(blockIdx.x, gridDim.x);
    if (i >= natoms) return;   // the whole block
    NbrLDS<real> L = carve<real>(base, A.sel, ENV_BWD);
    char *p = base + nbr_lds_bytes<real>(A.sel, ENV_BWD);
    V4<real> *dTl = reinterpret_cast<V4<real> *>(p);   // per column
    p += kM * sizeof(V4<real>);
    real *Bs = reinterpret_cast<real *>(p) + wave * kSegRound * 24;   // kSegRound x 24 of each wave
    p += kWide * kSegRound * 24 * sizeof(real);
    int *seg = reinterpret_cast<int *>(p + wave * seg_bytes(A.sel));
    p = base + (p - base + kWide * seg_bytes(A.sel) + 31) / 32 * 32;
    real *G = reinterpret_cast<real *>(p);   // the pair gradients, sel x 3
    DTRegs<real> dt;
    if (wave == 0) dt.load(i, natoms, lane, dT, dTp, nparts);
    const int nn = load_env<real, ENV_BWD, kWide>(i, A, L, threadIdx.x);
    if (wave == 0) dt.finish(lane, sigma, dTl);
    __syncthreads();
    const int nseg = find_segments(L, nn, lane, seg);

    for (int s0 = wave * kSegRound; s0 < nseg; s0 += kSegRound * kWide) {
        const int ns = min(kSegRound, nseg - s0);
        round_B(L, seg, s0, ns, tab, dTl, Bs, lane);
        each_neighbor(L, seg, s0, ns, lane, [&](int k, int sidx) {
            V4<real> d;
            real g0, g1, g2;
            pair_grad(A, L, i, k, Bs + sidx * 24, d, g0, g1, g2);
            G[3 * k] = g0;
            G[3 * k + 1] = g1;
            G[3 * k + 2] = g2;
        });
        wave_sync();   // Bs is rewritten by the next round
    }
    __syncthreads();
    // wave 0 the force, the others a row of the virial each: per lane over the
    // rounds as in the kernel of one wave, then over the lanes
    real v0 = 0, v1 = 0, v2 = 0;
    for (int s0 = 0; s0 < nseg; s0 += kSegRound)
        for (int k = seg[s0] + lane, ke = seg[min(s0 + kSegRound, nseg)]; k < ke; k += 64) {
            const real g0 = G[3 * k], g1 = G[3 * k + 1], g2 = G[3 * k + 2];
            if (wave == 0) {
                v0 += g0;
                v1 += g1;
                v2 += g2;
            } else {
                const V4<real> d = L.Dv[k];
                const real x = wave == 1 ? d.x : wave == 2 ? d.y : d.z;
                v0 -= x * g0;
                v1 -= x * g1;
                v2 -= x * g2;
            }
        }
    for (int off = 32; off > 0; off >>= 1) {
        v0 += __shfl_xor(v0, off);
        v1 += __shfl_xor(v1, off);
        v2 += __shfl_xor(v2, off);
    }
    if (lane == 0) {
        double *o = wave == 0 ? force + 3 * i : w_atom + (long)i * 9 + (wave - 1) * 3;
        o[0] = (double)v0;
        o[1] = (double)v1;
        o[2] = (double)v2;
    }
}

}  // namespace

// ---------------------------------------------------------- launchers
// Up to this many atoms four waves take one: with a wave an atom that many would
// have one wave to each SIMD of the chip.  Past it the redundant parts (segments,
// barriers) cost more than the idle SIMDs did.  Forward and backward together,
// microseconds, four waves | one: FP32 500 atoms 34 | 45, 800 45 | 45, 1,024 44 | 44,
// 1,371 59 | 49; FP64 500 38 | 49, 800 61 | 52, 1,024 62 | 53, 1,371 81 | 61.  FP64
// crosses between 500 and 800; one line, FP32's, serves both.
constexpr int kWideAtoms = 1024;
static_assert(wide_lds_bytes<double>(512, false) <= 65536 && wide_lds_bytes<double>(512, true) <= 65536,
              "fits a block's LDS at the largest sel");

template <typename real, typename TD>
static void launch_fwd_t(const dp_model *m, const dp_nlist *nl, int n, const double *x, void *T,
                         void *D, void *rec, int *rcnt, unsigned short *slots, int *nnei, int *nseg,
                         hipStream_t st)
{
    EnvArgs A = make_env_args(m, nl, x);
    A.rec = rec;
    A.rcnt = rcnt;
    A.slots = slots;
    A.pg = nl->pg;
    const real *tab = std::is_same<real, double>::value ? (const real *)m->tab64 : (const real *)m->tab32;
    if (n <= kWideAtoms && !D) {
        hipLaunchKernelGGL(k_emb_fwd_wide<real>, dim3(xcd_grid(n)), dim3(64 * kWide), wide_lds_bytes<real>(A.sel, true), st,
                           n, A, tab, (real)m->cfg.desc_scale, (real *)T, nnei, nseg);
        return;
    }
    hipLaunchKernelGGL((k_emb_fwd<real, TD>), dim3(xcd_grid(n)), dim3(64), fwd_lds_bytes<real>(A.sel), st, n, A, tab,
                       (real)m->cfg.desc_scale, (real *)T, (TD *)D, nnei, nseg);
}

template <typename real>
static void launch_bwd_t(const dp_model *m, const dp_nlist *nl, int n, const double *x, const void *dT,
                         const void *dTp, int nparts, const void *rec, const int *rcnt, double *force, double *w_atom,
                         hipStream_t st)
{
    EnvArgs A = make_env_args(m, nl, x);
    A.rec = const_cast<void *>(rec);
    A.rcnt = const_cast<int *>(rcnt);
    A.pg = nl->pg;
    const real *tab = std::is_same<real, double>::value ? (const real *)m->tab64 : (const real *)m->tab32;
    if (n <= kWideAtoms) {
        hipLaunchKernelGGL(k_emb_bwd_wide<real>, dim3(xcd_grid(n)), dim3(64 * kWide), wide_lds_bytes<real>(A.sel, false), st,
                           n, A, tab, (real)m->cfg.desc_scale, (const real *)dT, (const real *)dTp, nparts, force, w_atom);
        return;
    }
    hipLaunchKernelGGL((k_emb_bwd<real>), dim3(xcd_grid(n)), dim3(64), bwd_lds_bytes<real>(A.sel), st, n, A, tab,
                       (real)m->cfg.desc_scale, (const real *)dT, (const real *)dTp, nparts,
                       force, w_atom);
}

void launch_emb_fwd(const dp_model *m, const dp_nlist *nl, int n, const double *x, int precision,
                    void *T, void *D, void *rec, int *rcnt, unsigned short *slots, int *nnei, int *nseg,
                         hipStream_t st)
{
    if (precision == DP_FP64) launch_fwd_t<double, double>(m, nl, n, x, T, D, rec, rcnt, slots, nnei, nseg, st);
    else if (precision == DP_FP32) launch_fwd_t<float, float>(m, nl, n, x, T, D, rec, rcnt, slots, nnei, nseg, st);
    else launch_fwd_t<float, __bf16>(m, nl, n, x, T, D, rec, rcnt, slots, nnei, nseg, st);
}

void launch_emb_bwd(const dp_model *m, const dp_nlist *nl, int n, const double *x, int precision, const void *dT,
                    const void *dTp, int nparts, const void *rec, const int *rcnt, double *force, double *w_atom,
                    hipStream_t st)
{
    if (precision == DP_FP64) launch_bwd_t<double>(m, nl, n, x, dT, dTp, nparts, rec, rcnt, force, w_atom, st);
    else launch_bwd_t<float>(m, nl, n, x, dT, dTp, nparts, rec, rcnt, force, w_atom, st);
}

}  // namespace dp
