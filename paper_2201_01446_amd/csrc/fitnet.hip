// fitnet.hip -- the fitting net of the compressed step in FP64 and FP32, from T
// to dE/dT, with every operand in MFMA register order (gfx950).
//
// The transposed products put the atoms on the columns of the 16 x 16 MFMA
// tile: A holds 16 outputs of a layer (weights), B holds 16 atoms.  Lane
// (r, q) = (lane mod 16, lane / 16) then carries atom r throughout, and
// register i of a result tile holds its column col(i, q) (4 i + q in FP64,
// 4 q + i in FP32), which is what K step i of the next product takes from lane
// group q.  So a layer's result is the next layer's operand as it stands:
// tiles go through LDS only to reach the other waves, each lane reading back
// what the lane of its own number wrote (16 bytes a lane, contiguous, no
// conflicts).  The weights are stored in the order the lanes read them (a
// tile and four K steps contiguous) and stream from L2 straight into
// registers, once per 16 or 32 atoms.
//
//   k_fit_in    z1 = D V1 (D = T<^T T formed once per block, shared in LDS)
//   k_fit_mid   y1 = tanh(z1 + c1), the two inner layers, E_i, and their
//               input gradients down to dz1
//   k_fit_out   dE/dD = dz1 V1^T tile by tile, contracted at once with T into
//               dE/dT (dE/dD is never stored)
//
// Sums run in the same order whatever the number of rows, so an atom's
// results do not depend on the atoms beside it: z1 is the sum of four
// segments of K, added in order (FP32: one chain), and the part of dE/dT that sums over all
// columns b is built from groups of 4, 16 and 128 of them; few rows compute
// the innermost ones side by side.
//
// Bound by the matrix cores.  FP64 MFMA and FP64 vector instructions take
// turns on one pipe (measured: an FMA between two MFMAs costs its full four
// cycles), and the chip clocks down to about 2.13 GHz under FP64 MFMA, so 71
// TFLOP/s is the ceiling here.  Against the tiled GEMMs that kept D or dE/dD in
// HBM (FP64, microseconds; 108 / 2,917 / 108,000 atoms): first layer 104 / 110 /
// 1,990 -> 13 / 68 / 1,800, the
// 240-wide layers 106 / 110 / 1,180 -> 38 / 43 / 990, dE/dD and dE/dT 14 + / 59 +
// / 1,620 + 450 (in the embedding backward) -> 14 / 67 / 1,840.  FP32, 500 /
// 108,000 atoms: first layer 159 / 1,010 -> 24 / 1,000 (one chain of 2,048 terms, D
// formed beside it), the 240-wide layers 50 / 580 -> 21 / 475; dE/dD 900, and dE/dT in
// the embedding backward, -> 940 at 108,000.

#include "dp_internal.h"
#include "emb_common.h"
#include "fit_common.h"

#include <algorithm>
#include <type_traits>

namespace dp {

namespace {

// Four values of a lane (one tile, or one operand of four K steps), the MFMA
// on them, and their place in memory: a piece of 256 reals per tile, read 16
// bytes a lane at a time.
template <typename real> struct Net;
template <> struct Net<double> {
    using v4 = d4v;
    static __host__ __device__ constexpr int col(int i, int q) { return 4 * i + q; }
    static __device__ inline v4 mfma(double a, double b, const v4 &c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ inline v4 get(const double *p, int lane)
    {
        const d2v a = reinterpret_cast<const d2v *>(p)[lane], b = reinterpret_cast<const d2v *>(p)[lane + 64];
        return v4{a[0], a[1], b[0], b[1]};
    }
    static __device__ inline void put(double *p, int lane, const v4 &v)
    {
        reinterpret_cast<d2v *>(p)[lane] = d2v{v[0], v[1]};
        reinterpret_cast<d2v *>(p)[lane + 64] = d2v{v[2], v[3]};
    }
};
template <> struct Net<float> {
    using v4 = f4v;
    static __host__ __device__ constexpr int col(int i, int q) { return 4 * q + i; }
    static __device__ inline v4 mfma(float a, float b, const v4 &c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ inline v4 get(const float *p, int lane) { return reinterpret_cast<const v4 *>(p)[lane]; }
    static __device__ inline void put(float *p, int lane, const v4 &v) { reinterpret_cast<v4 *>(p)[lane] = v; }
};
constexpr int kPiece = 256;   // reals of a tile

// ------------------------------------------------------------ first layer
// One block per RT row tiles and part of K, wave w owns output tile w.  K step
// (b, s): a = col(s, q) in lane group q.  D of the chunk's kInItems (row tile,
// b) pairs is formed once per block, for the next chunk while the products of
// the present one run, and read by all waves from LDS: formed by every wave for
// its own columns, as FP64 vector and matrix instructions share a pipe, it cost
// 8 % of the products (five groups of three column tiles).  The weights of the
// next PD values of b are in flight.  WHOLE: all of K in one block, segment
// after segment; else the block's part is one segment.
constexpr int kInItems = 16;

// Segments of K, whose sums are added in order: FP64 4; FP32 one chain, as each
// rounding of a sum of 2,048 terms is felt by the forces (that of other orders
// and of products split into BF16 parts moved them by up to 4e-5).
template <typename real> constexpr int in_segs() { return sizeof(real) == 8 ? kFitSegs : 1; }

template <typename real, int RT, bool WHOLE>
__global__ void __launch_bounds__(1024, sizeof(real) == 4 && RT < 4 ? 8 : 4) k_fit_in(FitRows fr, int nrt, int nt, const real *__restrict__ T,
                                                 const real *__restrict__ W, real *__restrict__ z)
{
    using N = Net<real>;
    using v4 = typename N::v4;
    HIP_DYNAMIC_SHARED(uint4, smem_raw)
    constexpr int KC = kInItems / RT;                       // b of a chunk
    constexpr int kSegB = kM / in_segs<real>();                  // b of a segment
    constexpr int PD = RT == 4 ? 2 : 4, NB = WHOLE ? kM : kSegB, NP = WHOLE ? 1 : in_segs<real>();
    static_assert(kSegB % KC == 0 && KC % PD == 0, "whole chunks, whole turns of the ring");
    const int wave = wave_id(), lane = threadIdx.x & 63;   // wave < nt <= 16
    const int r = lane & 15, q = lane >> 4;
    const int part = blockIdx.x % NP, tile0 = blockIdx.x / NP * RT;
    if (row_atom(fr, tile0 * 16) < 0) return;   // padding rows only
    real *Db = reinterpret_cast<real *>(smem_raw);         // [2][item][piece]
    v4 *Tl = reinterpret_cast<v4 *>(Db + 2 * kInItems * kPiece);   // [RT][4][64]: T(a = col(s, q))
    const v4 *Tg = reinterpret_cast<const v4 *>(T);
    auto atom_of = [&](int t) { return tile0 + t < nrt ? row_atom(fr, (tile0 + t) * 16 + r) : -1; };
    const real *Wl = W + (long)row_type(fr, tile0 * 16) * fr.w_in + (long)wave * kPiece;   // [b][tile][piece]
    const int b0 = part * NB;
    v4 w[PD];
    auto load_w = [&](int b, int u) { w[u] = N::get(Wl + (long)b * nt * kPiece, lane); };
#pragma unroll
    for (int u = 0; u < PD; u++) load_w(b0 + u, u);
    // item it: row tile it % RT, b = chunk's first + it / RT; this wave forms it0 and it0 + nt, ..
    auto load_t = [&](int it, int b) {
        const int at = atom_of(it % RT);
        return Tg[(long)(at >= 0 ? at : 0) * kM + b + it / RT];
    };
    auto put_d = [&](int it, const v4 &tb, real *buf) {
        v4 d;
#pragma unroll
        for (int s = 0; s < 4; s++) {
            const v4 t = Tl[((it % RT) * 4 + s) * 64 + lane];
            real x = t[0] * tb[0];
#pragma unroll
            for (int k = 1; k < 4; k++) x = fma(t[k], tb[k], x);
            d[s] = x;
        }
        N::put(buf + it * kPiece, lane, d);
    };
    v4 tb = load_t(wave, b0);
    // the chunk at b into buf; then the load of the one after it
    auto put_chunk = [&](int b, real *buf) {
        put_d(wave, tb, buf);
        for (int it = wave + nt; it < kInItems; it += nt) put_d(it, load_t(it, b), buf);
        if (b + KC < b0 + NB) tb = load_t(wave, b + KC);
    };
    // the four waves of a SIMD do that at different times, so that the others'
    // products go on (all at once, at the barrier, left the matrix cores idle)
    const int turn = (wave >> 2) * (KC / 4);
    for (int k = wave; k < RT * 4; k += nt) {
        const int at = atom_of(k >> 2);
        const v4 v = Tg[(long)(at >= 0 ? at : 0) * kM + N::col(k & 3, q)];
        Tl[k * 64 + lane] = at >= 0 ? v : v4{0, 0, 0, 0};   // rows without an atom: D = 0
    }
    v4 acc[RT], tot[RT];
#pragma unroll
    for (int t = 0; t < RT; t++) acc[t] = tot[t] = v4{0, 0, 0, 0};
    __syncthreads();
    put_chunk(b0, Db);
    __syncthreads();
    for (int b = b0; b < b0 + NB; b += KC) {
        const int buf = ((b - b0) / KC) & 1;
        const bool more = b + KC < b0 + NB;
        const real *D = Db + buf * kInItems * kPiece;
#pragma unroll
        for (int k = 0; k < KC; k++) {
            if (k % (KC / 4) == 0 && more && k == turn) put_chunk(b + KC, Db + (buf ^ 1) * kInItems * kPiece);
            v4 x[RT];
#pragma unroll
            for (int t = 0; t < RT; t++) x[t] = N::get(D + (k * RT + t) * kPiece, lane);
#pragma unroll
            for (int s = 0; s < 4; s++)
#pragma unroll
                for (int t = 0; t < RT; t++) acc[t] = N::mfma(w[k % PD][s], x[t][s], acc[t]);
            load_w(min(b + k + PD, b0 + NB - 1), k % PD);
            keep_order();
        }
        if (WHOLE && (b + KC) % kSegB == 0) {
#pragma unroll
            for (int t = 0; t < RT; t++) {
                tot[t] += acc[t];
                acc[t] = v4{0, 0, 0, 0};
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < RT; t++)
        if (tile0 + t < nrt)
            N::put(z + ((long)(part * nrt + tile0 + t) * nt + wave) * kPiece, lane, WHOLE ? tot[t] : acc[t]);
}

// The same for few rows: one wave per row tile, output tile and segment of K,
// D formed in its registers (four waves of a block share the weights).
template <typename real>
__global__ void __launch_bounds__(256) k_fit_in_few(FitRows fr, int nrt, int nt, const real *__restrict__ T,
                                                    const real *__restrict__ W, real *__restrict__ z)
{
    using N = Net<real>;
    using v4 = typename N::v4;
    constexpr int PD = 4, NS = in_segs<real>(), NB = kM / NS;
    const int wave = wave_id(), lane = threadIdx.x & 63;
    const int r = lane & 15, q = lane >> 4;
    int item = xcd_item(blockIdx.x, gridDim.x);   // the column tiles of one row block on one XCD
    if (item >= (nrt + 3) / 4 * nt * NS) return;
    const int ct = item % nt;
    item /= nt;
    const int part = item % NS, tile = item / NS * 4 + wave;
    if (tile >= nrt || row_atom(fr, tile * 16) < 0) return;   // beyond the rows, or padding
    const int atom = row_atom(fr, tile * 16 + r);
    const v4 *Trow = reinterpret_cast<const v4 *>(T) + (long)(atom >= 0 ? atom : 0) * kM;
    const real *Wl = W + (long)row_type(fr, tile * 16) * fr.w_in + (long)ct * kPiece;
    const int b0 = part * NB, b1 = b0 + NB;
    v4 tl[4], w[PD], tb[PD], acc = v4{0, 0, 0, 0};
    auto load = [&](int b, int u) {
        w[u] = N::get(Wl + (long)b * nt * kPiece, lane);
        tb[u] = Trow[b];
    };
#pragma unroll
    for (int u = 0; u < PD; u++) load(b0 + u, u);
#pragma unroll
    for (int s = 0; s < 4; s++) {
        tl[s] = Trow[N::col(s, q)];
        if (atom < 0) tl[s] = v4{0, 0, 0, 0};
    }
    for (int b = b0; b < b1; b += PD)
#pragma unroll
        for (int u = 0; u < PD; u++) {
#pragma unroll
            for (int s = 0; s < 4; s++) {
                real x = tl[s][0] * tb[u][0];
#pragma unroll
                for (int k = 1; k < 4; k++) x = fma(tl[s][k], tb[u][k], x);
                acc = N::mfma(w[u][s], x, acc);
            }
            load(min(b + u + PD, b1 - 1), u);
            keep_order();
        }
    N::put(z + ((long)(part * nrt + tile) * nt + ct) * kPiece, lane, acc);
}

// --------------------------------------------------- the 256-wide layers
// One block per RT row tiles; wave w owns output tile w of every layer, so
// what a later product needs of an earlier one (y1, t2, dy2) stays in its
// lanes' registers.  Two LDS buffers of one operand (a piece per row and
// column tile) alternate between the products: one barrier per product.  The
// weights are PD k tiles ahead of the products: the four products read one
// stream (matrix after matrix), so a product's first tiles are in flight while
// the previous one ends and its results pass the barrier.
// NTC: nt when it is known at compile time (the loops then unroll whole, and an
// operand of the next k tile is in flight without a copy), else 0.
template <typename real, int RT, int PD, int NTC>
struct MidRing {
    using N = Net<real>;
    using v4 = typename N::v4;
    const real *W;   // the wave's tile in the first matrix
    long wm;         // from one matrix to the next
    int nt, lane;
    v4 w[PD];
    __device__ inline void load(int mat, int kt, int u)
    {
        w[u] = N::get(W + mat * wm + (long)min(kt, nt - 1) * kPiece, lane);
    }
    __device__ inline void start(const real *Wt, int nt_, int wave, int lane_)
    {
        nt = nt_;
        lane = lane_;
        wm = (long)nt * nt * kPiece;
        W = Wt + (long)wave * nt * kPiece;
#pragma unroll
        for (int u = 0; u < PD; u++) load(0, u, u);
    }
    // acc = (matrix mat's tile of the wave) x (the operand in B)
    __device__ inline void product(int mat, const real *B, v4 (&acc)[RT])
    {
#pragma unroll
        for (int rt = 0; rt < RT; rt++) acc[rt] = v4{0, 0, 0, 0};
        const int n = NTC ? NTC : nt, nr = (n + PD - 1) / PD * PD;
        v4 x[RT], xn[RT];   // the operand of this and of the next k tile
        auto fetch = [&](int kt) {
#pragma unroll
            for (int rt = 0; rt < RT; rt++) xn[rt] = N::get(B + (kt * RT + rt) * kPiece, lane);
        };
        auto step = [&](int kt, int u) {
            if (NTC || kt < n) {
#pragma unroll
                for (int rt = 0; rt < RT; rt++) x[rt] = xn[rt];
                if (kt + 1 < n) fetch(kt + 1);
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int rt = 0; rt < RT; rt++) acc[rt] = N::mfma(w[u][i], x[rt][i], acc[rt]);
            }
            if (kt + PD < nr) load(mat, kt + PD, u);
            else load(min(mat + 1, 3), kt + PD - nr, u);
            keep_order();
        };
        fetch(0);
        if constexpr (NTC) {
            static_assert(NTC % PD == 0, "whole turns of the ring");
#pragma unroll
            for (int kt = 0; kt < NTC; kt++) step(kt, kt % PD);
        } else {
            for (int k0 = 0; k0 < nr; k0 += PD)
#pragma unroll
                for (int u = 0; u < PD; u++) step(k0 + u, u);
        }
    }
};

template <typename real, int RT, int PD, int NTC, bool TAB>
__global__ void __launch_bounds__(1024, sizeof(real) == 4 ? 8 : 4) k_fit_mid(FitRows fr, int nrt, int nt, int parts,
                                                  const real *__restrict__ z, const real *__restrict__ W,
                                                  const real *__restrict__ fb, const real *__restrict__ tanh_tab,
                                                  double *__restrict__ e_atom, real *__restrict__ dz1)
{
    using N = Net<real>;
    using v4 = typename N::v4;
    HIP_DYNAMIC_SHARED(uint4, smem_raw)
    __shared__ real Ep[16][RT * 16];
    const int wave = wave_id(), lane = threadIdx.x & 63;   // wave < nt <= 16
    const int r = lane & 15, q = lane >> 4;
    const int tile0 = blockIdx.x * RT;
    real *A = reinterpret_cast<real *>(smem_raw), *B = A + nt * RT * kPiece;
    // rows of padding follow the atoms of their type: nothing to do from the first on
    if (row_atom(fr, tile0 * 16) < 0) return;
    const int ty = row_type(fr, tile0 * 16);
    MidRing<real, RT, PD, NTC> ring;   // V2t, V3t, V3, V2
    ring.start(W + (long)ty * fr.w_mid, nt, wave, lane);
    const real *c1 = fb + (long)ty * kFitB + 16 * wave, *c2 = c1 + kFitPad, *c3 = c2 + kFitPad, *w4 = c3 + kFitPad;
    const real *tab = TAB ? tanh_tab : nullptr;
    auto put = [&](real *buf, const v4 (&v)[RT]) {
#pragma unroll
        for (int rt = 0; rt < RT; rt++) N::put(buf + (wave * RT + rt) * kPiece, lane, v[rt]);
    };

    v4 y1[RT], t2[RT], dy2[RT], acc[RT];
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
        const real *p = z + ((long)min(tile0 + rt, nrt - 1) * nt + wave) * kPiece;
        v4 v = N::get(p, lane);
        for (int s = 1; s < parts; s++) v += N::get(p + (long)s * nrt * nt * kPiece, lane);
#pragma unroll
        for (int i = 0; i < 4; i++) y1[rt][i] = tanh_e(v[i] + c1[N::col(i, q)], tab);
    }
    put(A, y1);
    __syncthreads();
    ring.product(0, A, acc);
#pragma unroll
    for (int rt = 0; rt < RT; rt++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            t2[rt][i] = tanh_e(acc[rt][i] + c2[N::col(i, q)], tab);
            dy2[rt][i] = y1[rt][i] + t2[rt][i];   // y2, until dy2 is known
        }
    put(B, dy2);
    __syncthreads();
    ring.product(1, B, acc);
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
        real es = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const real t3 = tanh_e(acc[rt][i] + c3[N::col(i, q)], tab), w = w4[N::col(i, q)];
            es += (dy2[rt][i] + t3) * w;
            acc[rt][i] = w * ((real)1 - t3 * t3);   // dz3
        }
        es += __shfl_xor(es, 16);
        es += __shfl_xor(es, 32);
        if (q == 0) Ep[wave][rt * 16 + r] = es;
    }
    put(A, acc);
    __syncthreads();
    if (threadIdx.x < RT * 16) {
        real e = Ep[0][threadIdx.x];
        for (int w = 1; w < nt; w++) e += Ep[w][threadIdx.x];
        const int row = tile0 * 16 + threadIdx.x;
        const int atom = row < nrt * 16 ? row_atom(fr, row) : -1;
        if (atom >= 0) e_atom[atom] = (double)e + fr.b4[ty];
    }
    ring.product(2, A, acc);
#pragma unroll
    for (int rt = 0; rt < RT; rt++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
            dy2[rt][i] = w4[N::col(i, q)] + acc[rt][i];
            acc[rt][i] = dy2[rt][i] * ((real)1 - t2[rt][i] * t2[rt][i]);   // dz2
        }
    put(B, acc);
    __syncthreads();
    ring.product(3, B, acc);
#pragma unroll
    for (int rt = 0; rt < RT; rt++) {
        v4 o;
#pragma unroll
        for (int i = 0; i < 4; i++) o[i] = (dy2[rt][i] + acc[rt][i]) * ((real)1 - y1[rt][i] * y1[rt][i]);
        if (tile0 + rt < nrt) N::put(dz1 + ((long)(tile0 + rt) * nt + wave) * kPiece, lane, o);
    }
}

// ---------------------------------------------- input gradient and dE/dT
// dE/dD[a][b] of 16 atoms and one b is one tile: rows a = col(i, q), columns
// the atoms.  With T of the lane's atom it gives
//   dT1[k][b]  = sum_a dD[a][b] T<[k][a]   (4 FMA per k in the lane, then a
//                transposing sum over the four lane groups: group q keeps k = q)
//   dT2[k][a] += dD[a][b] T[k][b]          (16 sums in the lane, over all b)
// and dE/dT[k][c] = dT1[k][c] + [c < M<] dT2[k][c].  A wave takes consecutive
// b, two at a time; the block's rows of dz1 sit in LDS.
constexpr int kOutB0 = 4;    // b of the innermost sums of dT2
constexpr int kOutB1 = 16;   // b of the middle ones

// A wave takes NBW columns.  LEVEL 0: it writes the sums over kOutB0 of them
// (32 parts); 1: over kOutB1 (8 parts, NBW = kOutB1); 2: the block's eight waves
// cover all 128 and add theirs (one part, NBW = kOutB1).  part: [part][atom][16
// a][4 k].  The weights of the next PD k tiles are in flight, across the pairs
// of b.
constexpr int out_waves(int level) { return level == 2 ? 8 : 4; }

template <typename real, int LEVEL, int NBW, int NTC>
__global__ void __launch_bounds__(64 * out_waves(LEVEL), 2) k_fit_out(FitRows fr, int nrt, int nt, long natoms,
                                                                      const real *__restrict__ dz1,
                                                                      const real *__restrict__ T,
                                                                      const real *__restrict__ W, real *__restrict__ dT,
                                                                      real *__restrict__ part)
{
    using N = Net<real>;
    using v4 = typename N::v4;
    HIP_DYNAMIC_SHARED(uint4, smem_raw)
    constexpr int NW = out_waves(LEVEL), BPT = kM / (NBW * NW), PD = 3;   // blocks per row tile
    const int wave = wave_id(), lane = threadIdx.x & 63;
    const int r = lane & 15, q = lane >> 4;
    const int tile = blockIdx.x / BPT, b0 = (blockIdx.x % BPT * NW + wave) * NBW;
    if (row_atom(fr, tile * 16) < 0) return;   // padding rows only
    const real *Wl = W + (long)row_type(fr, tile * 16) * fr.w_out;   // [b][tile][piece]
    real *S = reinterpret_cast<real *>(smem_raw);                     // [tile][piece]
    for (int k = wave; k < nt; k += NW) N::put(S + k * kPiece, lane, N::get(dz1 + ((long)tile * nt + k) * kPiece, lane));
    const int atom = row_atom(fr, tile * 16 + r);
    const v4 *Ta = reinterpret_cast<const v4 *>(T) + (long)(atom >= 0 ? atom : 0) * kM;
    v4 tl[4];   // T<[.][col(i, q)]
#pragma unroll
    for (int i = 0; i < 4; i++) tl[i] = Ta[N::col(i, q)];
    const int nk = NTC ? NTC : nt, nr = (nk + PD - 1) / PD * PD;
    v4 w[PD][2];
    auto load = [&](int b, int kt, int u) {
        const real *p = Wl + ((long)b * nt + min(kt, nt - 1)) * kPiece;
        w[u][0] = N::get(p, lane);
        w[u][1] = N::get(p + nt * kPiece, lane);
    };
#pragma unroll
    for (int u = 0; u < PD; u++) load(b0, u, u);
    // (everything read so far has arrived: no wait for it is left in the loops)
    __builtin_amdgcn_s_waitcnt(0);
    __syncthreads();
    v4 x, xn = N::get(S, lane);   // the operand of this and of the next k tile
    v4 acc2[4], tot2[4];   // dT2[.][col(i, q)]
#pragma unroll
    for (int i = 0; i < 4; i++) tot2[i] = v4{0, 0, 0, 0};
    for (int g = 0; g < NBW; g += kOutB0) {
#pragma unroll
        for (int i = 0; i < 4; i++) acc2[i] = v4{0, 0, 0, 0};
        for (int h = 0; h < kOutB0; h += 2) {
            const int b = b0 + g + h;
            const v4 tb[2] = {Ta[b], Ta[b + 1]};
            v4 c[2] = {v4{0, 0, 0, 0}, v4{0, 0, 0, 0}};
            auto step = [&](int kt, int u) {
                if (NTC || kt < nk) {
                    x = xn;
                    xn = N::get(S + (kt + 1 < nk ? kt + 1 : 0) * kPiece, lane);
#pragma unroll
                    for (int i = 0; i < 4; i++) {
                        c[0] = N::mfma(w[u][0][i], x[i], c[0]);
                        c[1] = N::mfma(w[u][1][i], x[i], c[1]);
                    }
                }
                if (kt + PD < nr) load(b, kt + PD, u);
                else load(min(b + 2, b0 + NBW - 2), kt + PD - nr, u);
                keep_order();
            };
            if constexpr (NTC) {
                static_assert(NTC % PD == 0, "whole turns of the ring");
#pragma unroll
                for (int kt = 0; kt < NTC; kt++) step(kt, kt % PD);
            } else {
                for (int k0 = 0; k0 < nr; k0 += PD)
#pragma unroll
                    for (int u = 0; u < PD; u++) step(k0 + u, u);
            }
#pragma unroll
            for (int u = 0; u < 2; u++) {
                const v4 cc = c[u];
                real p[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    real s = cc[0] * tl[0][k];
#pragma unroll
                    for (int i = 1; i < 4; i++) s = fma(cc[i], tl[i][k], s);
                    p[k] = s;
                }
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int k = 0; k < 4; k++) acc2[i][k] = fma(cc[i], tb[u][k], acc2[i][k]);
                const real v = swap_add<true>(swap_add<false>(p[0], p[1]), swap_add<false>(p[2], p[3]));
                if (atom >= 0) dT[((long)atom * kM + b + u) * 4 + q] = v;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
            if (LEVEL > 0) tot2[i] += acc2[i];
            else if (atom >= 0)
                reinterpret_cast<v4 *>(part)[((long)((b0 + g) / kOutB0) * natoms + atom) * 16 + N::col(i, q)] = acc2[i];
        }
    }
    if (LEVEL == 0) return;
    if (LEVEL == 1) {
        if (atom >= 0)
#pragma unroll
            for (int i = 0; i < 4; i++)
                reinterpret_cast<v4 *>(part)[((long)(b0 / kOutB1) * natoms + atom) * 16 + N::col(i, q)] = tot2[i];
        return;
    }
    // the eight waves' sums in wave order, through LDS, a quarter of them at a time
    v4 *X = reinterpret_cast<v4 *>(smem_raw);
#pragma unroll
    for (int i = 0; i < 4; i++) {
        __syncthreads();
        X[wave * 64 + lane] = tot2[i];
        __syncthreads();
        if (wave == i) {
            v4 s = X[lane];
#pragma unroll
            for (int w = 1; w < NW; w++) s += X[w * 64 + lane];
            if (atom >= 0) reinterpret_cast<v4 *>(part)[(long)atom * 16 + N::col(i, q)] = s;
        }
    }
}

// Where the launches change, in row tiles (16 atoms each; width 240, copper;
// microseconds of the kernel on either side, "fewer rows | more rows").  Blocks of
// one tile fill the 256 CUs at 256 of them, so times go in steps, and the better
// side changes back and forth about each line; one set of lines serves FP64
// and FP32.
//
// First layer.  Up to kInFewTiles single waves, four times as many in FP64 (four
// segments of K) as in FP32 (one chain), so that the two cross at different
// places: FP64 at 16 tiles 16 | 23, at 20 26 | 24, at 48 37 | 24; FP32 at 48 25 | 47,
// at 125 41 | 48, at 144 60 | 48.  The line lies between.
// Below kInOneTiles a block takes one tile, then two, which share its weights:
// FP64 at 256 82 | 76, at 282 100 | 108, at 512 159 | 146, at 844 277 | 251; FP32 at 250
// 49 | 82, at 512 87 | 84, at 625 125 | 154, at 844 164 | 155.
// From kInWholeTiles on four tiles, in FP64 with all of K (the inner layers then read
// one part instead of four), both kernels together: FP64 at 512 229 | 329, at 1,024 443 |
// 401, at 1,250 579 | 710, at 2,000 886 | 789; FP32 at 1,024 227 | 214, at 1,250 328 | 376, at
// 2,000 436 | 414.
constexpr int kInFewTiles = 48, kInOneTiles = 512, kInWholeTiles = 1250;
// Inner layers: one tile to a block up to here, then two: FP64 at 250 43 | 72, at 375
// 78 | 73, at 512 84 | 78, at 625 120 | 145, at 844 157 | 148; FP32 at 250 23 | 38, at 512 39 | 40,
// at 625 56 | 68, at 844 72 | 69.
constexpr int kMidOneTiles = 512;
// Input gradient: the sums over all columns are left in 32 parts up to
// kOut32Tiles (a wave has 4 columns up to kOut4Tiles, then 8), in 8 up to
// kOut8Tiles, then added by the block; more parts are more waves, and more to read
// for the backward embedding, whose time is in the last two.  4 | 8 columns: FP64 at 32
// tiles 18 | 25, at 64 29 | 27, at 125 50 | 44; FP32 at 32 12 | 16, at 64 19 | 19, at 125 29 |
// 27.  32 | 8 parts: FP64 at 125 78 | 72, at 183 105 | 109, at 256 133 | 120, at 500 257 | 222; FP32
// at 183 64 | 66, at 256 79 | 70, at 500 139 | 126.  8 | 1: FP64 at 625 276 | 299, at 1,024 464 | 437,
// at 1,875 847 | 818; FP32 at 625 155 | 162, at 1,024 239 | 225, at 1,875 443 | 422.
constexpr int kOut4Tiles = 64, kOut32Tiles = 256, kOut8Tiles = 1024;

}  // namespace

// ----------------------------------------------------------- launchers
template <typename real>
int fit_in_parts(const FitRows &fr) { return row_tiles(fr) < kInWholeTiles ? in_segs<real>() : 1; }
template int fit_in_parts<double>(const FitRows &);
template int fit_in_parts<float>(const FitRows &);

template <typename real>
void launch_fit_in(const FitRows &fr, int nt, const real *T, const void *W, real *z, hipStream_t st)
{
    constexpr bool f64 = sizeof(real) == 8;
    const int nrt = row_tiles(fr), segs = in_segs<real>();
    auto go = [&](auto kern, int RT, int parts) {
        const size_t lds = (size_t)(2 * kInItems + 4 * RT) * kPiece * sizeof(real);
        hipLaunchKernelGGL(kern, dim3(div_up(nrt, RT) * parts), dim3(64 * nt), lds, st, fr, nrt, nt, T, (const real *)W, z);
    };
    if (nrt <= kInFewTiles)
        hipLaunchKernelGGL(k_fit_in_few<real>, dim3(xcd_grid(div_up(nrt, 4) * nt * segs)), dim3(256), 0, st, fr, nrt, nt, T,
                           (const real *)W, z);
    else if (nrt < kInOneTiles) go(k_fit_in<real, 1, !f64>, 1, segs);
    else if (nrt < kInWholeTiles) go(k_fit_in<real, 2, !f64>, 2, segs);
    else go(k_fit_in<real, 4, true>, 4, 1);
}
template void launch_fit_in<double>(const FitRows &, int, const double *, const void *, double *, hipStream_t);
template void launch_fit_in<float>(const FitRows &, int, const float *, const void *, float *, hipStream_t);

template <typename real>
void launch_fit_mid(const FitRows &fr, int nt, int parts, const real *z, const void *W, const real *fb,
                    const real *tanh_tab, double *e_atom, real *dz1, hipStream_t st)
{
    const int nrt = row_tiles(fr);
    auto go = [&](auto kern, int RT) {
        hipLaunchKernelGGL(kern, dim3(div_up(nrt, RT)), dim3(64 * nt), (size_t)2 * nt * RT * kPiece * sizeof(real), st, fr,
                           nrt, nt, parts, z, (const real *)W, fb, tanh_tab, e_atom, dz1);
    };
    // widths of 15 tiles (225 to 240, the paper's 240 among them) have loops of their own
    const int RT = nrt <= kMidOneTiles ? 1 : 2;
    // FP32: the registers of eight waves a SIMD, so that two blocks of 15 waves
    // share a CU (503 -> 475 us at 108,000 atoms); one tile of weights ahead is
    // what fits
    constexpr int PD2 = sizeof(real) == 4 ? 1 : 3;
    if (nt == 15 && !tanh_tab) {
        if (RT == 1) go(k_fit_mid<real, 1, 5, 15, false>, 1);
        else go(k_fit_mid<real, 2, PD2, 15, false>, 2);
    } else if (!tanh_tab) {
        if (RT == 1) go(k_fit_mid<real, 1, 5, 0, false>, 1);
        else go(k_fit_mid<real, 2, PD2, 0, false>, 2);
    } else {
        if (RT == 1) go(k_fit_mid<real, 1, 5, 0, true>, 1);
        else go(k_fit_mid<real, 2, PD2, 0, true>, 2);
    }
}
template void launch_fit_mid<double>(const FitRows &, int, int, const double *, const void *, const double *,
                                     const double *, double *, double *, hipStream_t);
template void launch_fit_mid<float>(const FitRows &, int, int, const float *, const void *, const float *,
                                    const float *, double *, float *, hipStream_t);

int fit_out_parts(const FitRows &fr)
{
    const int nrt = row_tiles(fr);
    return nrt <= kOut32Tiles ? kM / kOutB0 : nrt <= kOut8Tiles ? kM / kOutB1 : 1;
}

template <typename real>
void launch_fit_out(const FitRows &fr, int nt, long natoms, const real *dz1, const real *T, const void *W, real *dT,
                    real *part, hipStream_t st)
{
    const int nrt = row_tiles(fr);
    auto go = [&](auto kern, int level, int nbw) {
        // the combination of the waves' sums takes 8 pieces, dz1 one per tile
        const size_t lds = (size_t)std::max(nt, 8) * kPiece * sizeof(real);
        const int waves = out_waves(level);
        hipLaunchKernelGGL(kern, dim3(nrt * (kM / (nbw * waves))), dim3(64 * waves), lds, st, fr, nrt, nt, natoms, dz1, T,
                           (const real *)W, dT, part);
    };
    auto pick = [&](auto ntc) {
        constexpr int NTC = decltype(ntc)::value;
        if (nrt <= kOut4Tiles) go(k_fit_out<real, 0, 4, NTC>, 0, 4);
        else if (nrt <= kOut32Tiles) go(k_fit_out<real, 0, 8, NTC>, 0, 8);
        else if (nrt <= kOut8Tiles) go(k_fit_out<real, 1, 16, NTC>, 1, 16);
        else go(k_fit_out<real, 2, 16, NTC>, 2, 16);
    };
    if (nt == 15) pick(std::integral_constant<int, 15>());
    else pick(std::integral_constant<int, 0>());
}
template void launch_fit_out<double>(const FitRows &, int, long, const double *, const double *, const void *, double *,
                                     double *, hipStream_t);
template void launch_fit_out<float>(const FitRows &, int, long, const float *, const float *, const void *, float *,
                                    float *, hipStream_t);

}  // namespace dp
