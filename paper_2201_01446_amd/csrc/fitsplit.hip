// fitsplit.hip -- the compressed step's fitting net in mixed precision, from T to
// dE/dT, as products on the BF16 matrix cores over operands split into two BF16
// parts (gfx950).
//
// An operand x is the sum of x0 = bf16(x) and x1 = bf16(x - x0) to 16 bits, and a
// product the sum of w0 x0 over all of K, then w1 x0, then w0 x1, accumulated in
// FP32.  (FP32 products as six of three parts each were as exact as, and 1.8 times
// as fast as, the FP32 first layer, but their other rounding moved the forces of
// one model in eleven by more than 2e-5; so that precision stays on the FP32
// instructions, in fitnet.hip.)
//
// The layout is that of fitnet.hip: lane (r, q) carries atom r, and a result
// tile holds columns 4 q + i in register i.  A block has one wave per pair of
// column tiles; each wave reads its own weights from L2 (1 KB per tile, part
// and K step, contiguous) and the atoms' operands, shared by all, from LDS.
// Up to 64 rows to a block: an operand fragment then serves 4 x 2 tiles.
//
// Sums run in an order that does not depend on the number of rows.
//
// Measured (microseconds), 62,500 atoms:
// first layer, inner layers and energy 333 + 430 -> 476, dE/dD and dE/dT 337 +
// 130 -> 314, and no D through HBM (embedding forward 533 -> 400).

#include "dp_internal.h"
#include "emb_common.h"
#include "fit_common.h"

#include <algorithm>
#include <type_traits>

namespace dp {

namespace {

// ---------------------------------------------------------------- mixed
// K runs in its natural order, K step g: element j of lane group q is k = 32 g
// + 8 q + j (k = a M + b for D).  Four values of a result tile, columns 16 t +
// 4 q .. + 4, are half of the eight of lane (r, 2 (t mod 2) + q / 2) of K step
// t / 2.
constexpr int kMixSteps = kDdim / 32;   // K steps of the first layer

// The parts of one result tile (t) into an operand buffer [K step][RT][2][64] of 16 bytes.
template <int RT>
__device__ inline void mix_put(bf8v *buf, int t, int rt, int r, int q, const f4v &v)
{
    typedef __bf16 bf4v __attribute__((ext_vector_type(4)));
    bf4v hi, lo;
#pragma unroll
    for (int i = 0; i < 4; i++) {
        hi[i] = (__bf16)v[i];
        lo[i] = (__bf16)(v[i] - (float)hi[i]);
    }
    bf4v *p = reinterpret_cast<bf4v *>(buf + ((t >> 1) * RT + rt) * 2 * 64 + (2 * (t & 1) + (q >> 1)) * 16 + r) + (q & 1);
    p[0] = hi;
    p[128] = lo;
}

// First layer: D = T<^T T formed per K step (a = g / 4, b = 32 (g mod 4) + 8 q
// + j) and split, its first parts in the first two passes over K, its second
// parts in the third.  Eight waves always: item it of a chunk of 16 (row tile,
// a, quarter of b) is formed by wave it mod 8, which therefore keeps to one
// quarter and holds its T columns in registers.
template <int RT>
__global__ void __launch_bounds__(512) k_mix_in(FitRows fr, int nrt, int ks, const float *__restrict__ T,
                                                const bf8v *__restrict__ W, float *__restrict__ z)
{
    HIP_DYNAMIC_SHARED(uint4, smem_raw)
    constexpr int AC = 4 / RT;             // rows a of D in a chunk
    constexpr int KC = 4 * AC;             // K steps of a chunk
    constexpr int NH = RT == 4 ? 2 : 1;    // row tiles a wave forms D for
    const int wave = wave_id(), lane = threadIdx.x & 63;
    const int r = lane & 15, q = lane >> 4;
    const int tile0 = blockIdx.x * RT;
    if (row_atom(fr, tile0 * 16) < 0) return;   // padding rows only
    const int ty = row_type(fr, tile0 * 16);
    bf8v *Db = reinterpret_cast<bf8v *>(smem_raw);             // [2][KC][RT][64]
    f4v *Tl = reinterpret_cast<f4v *>(Db + 2 * KC * RT * 64);   // [RT][a][16 atoms]
    const f4v *Tg = reinterpret_cast<const f4v *>(T);
    auto atom_of = [&](int t) { return tile0 + t < nrt ? row_atom(fr, (tile0 + t) * 16 + r) : -1; };
    for (int k = wave; k < RT * 4; k += 8) {   // a = 4 (k mod 4) + q
        const int at = atom_of(k >> 2);
        const f4v v = Tg[(long)(at >= 0 ? at : 0) * kM + 4 * (k & 3) + q];
        Tl[((k >> 2) * kMlt + 4 * (k & 3) + q) * 16 + r] = at >= 0 ? v : f4v{0, 0, 0, 0};   // no atom: D = 0
    }
    // items wave and wave + 8: quarter wave mod 4; with it / 4 = wave / 4 + {0, 2}
    // the row tile (RT = 4), the row tile and a (2) or a (1) of the chunk
    const int qb = wave & 3;
    f4v tb[NH][8];
#pragma unroll
    for (int h = 0; h < NH; h++) {
        const int at = atom_of(RT == 4 ? (wave >> 2) + 2 * h : RT == 2 ? wave >> 2 : 0);
        const f4v *p = Tg + (long)(at >= 0 ? at : 0) * kM + 32 * qb + 8 * q;
#pragma unroll
        for (int j = 0; j < 8; j++) tb[h][j] = p[j];
    }
    auto put_chunk = [&](int a0, bool second, bf8v *buf) {
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int m = (wave >> 2) + 2 * h;
            const int rt = RT == 4 ? m : RT == 2 ? wave >> 2 : 0, as = RT == 4 ? 0 : RT == 2 ? h : m;
            const f4v ta = Tl[(rt * kMlt + a0 + as) * 16 + r];
            bf8v p;
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const f4v t = tb[NH == 2 ? h : 0][j];
                float x = ta[0] * t[0];
#pragma unroll
                for (int k = 1; k < 4; k++) x = fmaf(ta[k], t[k], x);
                __bf16 hi = (__bf16)x;
                p[j] = second ? (__bf16)(x - (float)hi) : hi;
            }
            buf[((as * 4 + qb) * RT + rt) * 64 + lane] = p;
        }
    };
    // weights [pass][K step][tile][lane]: parts 0, 1, 0; a chunk ahead is KC steps
    const bool mine = wave < ks;
    const bf8v *Wl = W + (long)ty * fr.w_in + (long)min(wave, ks - 1) * 2 * 64;
    constexpr int PD = 4;
    bf8v w[PD][2];
    auto load_w = [&](int step, int u) {
        const int s = min(step, 3 * kMixSteps - 1);
        const bf8v *p = Wl + ((long)(s / kMixSteps == 1 ? kMixSteps : 0) + s % kMixSteps) * ks * 2 * 64;
        w[u][0] = p[lane];
        w[u][1] = p[lane + 64];
    };
    f4v acc[2][RT];
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int t = 0; t < RT; t++) acc[c][t] = f4v{0, 0, 0, 0};
#pragma unroll
    for (int u = 0; u < PD; u++) load_w(u, u);
    __syncthreads();
    put_chunk(0, false, Db);
    __syncthreads();
    // the two waves of a SIMD form the next chunk at different times, so that the
    // other's products go on
    const int turn = (wave >> 2) * (KC / 2);
    constexpr int NCH = 3 * kMixSteps / KC, CPP = kMixSteps / KC;   // chunks, chunks of a pass
    for (int ch = 0; ch < NCH; ch++) {
        const bf8v *D = Db + (ch & 1) * KC * RT * 64;
        const bool more = ch + 1 < NCH;
        auto put_next = [&] { put_chunk((ch + 1) % CPP * AC, ch + 1 >= 2 * CPP, Db + ((ch + 1) & 1) * KC * RT * 64); };
        if (!mine && more) put_next();
        if (mine) {
#pragma unroll
            for (int k = 0; k < KC; k++) {
                if (k % (KC / 2) == 0 && more && k == turn) put_next();
#pragma unroll
                for (int t = 0; t < RT; t++) {
                    const bf8v x = D[(k * RT + t) * 64 + lane];
#pragma unroll
                    for (int c = 0; c < 2; c++)
                        acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[k % PD][c], x, acc[c][t], 0, 0, 0);
                }
                load_w(ch * KC + k + PD, k % PD);
                keep_order();
            }
        }
        __syncthreads();
    }
    if (!mine) return;
#pragma unroll
    for (int t = 0; t < RT; t++)
        if (tile0 + t < nrt) {
#pragma unroll
            for (int c = 0; c < 2; c++)
                reinterpret_cast<f4v *>(z)[((long)(tile0 + t) * 2 * ks + 2 * wave + c) * 64 + lane] = acc[c][t];
        }
}

// The 256-wide layers: one block per RT row tiles, one wave per pair of column
// tiles in every layer (what a later product needs of an earlier one stays in
// registers).  The operand of a product in LDS, two buffers in turn; the
// weights [matrix][part][K step][tile][lane] in one stream over the four
// products, PD steps ahead.  The registers of four waves a SIMD, so that two
// blocks share a CU and one computes while the other meets at its barriers, and
// KS K steps known at compile time, so that the 24 steps of a product are
// unrolled whole and pass and place cost no division: 311 us before, 240 with the
// first and 175 with both (62,500 atoms; its products alone are 80).
template <int RT, int KS, bool TAB>
__global__ void __launch_bounds__(512, 4) k_mix_mid(FitRows fr, int nrt, int ks_, const float *__restrict__ z,
                                                 const bf8v *__restrict__ W, const float *__restrict__ fb,
                                                 const float *__restrict__ tanh_tab, double *__restrict__ e_atom,
                                                 bf8v *__restrict__ dz1)
{
    HIP_DYNAMIC_SHARED(uint4, smem_raw)
    __shared__ float Ep[8][RT * 16];
    const int ks = KS ? KS : ks_;
    const int wave = wave_id(), lane = threadIdx.x & 63;
    const int r = lane & 15, q = lane >> 4;
    const int tile0 = blockIdx.x * RT;
    if (row_atom(fr, tile0 * 16) < 0) return;   // padding rows only
    const int ty = row_type(fr, tile0 * 16);
    bf8v *A = reinterpret_cast<bf8v *>(smem_raw), *B = A + ks * RT * 2 * 64;
    const float *c1 = fb + (long)ty * kFitB + 32 * wave + 4 * q, *c2 = c1 + kFitPad, *c3 = c2 + kFitPad, *w4 = c3 + kFitPad;
    const float *tab = TAB ? tanh_tab : nullptr;
    auto vec = [&](const float *v, int c) { return *reinterpret_cast<const f4v *>(v + 16 * c); };

    constexpr int PD = 2;
    static_assert(3 * KS % PD == 0, "whole turns of the ring");
    const int ns = 3 * ks, nr = (ns + PD - 1) / PD * PD;   // steps of a product, and of the ring
    const bf8v *Wl = W + (long)ty * fr.w_mid + (long)wave * 2 * 64;
    const long wm = (long)4 * ks * ks * 64;   // one matrix
    bf8v w[PD][2];
    auto load_w = [&](int m, int s, int u) {
        s = min(s, ns - 1);
        const int pass = s / ks;
        const bf8v *p = Wl + m * wm + ((long)(pass == 1 ? ks : 0) + s - pass * ks) * ks * 2 * 64;
        w[u][0] = p[lane];
        w[u][1] = p[lane + 64];
    };
    auto put = [&](bf8v *buf, const f4v (&v)[2][RT]) {
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int t = 0; t < RT; t++) mix_put<RT>(buf, 2 * wave + c, t, r, q, v[c][t]);
    };
    f4v acc[2][RT];
    auto product = [&](int m, const bf8v *buf) {
#pragma unroll
        for (int c = 0; c < 2; c++)
#pragma unroll
            for (int t = 0; t < RT; t++) acc[c][t] = f4v{0, 0, 0, 0};
        auto step = [&](int s, int u) {
            if (KS || s < ns) {
                const int pass = s / ks, k = s - pass * ks;
#pragma unroll
                for (int t = 0; t < RT; t++) {
                    const bf8v x = buf[((k * RT + t) * 2 + (pass == 2 ? 1 : 0)) * 64 + lane];
#pragma unroll
                    for (int c = 0; c < 2; c++)
                        acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[u][c], x, acc[c][t], 0, 0, 0);
                }
            }
            if (s + PD < nr) load_w(m, s + PD, u);
            else load_w(min(m + 1, 3), s + PD - nr, u);
            keep_order();
        };
        if constexpr (KS) {
#pragma unroll
            for (int s = 0; s < 3 * KS; s++) step(s, s % PD);
        } else {
            for (int s0 = 0; s0 < nr; s0 += PD)
#pragma unroll
                for (int u = 0; u < PD; u++) step(s0 + u, u);
        }
    };
#pragma unroll
    for (int u = 0; u < PD; u++) load_w(0, u, u);
    f4v y1[2][RT], t2[2][RT], dy2[2][RT];
#pragma unroll
    for (int c = 0; c < 2; c++)
#pragma unroll
        for (int t = 0; t < RT; t++) {
            const f4v v = reinterpret_cast<const f4v *>(z)[((long)min(tile0 + t, nrt - 1) * 2 * ks + 2 * wave + c) * 64 + lane];
            const f4v b = vec(c1, c);
#pragma unroll
            for (int i = 0; i < 4; i++) y1[c][t][i] = tanh_e(v[i] + b[i], tab);
        }
    put(A, y1);
    __syncthreads();
    product(0, A);
#pragma unroll
    for (int c = 0; c < 2; c++) {
        const f4v b = vec(c2, c);
#pragma unroll
        for (int t = 0; t < RT; t++) {
#pragma unroll
            for (int i = 0; i < 4; i++) t2[c][t][i] = tanh_e(acc[c][t][i] + b[i], tab);
            dy2[c][t] = y1[c][t] + t2[c][t];   // y2, until dy2 is known
        }
    }
    put(B, dy2);
    __syncthreads();
    product(1, B);
    float es[RT];
#pragma unroll
    for (int t = 0; t < RT; t++) es[t] = 0;
#pragma unroll
    for (int c = 0; c < 2; c++) {
        const f4v b = vec(c3, c), v4 = vec(w4, c);
#pragma unroll
        for (int t = 0; t < RT; t++)
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const float t3 = tanh_e(acc[c][t][i] + b[i], tab);
                es[t] += (dy2[c][t][i] + t3) * v4[i];
                acc[c][t][i] = v4[i] * (1.f - t3 * t3);   // dz3
            }
    }
#pragma unroll
    for (int t = 0; t < RT; t++) {
        es[t] += __shfl_xor(es[t], 16);
        es[t] += __shfl_xor(es[t], 32);
        if (q == 0) Ep[wave][t * 16 + r] = es[t];
    }
    put(A, acc);
    __syncthreads();
    if (threadIdx.x < RT * 16) {
        float e = Ep[0][threadIdx.x];
        for (int v = 1; v < ks; v++) e += Ep[v][threadIdx.x];
        const int row = tile0 * 16 + threadIdx.x;
        const int atom = row < nrt * 16 ? row_atom(fr, row) : -1;
        if (atom >= 0) e_atom[atom] = (double)e + fr.b4[ty];
    }
    product(2, A);
#pragma unroll
    for (int c = 0; c < 2; c++) {
        const f4v v4 = vec(w4, c);
#pragma unroll
        for (int t = 0; t < RT; t++) {
            dy2[c][t] = v4 + acc[c][t];
#pragma unroll
            for (int i = 0; i < 4; i++) acc[c][t][i] = dy2[c][t][i] * (1.f - t2[c][t][i] * t2[c][t][i]);   // dz2
        }
    }
    put(B, acc);
    __syncthreads();
    product(3, B);
    // dz1, split: [row tile][K step][part][64] of 16 bytes
#pragma unroll
    for (int t = 0; t < RT; t++) {
        if (tile0 + t >= nrt) break;
#pragma unroll
        for (int c = 0; c < 2; c++) {
            f4v o;
#pragma unroll
            for (int i = 0; i < 4; i++) o[i] = (dy2[c][t][i] + acc[c][t][i]) * (1.f - y1[c][t][i] * y1[c][t][i]);
            mix_put<1>(dz1 + (long)(tile0 + t) * ks * 2 * 64, 2 * wave + c, 0, r, q, o);
        }
    }
}

// Input gradient and dE/dT, as k_fit_out of fitnet.hip (rows a = 4 q + i): a
// wave takes 16 columns b, two at a time, for RT row tiles whose dz1 sits in
// LDS.  WPB waves to a block; 8: the block covers all 128 columns and adds the
// waves' dT2 in order; fewer: each wave writes its own to part[b / 16].
constexpr int kMixOutB = 16;   // columns of a wave

template <int RT, int WPB, int KS>
__global__ void __launch_bounds__(64 * WPB) k_mix_out(FitRows fr, int nrt, int ks_, long natoms,
                                                      const bf8v *__restrict__ dz1, const float *__restrict__ T,
                                                      const bf8v *__restrict__ W, float *__restrict__ dT,
                                                      float *__restrict__ part)
{
    HIP_DYNAMIC_SHARED(uint4, smem_raw)
    constexpr int BPT = 8 / WPB;   // blocks per RT row tiles
    const int ks = KS ? KS : ks_;
    const int wave = wave_id(), lane = threadIdx.x & 63;
    const int r = lane & 15, q = lane >> 4;
    const int tile0 = blockIdx.x / BPT * RT, b0 = (blockIdx.x % BPT * WPB + wave) * kMixOutB;
    if (row_atom(fr, tile0 * 16) < 0) return;   // padding rows only
    const int ty = row_type(fr, tile0 * 16);
    bf8v *S = reinterpret_cast<bf8v *>(smem_raw);          // [part][K step][RT][64]
    f4v *Tl = reinterpret_cast<f4v *>(S + 2 * ks * RT * 64);   // [RT][4][64]: T(a = 4 q + i)
    const f4v *Tg = reinterpret_cast<const f4v *>(T);
    int atom[RT];
#pragma unroll
    for (int t = 0; t < RT; t++) atom[t] = tile0 + t < nrt ? row_atom(fr, (tile0 + t) * 16 + r) : -1;
    for (int k = wave; k < ks * 2 * RT; k += WPB) {
        const int t = k % RT, kn = k / RT;   // kn = 2 K step + part
        S[((kn & 1) * ks * RT + (kn >> 1) * RT + t) * 64 + lane] =
            dz1[((long)min(tile0 + t, nrt - 1) * ks * 2 + kn) * 64 + lane];
    }
#pragma unroll
    for (int t = 0; t < RT; t++)
        for (int j = wave; j < 4; j += WPB)
            Tl[(t * 4 + j) * 64 + lane] = Tg[(long)(atom[t] >= 0 ? atom[t] : 0) * kM + 4 * q + j];
    constexpr int PD = 3;
    static_assert(3 * KS % PD == 0, "whole turns of the ring");
    const int ns = 3 * ks, nr = (ns + PD - 1) / PD * PD;
    const bf8v *Wl = W + (long)ty * fr.w_out;   // [b][part][K step][lane]
    bf8v w[PD][2];
    auto load_w = [&](int b, int s, int u) {
        s = min(s, ns - 1);
        const bf8v *p = Wl + ((long)b * 2 * ks + (s >= 2 * ks ? s - 2 * ks : s)) * 64;
        // steps: part 0, part 1, part 0 again
        w[u][0] = p[lane];
        w[u][1] = (p + (long)2 * ks * 64)[lane];
    };
#pragma unroll
    for (int u = 0; u < PD; u++) load_w(b0, u, u);
    f4v acc2[RT][4];   // dT2[.][4 q + i]
#pragma unroll
    for (int t = 0; t < RT; t++)
#pragma unroll
        for (int i = 0; i < 4; i++) acc2[t][i] = f4v{0, 0, 0, 0};
    __syncthreads();
    for (int b = b0; b < b0 + kMixOutB; b += 2) {
        const int bn = min(b + 2, b0 + kMixOutB - 2);
        f4v c[2][RT];
#pragma unroll
        for (int u = 0; u < 2; u++)
#pragma unroll
            for (int t = 0; t < RT; t++) c[u][t] = f4v{0, 0, 0, 0};
        auto step = [&](int s, int v) {
            if (KS || s < ns) {
                // the operand: part 0 for the first two passes, then part 1
                const int k = s < ks ? s : s - ks;   // index into [part][K step]
#pragma unroll
                for (int t = 0; t < RT; t++) {
                    const bf8v x = S[(k * RT + t) * 64 + lane];
                    c[0][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[v][0], x, c[0][t], 0, 0, 0);
                    c[1][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[v][1], x, c[1][t], 0, 0, 0);
                }
            }
            if (s + PD < nr) load_w(b, s + PD, v);
            else load_w(bn, s + PD - nr, v);
            keep_order();
        };
        if constexpr (KS) {
#pragma unroll
            for (int s = 0; s < 3 * KS; s++) step(s, s % PD);
        } else {
            for (int s0 = 0; s0 < nr; s0 += PD)
#pragma unroll
                for (int v = 0; v < PD; v++) step(s0 + v, v);
        }
#pragma unroll
        for (int t = 0; t < RT; t++) {
            const f4v *Tr = Tg + (long)(atom[t] >= 0 ? atom[t] : 0) * kM + b;
            f4v tl[4];
#pragma unroll
            for (int i = 0; i < 4; i++) tl[i] = Tl[(t * 4 + i) * 64 + lane];
#pragma unroll
            for (int u = 0; u < 2; u++) {
                const f4v cc = c[u][t], tb = Tr[u];
                float p[4];
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    float s = cc[0] * tl[0][k];
#pragma unroll
                    for (int i = 1; i < 4; i++) s = fmaf(cc[i], tl[i][k], s);
                    p[k] = s;
                }
#pragma unroll
                for (int i = 0; i < 4; i++)
#pragma unroll
                    for (int k = 0; k < 4; k++) acc2[t][i][k] = fmaf(cc[i], tb[k], acc2[t][i][k]);
                // lane group q ends with k = q
                const float v = swap_add<true>(swap_add<false>(p[0], p[1]), swap_add<false>(p[2], p[3]));
                if (atom[t] >= 0) dT[((long)atom[t] * kM + b + u) * 4 + q] = v;
            }
        }
    }
    if (WPB < 8) {
#pragma unroll
        for (int t = 0; t < RT; t++)
            if (atom[t] >= 0) {
                f4v *o = reinterpret_cast<f4v *>(part) + ((long)(b0 / kMixOutB) * natoms + atom[t]) * 16 + 4 * q;
#pragma unroll
                for (int i = 0; i < 4; i++) o[i] = acc2[t][i];
            }
        return;
    }
    // the waves' sums in wave order, through LDS one row tile at a time
    f4v *X = reinterpret_cast<f4v *>(smem_raw);   // [wave][4][64]
#pragma unroll
    for (int t = 0; t < RT; t++) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 4; i++) X[(wave * 4 + i) * 64 + lane] = acc2[t][i];
        __syncthreads();
        if (wave < 4) {
            f4v s = X[wave * 64 + lane];
#pragma unroll
            for (int v = 1; v < WPB; v++) s += X[(v * 4 + wave) * 64 + lane];
            if (atom[t] >= 0) reinterpret_cast<f4v *>(part)[(long)atom[t] * 16 + 4 * q + wave] = s;
        }
    }
}

// Where the launches change, in row tiles (16 atoms each; width 240, copper;
// microseconds on either side, "fewer rows | more rows"; the times go in steps,
// as the blocks fill the 256 CUs).
// First layer: one tile to a block up to kInOneTiles (with the inner layers at 183
// tiles 56 | 67, at 256 58 | 68, at 375 81 | 73, at 512 88 | 76), two up to kInTwoTiles, then
// four (at 512 76 | 91, at 750 103 | 99, at 1,024 121 | 114, at 1,500 179 | 198, at 2,500 281 | 295:
// four lose there what they gain where they fill the chip).
// Inner layers: one up to kMidOneTiles, then two (at 256 58 | 62, at 375 77 | 73, at
// 512 80 | 76).
// Input gradient: up to kSplitTiles groups of 16 columns in blocks of their own, of
// one tile up to kOutOneTiles, then two (at 64 24 | 29, at 125 26 | 30, at 183 32 | 31), then whole rows of
// four tiles (with the backward embedding, which reads the parts: at 375 89 | 101, at
// 512 103 | 111, at 750 139 | 126, at 1,875 362 | 292).
constexpr int kInOneTiles = 256, kInTwoTiles = 1024, kMidOneTiles = 256, kOutOneTiles = 64, kSplitTiles = 512;

}  // namespace

// ----------------------------------------------------------- launchers
void launch_mix_fwd(const FitRows &fr, int nt, const float *T, const FitWeights &fw, const float *fb,
                    const float *tanh_tab, float *z, double *e_atom, void *dz1, hipStream_t st)
{
    const int nrt = row_tiles(fr), ks = div_up(nt, 2);
    auto in = [&](auto kern, int RT) {
        const size_t lds = (size_t)2 * 16 * 1024 + RT * kMlt * 256;
        hipLaunchKernelGGL(kern, dim3(div_up(nrt, RT)), dim3(512), lds, st, fr, nrt, ks, T, (const bf8v *)fw.in, z);
    };
    if (nrt <= kInOneTiles) in(k_mix_in<1>, 1);
    else if (nrt <= kInTwoTiles) in(k_mix_in<2>, 2);
    else in(k_mix_in<4>, 4);
    auto mid = [&](auto kern, int RT) {
        const size_t lds = (size_t)2 * ks * RT * 2 * 1024;
        hipLaunchKernelGGL(kern, dim3(div_up(nrt, RT)), dim3(64 * ks), lds, st, fr, nrt, ks, z, (const bf8v *)fw.mid, fb,
                           tanh_tab, e_atom, (bf8v *)dz1);
    };
    // (widths of 225 to 256 columns, 240 among them, with the steps unrolled whole)
    auto mids = [&](auto KS) {
        constexpr int k = decltype(KS)::value;
        if (nrt <= kMidOneTiles) {
            if (tanh_tab) mid(k_mix_mid<1, k, true>, 1);
            else mid(k_mix_mid<1, k, false>, 1);
        } else {
            if (tanh_tab) mid(k_mix_mid<2, k, true>, 2);
            else mid(k_mix_mid<2, k, false>, 2);
        }
    };
    if (ks == 8) mids(std::integral_constant<int, 8>{});
    else mids(std::integral_constant<int, 0>{});
}

int mix_out_parts(const FitRows &fr) { return row_tiles(fr) <= kSplitTiles ? kM / kMixOutB : 1; }

void launch_mix_out(const FitRows &fr, int nt, long natoms, const void *dz1, const float *T, const void *W, float *dT,
                    float *part, hipStream_t st)
{
    const int nrt = row_tiles(fr), ks = div_up(nt, 2);
    auto go = [&](auto kern, int RT, int WPB) {
        const size_t lds = std::max((size_t)2 * ks * RT * 1024 + RT * 4096, WPB == 8 ? (size_t)32768 : 0);
        hipLaunchKernelGGL(kern, dim3(div_up(nrt, RT) * (8 / WPB)), dim3(64 * WPB), lds, st, fr, nrt, ks, natoms,
                           (const bf8v *)dz1, T, (const bf8v *)W, dT, part);
    };
    auto out = [&](auto KS) {
        constexpr int k = decltype(KS)::value;
        if (mix_out_parts(fr) == 1) go(k_mix_out<4, 8, k>, 4, 8);
        else if (nrt <= kOutOneTiles) go(k_mix_out<1, 2, k>, 1, 2);
        else go(k_mix_out<2, 4, k>, 2, 4);
    };
    if (ks == 8) out(std::integral_constant<int, 8>{});
    else out(std::integral_constant<int, 0>{});
}

}  // namespace dp
