// pack.hip -- the fitting net's weights in the layouts of the kernels that read
// them, formed on the device from the FP64 matrices when a model is created.
//
// A dozen layouts of some 2.4 MB to 12 MB each: filled on the host they took
// most of dp_model_create (11 ms for one type of atom, most of it
// strided loops; the copies went on top).  Here one thread forms one element,
// reading through the caches, and only the FP64 matrices are copied; a model of
// one type takes 1.5 ms.

#include "dp_internal.h"

namespace dp {

namespace {

// float -> bfloat16 bits, round to nearest even (finite values)
__device__ inline unsigned short bf16_of(float f)
{
    unsigned u = __builtin_bit_cast(unsigned, f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
__device__ inline float bf16_value(unsigned short h) { return __builtin_bit_cast(float, (unsigned)h << 16); }

// Two BF16 parts of v (as FP32), pitch apart: the rounded value and what is left of it.
__device__ inline void put_parts(unsigned short *p, long pitch, double v)
{
    const float f = (float)v;
    const unsigned short h = bf16_of(f);
    p[0] = h;
    p[pitch] = bf16_of(f - bf16_value(h));
}

__device__ inline long thread_of() { return blockIdx.x * (long)blockDim.x + threadIdx.x; }

// V1t[t][o][a] = V1[t][a][o], 32 x 32 tiles.
__global__ void __launch_bounds__(256) k_transpose(const double *__restrict__ V1, double *__restrict__ V1t)
{
    __shared__ double s[32][33];
    const int a0 = blockIdx.x * 32, o0 = blockIdx.y * 32, c = threadIdx.x & 31, r0 = threadIdx.x >> 5;
    const long base = (long)blockIdx.z * kDdim * kFitPad;
    for (int r = r0; r < 32; r += 8) s[r][c] = V1[base + (long)(a0 + r) * kFitPad + o0 + c];
    __syncthreads();
    for (int r = r0; r < 32; r += 8) V1t[base + (long)(o0 + r) * kDdim + a0 + c] = s[c][r];
}

__global__ void k_to_float(long n, const double *__restrict__ a, float *__restrict__ b)
{
    const long i = thread_of();
    if (i < n) b[i] = (float)a[i];
}

// Rows of K elements as [hi | lo | hi] (see kSplitBf16).
__global__ void k_split_rows(long n, int K, const double *__restrict__ a, unsigned short *__restrict__ b)
{
    const long i = thread_of();
    if (i >= n) return;
    const long r = i / K;
    const int c = (int)(i % K);
    unsigned short *p = b + r * 3 * K + c;
    put_parts(p, K, a[i]);
    p[2 * K] = p[0];
}

// The four 256 x 256 matrices of the middle layers in the order of use: V2t,
// V3t (out by in), V3, V2 (in by out); rows are the product's outputs.
struct MidMats {
    const double *V[4];
};

// The lane order of fitnet.hip: a piece of 256 reals per tile of 16 columns (nt
// of them) and four K steps; lane l, K step i: row or column l mod 16, k = 4 i +
// l / 16 (FP64, the steps stored in pairs) or 4 (l / 16) + i (FP32).
template <typename real>
__device__ inline void piece_at(int e, int &x, int &k)
{
    if (sizeof(real) == 8) {
        const int i = e / 128 * 2 + e % 2, l = e % 128 / 2;
        x = l % 16;
        k = 4 * i + l / 16;
    } else {
        const int l = e / 4;
        x = l % 16;
        k = 4 * (l / 16) + e % 4;
    }
}

// [type][b][tile] pieces: IN, x the output, k the row a of b; else x = a, k the output.
template <typename real, bool IN>
__global__ void k_pack_first(long n, int nt, const double *__restrict__ V1, real *__restrict__ out)
{
    const long id = thread_of();
    if (id >= n) return;
    int x, k;
    piece_at<real>((int)(id % 256), x, k);
    const long p = id / 256;
    const int tile = (int)(p % nt), b = (int)(p / nt % kM);
    const long t = p / nt / kM;
    const int a = IN ? k : x, o = 16 * tile + (IN ? x : k);
    out[id] = (real)V1[t * kDdim * kFitPad + (long)(a * kM + b) * kFitPad + o];
}

// [type][matrix][output tile][k tile] pieces.
template <typename real>
__global__ void k_pack_mid(long n, int nt, MidMats M, real *__restrict__ out)
{
    const long id = thread_of();
    if (id >= n) return;
    int x, k;
    piece_at<real>((int)(id % 256), x, k);
    const long p = id / 256;
    const int kt = (int)(p % nt), ot = (int)(p / nt % nt), m = (int)(p / nt / nt % 4);
    const long t = p / nt / nt / 4;
    out[id] = (real)M.V[m][t * kFitPad * kFitPad + (long)(16 * ot + x) * kFitPad + 16 * kt + k];
}

constexpr int kBf = 512;   // BF16 elements of a tile and K step: 64 lanes x 8

// The weights as two BF16 parts in the lane order of the mixed kernels of
// fitsplit.hip: K in its natural order, element j of lane l of K step g: k =
// 32 g + 8 (l / 16) + j.  in [type][part][K step][tile][lane][8]; mid [type]
// [matrix][part][K step][tile][lane][8]; out [type][b][part][K step][lane][8].
__global__ void k_pack_mix_in(long n, int nt, const double *__restrict__ V1, unsigned short *__restrict__ out)
{
    const long id = thread_of();
    if (id >= n) return;
    const int e = (int)(id % kBf), l = e / 8, j = e % 8;
    const long p = id / kBf, part = (long)(kDdim / 32) * nt * kBf;
    const int ot = (int)(p % nt), g = (int)(p / nt % (kDdim / 32));
    const long t = p / nt / (kDdim / 32);
    put_parts(out + t * 2 * part + ((long)g * nt + ot) * kBf + e, part,
              V1[t * kDdim * kFitPad + (long)(32 * g + 8 * (l / 16) + j) * kFitPad + 16 * ot + l % 16]);
}
__global__ void k_pack_mix_mid(long n, int ks, MidMats M, unsigned short *__restrict__ out)
{
    const long id = thread_of();
    if (id >= n) return;
    const int nt = 2 * ks, e = (int)(id % kBf), l = e / 8, j = e % 8;
    const long p = id / kBf, part = (long)ks * nt * kBf;
    const int ot = (int)(p % nt), g = (int)(p / nt % ks), m = (int)(p / nt / ks % 4);
    const long t = p / nt / ks / 4;
    put_parts(out + (t * 4 + m) * 2 * part + ((long)g * nt + ot) * kBf + e, part,
              M.V[m][t * kFitPad * kFitPad + (long)(16 * ot + l % 16) * kFitPad + 32 * g + 8 * (l / 16) + j]);
}
__global__ void k_pack_mix_out(long n, int ks, const double *__restrict__ V1, unsigned short *__restrict__ out)
{
    const long id = thread_of();
    if (id >= n) return;
    const int e = (int)(id % kBf), l = e / 8, j = e % 8;
    const long p = id / kBf, part = (long)ks * kBf;
    const int g = (int)(p % ks), b = (int)(p / ks % kM);
    const long t = p / ks / kM;
    put_parts(out + (t * kM + b) * 2 * part + (long)g * kBf + e, part,
              V1[t * kDdim * kFitPad + (long)(l % 16 * kM + b) * kFitPad + 32 * g + 8 * (l / 16) + j]);
}

#define DP_PACK(kernel, n, ...) \
    hipLaunchKernelGGL(kernel, dim3(div_up(n, 256)), dim3(256), 0, (hipStream_t)0, n, __VA_ARGS__)

template <typename real>
dp_status pack_fitnet(const FitWeights &d, FitWeights &w, int ntypes, int nt, const MidMats &mm)
{
    const long nf = (long)ntypes * kM * nt * 256, nm = (long)ntypes * 4 * nt * nt * 256;
    DP_HIP(hipMalloc(&w.in, nf * sizeof(real)));
    DP_PACK((k_pack_first<real, true>), nf, nt, (const double *)d.V1, (real *)w.in);
    DP_HIP(hipMalloc(&w.mid, nm * sizeof(real)));
    DP_HIP(hipMalloc(&w.out, nf * sizeof(real)));
    DP_PACK(k_pack_mid<real>, nm, nt, mm, (real *)w.mid);
    DP_PACK((k_pack_first<real, false>), nf, nt, (const double *)d.V1, (real *)w.out);
    return DP_OK;
}

}  // namespace

// d: the FP64 operands, of which V1 [2048][256], V2, V2t, V3, V3t [256][256] per type
// are there; V1t and every layout of w32 and wbf are allocated and formed here.
// f1: the net's width.
dp_status pack_weights(FitWeights &d, FitWeights &w32, FitWeights &wbf, int ntypes, int f1)
{
    const long n1 = (long)ntypes * kDdim * kFitPad, n2 = (long)ntypes * kFitPad * kFitPad;
    DP_HIP(hipMalloc(&d.V1t, n1 * sizeof(double)));
    hipLaunchKernelGGL(k_transpose, dim3(kDdim / 32, kFitPad / 32, ntypes), dim3(256), 0, (hipStream_t)0,
                       (const double *)d.V1, (double *)d.V1t);
    void *const src[6] = {d.V1, d.V1t, d.V2, d.V2t, d.V3, d.V3t};
    void **const o32[6] = {&w32.V1, &w32.V1t, &w32.V2, &w32.V2t, &w32.V3, &w32.V3t};
    void **const obf[6] = {&wbf.V1, &wbf.V1t, &wbf.V2, &wbf.V2t, &wbf.V3, &wbf.V3t};
    for (int k = 0; k < 6; k++) {
        const long n = k < 2 ? n1 : n2;
        DP_HIP(hipMalloc(o32[k], n * sizeof(float)));
        DP_HIP(hipMalloc(obf[k], 3 * n * sizeof(short)));
        DP_PACK(k_to_float, n, (const double *)src[k], (float *)*o32[k]);
        // K (row length) of each matrix as a GEMM Bt operand
        DP_PACK(k_split_rows, n, k == 1 ? kDdim : kFitPad, (const double *)src[k], (unsigned short *)*obf[k]);
    }
    const MidMats mm{{(const double *)d.V2t, (const double *)d.V3t, (const double *)d.V3, (const double *)d.V2}};
    const int nt = div_up(f1, 16), ks = div_up(f1, 32);
    dp_status s;
    if ((s = pack_fitnet<double>(d, d, ntypes, nt, mm)) != DP_OK) return s;
    if ((s = pack_fitnet<float>(d, w32, ntypes, nt, mm)) != DP_OK) return s;
    const double *V1 = (const double *)d.V1;
    const long ni = (long)ntypes * (kDdim / 32) * 2 * ks * kBf,
               nm = (long)ntypes * 4 * ks * 2 * ks * kBf, no = (long)ntypes * kM * ks * kBf;
    DP_HIP(hipMalloc(&wbf.in, 2 * ni * sizeof(short)));
    DP_HIP(hipMalloc(&wbf.mid, 2 * nm * sizeof(short)));
    DP_HIP(hipMalloc(&wbf.out, 2 * no * sizeof(short)));
    DP_PACK(k_pack_mix_in, ni, 2 * ks, V1, (unsigned short *)wbf.in);
    DP_PACK(k_pack_mix_mid, nm, ks, mm, (unsigned short *)wbf.mid);
    DP_PACK(k_pack_mix_out, no, ks, V1, (unsigned short *)wbf.out);
    DP_HIP(hipGetLastError());
    DP_HIP(hipStreamSynchronize((hipStream_t)0));
    return DP_OK;
}

}  // namespace dp
