// Parity encoding: A'_{k+p} = sum_j P[p][j] A_j for the n-k parity blocks
// (Sec. III-A: the (n,k) code applied to every element of the k row-blocks;
// the k systematic blocks are A itself and are never copied).
//
// The contraction has k (<= a few dozen) terms per output element and the
// whole pass streams A once and writes the parity planes once, so it is bound
// by HBM bandwidth, not arithmetic (about 2 flops per byte, far below the
// matrix cores' ridge): each thread owns a short vector of columns of one
// block row t, walks the k blocks j with kBatch loads in flight, and keeps up
// to kGroup parity accumulators in registers; the sum runs over j in order.
// Parity rows beyond kGroup are handled by further groups, each re-reading A
// while the others of its rows do.
//
// Rows start at any element boundary and have any length: a thread's vector
// (VEC columns) that would pass the row's end is moved back to end with it, so
// the last two threads of a row form some columns twice, with the same values.
// A row of fewer than 256 vectors takes only as many threads, and a workgroup
// several rows ((3,2) on 300000 x 200: 242 us with one row each, 120 here; bf16
// 184 and 49; (25,23) on 11500 x 5750, scalar loads 76, here 57).
//
// Storage: with planes == 2 the exact sum (fp64 for fp32 inputs, fp32 for
// bf16 inputs) is stored as hi = round(sum) and lo = round(sum - hi).
#include "internal.h"

namespace coded {
namespace {

constexpr int kGroup = 8;       // parity rows per pass
constexpr int kThreads = 256;
constexpr int kBatch = 8;       // blocks whose loads are in flight together

__device__ inline uint16_t f32_to_bf16_rne(float f) {
    uint32_t b = __float_as_uint(f);
    b += 0x7FFFu + ((b >> 16) & 1u);
    return static_cast<uint16_t>(b >> 16);
}
__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float(static_cast<uint32_t>(h) << 16); }

typedef float f32x4e __attribute__((ext_vector_type(4), aligned(4)));
typedef unsigned int u32x4e __attribute__((ext_vector_type(4), aligned(2)));
typedef unsigned int u32x2e __attribute__((ext_vector_type(2), aligned(2)));

// Threads per block row (a workgroup takes kThreads / that many rows; one row
// without the division that tells several apart).
int row_threads(int64_t r, int vec) {
    const int64_t v = ceil_div(r, vec);
    return 2 * v <= kThreads ? static_cast<int>(v) : kThreads;
}

// Small planes take one column a thread: with few threads the call lasts as long
// as one of them walks its k blocks, eight parity sums for every column it owns
// (elements of a plane times groups; (32,24) on 2000 x 257 bf16 17.0 us with eight
// columns a thread, 11.5 with one; (128,96) on 8000 x 400, 134400, 56.8 and 41.7;
// (16,12) on 8000 x 400, 266800, 7.9 and 8.1; fp32 (128,96) on 8000 x 200, 67200,
// 44.9 and 43.0).
constexpr int64_t kSingleF32 = 96 << 10, kSingleBf16 = 256 << 10;

// The workgroup's row index (in units of the rows it takes) and first parity
// row.  Workgroups go to the 8 XCDs in turn, so the groups of parity rows that
// read the same rows of A sit 8 apart: they run on one XCD at about the same
// time, and A comes from HBM once ((64,48), 16 parity rows in two groups, on
// 40000 x 4000: 349 us with the groups one after the other, 241 here; 60000 x
// 4097 bf16 275).
__device__ inline void row_and_group(int groups, int64_t& t, int& p0) {
    const uint32_t b = blockIdx.x, rest = b >> 3, g = static_cast<uint32_t>(groups);
    t = groups > 1 ? static_cast<int64_t>(rest / g) * 8 + (b & 7) : b;
    p0 = groups > 1 ? static_cast<int>(rest % g) * kGroup : 0;
}

// One thread: VEC consecutive columns of block row t, parity rows
// [p0, p0 + np) with np <= kGroup.
template <int VEC>
__global__ __launch_bounds__(kThreads) void encode_f32_kernel(EncodeArgs a, int groups, int width) {
    __shared__ double sP[kGroup * kMaxN];
    int64_t t;
    int p0;
    row_and_group(groups, t, p0);
    int lane = threadIdx.x;
    if (width < kThreads) {               // several rows: this thread's row and place in it
        const int per = kThreads / width, row = lane / width;
        t = t * per + row;
        lane = row < per ? lane - row * width : kThreads;
    }
    const int64_t chunk = blockIdx.y;
    const int npar = a.n - a.k;
    const int np = min(kGroup, npar - p0);
    const int k = a.k;
    for (int e = threadIdx.x; e < np * k; e += kThreads) {
        const int p = e / k, j = e % k;
        sP[p * k + j] = a.G[(a.k + p0 + p) * k + j];
    }
    __syncthreads();
    int64_t c = (chunk * kThreads + lane) * VEC;
    if (c >= a.r || t >= a.qb) return;
    c = min(c, a.r - VEC);
    const float* A = static_cast<const float*>(a.A);

    double acc[kGroup][VEC];
#pragma unroll
    for (int p = 0; p < kGroup; ++p)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[p][v] = 0.0;

    // Blocks whose row t lies inside A (rows of later blocks are the zero
    // padding and contribute nothing); their loads go out kBatch at a time.
    const int kv = static_cast<int>(min<int64_t>(k, (a.q - t + a.qb - 1) / a.qb));
    for (int j0 = 0; j0 < kv; j0 += kBatch) {
        float v4[kBatch][VEC];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int j = min(j0 + u, kv - 1);   // past the last block: re-read it, not used
            const float* src = A + (static_cast<int64_t>(j) * a.qb + t) * a.lda + c;
            if constexpr (VEC == 4) {
                const f32x4e f = *reinterpret_cast<const f32x4e*>(src);
                v4[u][0] = f.x; v4[u][1] = f.y; v4[u][2] = f.z; v4[u][3] = f.w;
            } else {
#pragma unroll
                for (int v = 0; v < VEC; ++v) v4[u][v] = src[v];
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (j0 + u >= kv) break;
#pragma unroll
            for (int p = 0; p < kGroup; ++p) {
                if (p < np) {
                    const double g = sP[p * k + j0 + u];
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[p][v] = fma(g, static_cast<double>(v4[u][v]), acc[p][v]);
                }
            }
        }
    }

    float* par = static_cast<float*>(a.parity);
    const int64_t plane = static_cast<int64_t>(npar) * a.qb * a.r;
    // lo plane as bfloat16: after the fp32 hi plane, same element order
    uint16_t* par16 = reinterpret_cast<uint16_t*>(par + plane);
#pragma unroll
    for (int p = 0; p < kGroup; ++p) {
        if (p >= np) break;
        float hi[VEC], lo[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            hi[v] = static_cast<float>(acc[p][v]);
            lo[v] = static_cast<float>(acc[p][v] - static_cast<double>(hi[v]));   // exact remainder, rounded to fp32
        }
        const int64_t off = (static_cast<int64_t>(p0 + p) * a.qb + t) * a.r + c;
        float* dst = par + off;
        if constexpr (VEC == 4) {
            *reinterpret_cast<f32x4e*>(dst) = f32x4e{hi[0], hi[1], hi[2], hi[3]};
            if (a.planes == 2) {
                if (a.lo_bf16) {
                    u32x2e l;
                    l.x = f32_to_bf16_rne(lo[0]) | (static_cast<uint32_t>(f32_to_bf16_rne(lo[1])) << 16);
                    l.y = f32_to_bf16_rne(lo[2]) | (static_cast<uint32_t>(f32_to_bf16_rne(lo[3])) << 16);
                    *reinterpret_cast<u32x2e*>(par16 + off) = l;
                } else {
                    *reinterpret_cast<f32x4e*>(dst + plane) = f32x4e{lo[0], lo[1], lo[2], lo[3]};
                }
            }
        } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                dst[v] = hi[v];
                if (a.planes == 2) {
                    if (a.lo_bf16)
                        par16[off + v] = f32_to_bf16_rne(lo[v]);
                    else
                        dst[plane + v] = lo[v];
                }
            }
        }
    }
}

// bf16: products of two bf16 values are exact in fp32; the k-term sum is
// accumulated in fp32 and split into bf16 hi + lo.
template <int VEC>
__global__ __launch_bounds__(kThreads) void encode_bf16_kernel(EncodeArgs a, int groups, int width) {
    __shared__ float sP[kGroup * kMaxN];
    int64_t t;
    int p0;
    row_and_group(groups, t, p0);
    int lane = threadIdx.x;
    if (width < kThreads) {               // several rows: this thread's row and place in it
        const int per = kThreads / width, row = lane / width;
        t = t * per + row;
        lane = row < per ? lane - row * width : kThreads;
    }
    const int64_t chunk = blockIdx.y;
    const int npar = a.n - a.k;
    const int np = min(kGroup, npar - p0);
    const int k = a.k;
    for (int e = threadIdx.x; e < np * k; e += kThreads) {
        const int p = e / k, j = e % k;
        sP[p * k + j] = static_cast<float>(a.G[(a.k + p0 + p) * k + j]);
    }
    __syncthreads();
    int64_t c = (chunk * kThreads + lane) * VEC;
    if (c >= a.r || t >= a.qb) return;
    c = min(c, a.r - VEC);
    const uint16_t* A = static_cast<const uint16_t*>(a.A);

    float acc[kGroup][VEC];
#pragma unroll
    for (int p = 0; p < kGroup; ++p)
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[p][v] = 0.0f;

    const int kv = static_cast<int>(min<int64_t>(k, (a.q - t + a.qb - 1) / a.qb));   // blocks with row t inside A
    for (int j0 = 0; j0 < kv; j0 += kBatch) {
        float v8[kBatch][VEC];
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int j = min(j0 + u, kv - 1);   // past the last block: re-read it, not used
            const uint16_t* src = A + (static_cast<int64_t>(j) * a.qb + t) * a.lda + c;
            if constexpr (VEC == 8) {
                const u32x4e q4 = *reinterpret_cast<const u32x4e*>(src);
                const uint32_t w[4] = {q4.x, q4.y, q4.z, q4.w};
#pragma unroll
                for (int h = 0; h < 4; ++h) {
                    v8[u][2 * h] = __uint_as_float(w[h] << 16);
                    v8[u][2 * h + 1] = __uint_as_float(w[h] & 0xFFFF0000u);
                }
            } else {
#pragma unroll
                for (int v = 0; v < VEC; ++v) v8[u][v] = bf16_to_f32(src[v]);
            }
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            if (j0 + u >= kv) break;
#pragma unroll
            for (int p = 0; p < kGroup; ++p) {
                if (p < np) {
                    const float g = sP[p * k + j0 + u];
#pragma unroll
                    for (int v = 0; v < VEC; ++v) acc[p][v] = fmaf(g, v8[u][v], acc[p][v]);
                }
            }
        }
    }

    uint16_t* par = static_cast<uint16_t*>(a.parity);
    const int64_t plane = static_cast<int64_t>(npar) * a.qb * a.r;
#pragma unroll
    for (int p = 0; p < kGroup; ++p) {
        if (p >= np) break;
        uint16_t hi[VEC], lo[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            hi[v] = f32_to_bf16_rne(acc[p][v]);
            lo[v] = f32_to_bf16_rne(acc[p][v] - bf16_to_f32(hi[v]));
        }
        uint16_t* dst = par + (static_cast<int64_t>(p0 + p) * a.qb + t) * a.r + c;
        if constexpr (VEC == 8) {
            u32x4e h4, l4;
            h4.x = hi[0] | (uint32_t(hi[1]) << 16); h4.y = hi[2] | (uint32_t(hi[3]) << 16);
            h4.z = hi[4] | (uint32_t(hi[5]) << 16); h4.w = hi[6] | (uint32_t(hi[7]) << 16);
            l4.x = lo[0] | (uint32_t(lo[1]) << 16); l4.y = lo[2] | (uint32_t(lo[3]) << 16);
            l4.z = lo[4] | (uint32_t(lo[5]) << 16); l4.w = lo[6] | (uint32_t(lo[7]) << 16);
            *reinterpret_cast<u32x4e*>(dst) = h4;
            if (a.planes == 2) *reinterpret_cast<u32x4e*>(dst + plane) = l4;
        } else {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                dst[v] = hi[v];
                if (a.planes == 2) dst[plane + v] = lo[v];
            }
        }
    }
}

}  // namespace

hipError_t launch_encode_f32(const EncodeArgs& a, hipStream_t st) {
    const int npar = a.n - a.k;
    if (npar == 0 || a.qb == 0 || a.r == 0) return hipSuccess;
    const int groups = static_cast<int>(ceil_div(npar, kGroup));
    const bool vec = a.r >= 4 && a.qb * a.r * groups > kSingleF32;
    const int V = vec ? 4 : 1;
    const int64_t chunks = ceil_div(a.r, static_cast<int64_t>(kThreads) * V);
    if (chunks > 65535) return hipErrorInvalidConfiguration;
    const int width = row_threads(a.r, V);
    const int64_t rows = ceil_div(a.qb, kThreads / width);
    const int64_t blocks = groups > 1 ? ceil_div(rows, 8) * 8 * groups : rows;
    if (!grid_fits(blocks, kThreads)) return hipErrorInvalidConfiguration;
    dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>(chunks));
    if (vec)
        hipLaunchKernelGGL(encode_f32_kernel<4>, grid, dim3(kThreads), 0, st, a, groups, width);
    else
        hipLaunchKernelGGL(encode_f32_kernel<1>, grid, dim3(kThreads), 0, st, a, groups, width);
    return hipGetLastError();
}

hipError_t launch_encode_bf16(const EncodeArgs& a, hipStream_t st) {
    const int npar = a.n - a.k;
    if (npar == 0 || a.qb == 0 || a.r == 0) return hipSuccess;
    const int groups = static_cast<int>(ceil_div(npar, kGroup));
    const bool vec = a.r >= 8 && a.qb * a.r * groups > kSingleBf16;
    const int V = vec ? 8 : 1;
    const int64_t chunks = ceil_div(a.r, static_cast<int64_t>(kThreads) * V);
    if (chunks > 65535) return hipErrorInvalidConfiguration;
    const int width = row_threads(a.r, V);
    const int64_t rows = ceil_div(a.qb, kThreads / width);
    const int64_t blocks = groups > 1 ? ceil_div(rows, 8) * 8 * groups : rows;
    if (!grid_fits(blocks, kThreads)) return hipErrorInvalidConfiguration;
    dim3 grid(static_cast<unsigned>(blocks), static_cast<unsigned>(chunks));
    if (vec)
        hipLaunchKernelGGL(encode_bf16_kernel<8>, grid, dim3(kThreads), 0, st, a, groups, width);
    else
        hipLaunchKernelGGL(encode_bf16_kernel<1>, grid, dim3(kThreads), 0, st, a, groups, width);
    return hipGetLastError();
}

}  // namespace coded
