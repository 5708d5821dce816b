// Worker products Y_i = A'_i X for the simulated workers (Sec. III-A: each
// worker multiplies its stored coded block by the multicast input).
//
// All n blocks are served by one launch.  A systematic block is a window of A
// itself (rows i*qb .. i*qb+qb-1; rows at or beyond q are the zero padding and
// are never read).  A parity block is `planes` planes (hi, lo) in the parity
// buffer; its product is sum_h plane_h X.
//
// The single-vector case (s == 1) is the HBM-bound GEMV: every byte of A and
// of the parity planes is read exactly once, in 16-byte loads that a whole
// workgroup issues over one contiguous stretch of a long row at a time
// (streaming long rows through single wavefronts measurably loses bandwidth);
// short rows go to 16 or 64 lanes each.  Rows start at any fp32 boundary and
// have any length ((25,23) on 11500 x 5750: 52 us, 6.0 TB/s; scalar loads took
// 154).  Products of two fp32 values are exact in fp64 and are summed in fp64.
// s > 1 runs on the fp64 matrix cores (worker_f32_mfma.hip); what that cannot
// take runs a general vector kernel.
#include <type_traits>

#include "internal.h"
#include "worker_common.h"

namespace coded {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Four values from any fp32 boundary: 16-byte loads at a 4-byte boundary run
// at 6.7-6.9 TB/s against 7.1 aligned (scalar loads of the same rows: 5.5).
// NTL: non-temporal, for data that no later call finds in a cache.
typedef f32x4 f32x4_any __attribute__((aligned(4)));
template <bool NTL>
__device__ inline float4 load4(const float* p) {
    // a global-memory pointer, so the load is a global (not flat) load
    typedef const __attribute__((address_space(1))) f32x4_any* gptr;
    const f32x4 v = NTL ? __builtin_nontemporal_load((gptr)(p)) : *(gptr)(p);
    return make_float4(v.x, v.y, v.z, v.w);
}

// Four bfloat16 values (8 bytes, any bf16 boundary) as raw bits, and their
// exact widening to fp32 (kept apart so a select can take the raw load).
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_any __attribute__((aligned(2)));
template <bool NTL>
__device__ inline u32x2 load_bf16x4(const uint16_t* p) {
    typedef const __attribute__((address_space(1))) u32x2_any* gptr;
    return NTL ? __builtin_nontemporal_load((gptr)(p)) : *(gptr)(p);
}
__device__ inline float4 widen_bf16x4(u32x2 v) {
    return make_float4(__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u),
                       __uint_as_float(v.y << 16), __uint_as_float(v.y & 0xFFFF0000u));
}

__device__ inline float bf16_bits_to_f32(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// First element of the lo plane when it is stored as bfloat16: directly after
// the fp32 hi plane, in the same (worker, block row, column) order.
__device__ inline const uint16_t* lo16_base(const WorkerArgs& a) {
    return reinterpret_cast<const uint16_t*>(static_cast<const float*>(a.parity) +
                                             static_cast<int64_t>(a.n - a.k) * a.qb * a.r);
}

struct RowRef {
    const float* ptr;     // start of the plane row (null: zero padding / out of range)
    const uint16_t* p16;  // instead of ptr for a bfloat16 lo plane
    int64_t t;            // block row
};

// Plane row `pr` of worker `w`.
__device__ inline RowRef plane_row(const WorkerArgs& a, int w, int64_t pr, bool parity) {
    RowRef rr{nullptr, nullptr, 0};
    if (!parity) {
        rr.t = pr;
        const int64_t row = static_cast<int64_t>(w) * a.qb + pr;
        if (pr < a.qb && row < a.q) rr.ptr = static_cast<const float*>(a.A) + row * a.lda;
    } else {
        const int64_t t = pr / a.planes;
        const int h = static_cast<int>(pr % a.planes);
        rr.t = t;
        if (t < a.qb) {
            const int64_t plane = static_cast<int64_t>(a.n - a.k) * a.qb * a.r;
            const int64_t off = (static_cast<int64_t>(w - a.k) * a.qb + t) * a.r;
            if (h == 1 && a.lo_bf16)
                rr.p16 = lo16_base(a) + off;
            else
                rr.ptr = static_cast<const float*>(a.parity) + h * plane + off;
        }
    }
    return rr;
}

// s == 1, 16-byte vectors.  A workgroup of NT threads owns a tile of T
// consecutive rows of one worker's block and sweeps it one row at a time:
// thread tid covers column slots c = tid*4 + j*NT*4 (j < XR) of every row, so
// each load instruction of the workgroup reads NT*16 contiguous bytes, and
// its slice of x stays in registers for all T rows.  Rows wider than
// NT*4*XR are swept in column chunks (x reloaded per chunk).  A parity row's
// planes (hi, lo) are summed into the same fp64 accumulator.  Partial sums
// are combined across lanes (shuffles) and waves (LDS) in a fixed order.
// LO16: the lo plane is bfloat16 (8-byte loads of four values, widened
// exactly to fp32, so the products stay exact in fp64).
// TAIL: r is no multiple of 4; the last r % 4 elements go to the first threads.
template <int T, int XR, int NT, bool LO16, bool NTL, bool TAIL>
__global__ __launch_bounds__(NT) void gemv_wg_kernel(WorkerArgs a) {
    constexpr int NW = NT / 64;
    constexpr int kChunk = NT * 4 * XR;
    __shared__ double red[NW][T];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // The arguments the first loads depend on, fetched in one batch and held
    // in scalar registers (left alone, the compiler fetches them one
    // dependent round trip after another, inside the branches that use them).
    const float* Ap = static_cast<const float*>(a.A);
    const float* Pp = static_cast<const float*>(a.parity);
    const float* x = static_cast<const float*>(a.X);
    int64_t q = a.q, r = a.r, lda = a.lda, qb = a.qb;
    int32_t n = a.n, k = a.k, planes = a.planes, n_sys = a.n_sys, n_par = a.n_par;
    asm volatile("" : "+s"(Ap), "+s"(Pp), "+s"(x), "+s"(q), "+s"(r), "+s"(lda), "+s"(qb), "+s"(n), "+s"(k),
                 "+s"(planes), "+s"(n_sys), "+s"(n_par));
    // The grid has fewer than 2^31 workgroups (checked at launch), so the
    // tile arithmetic fits 32 bits.
    const uint32_t groups = static_cast<uint32_t>(ceil_div(qb, T));
    const uint32_t npar = groups * static_cast<uint32_t>(n_par);
    const uint32_t g = blockIdx.x;
    int worker;
    int64_t grp;
    bool parity;
    // Parity workgroups stream `planes` times the bytes: dispatch them first so
    // the launch does not end on a tail of long workgroups.  With every worker
    // active (the usual case) the worker follows from the index; otherwise
    // from the lists of active workers.
    if (g < npar) {
        const uint32_t wi = g / groups;
        worker = n_par == n - k ? k + static_cast<int>(wi) : a.par_ids[wi];
        grp = g - wi * groups;
        parity = true;
    } else {
        if (g - npar >= groups * static_cast<uint32_t>(n_sys)) return;
        const uint32_t wi = (g - npar) / groups;
        worker = n_sys == k ? static_cast<int>(wi) : a.sys_ids[wi];
        grp = (g - npar) - wi * groups;
        parity = false;
    }
    const int64_t t0 = grp * T;
    const int nplanes = parity ? planes : 1;
    const int64_t plane = static_cast<int64_t>(n - k) * qb * r;

    // Row pointers of the tile (null: padding row or beyond the block).
    const float* rows[T][2];
    const uint16_t* lo16[T];
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int64_t t = t0 + i;
        rows[i][0] = rows[i][1] = nullptr;
        lo16[i] = nullptr;
        if (t >= qb) continue;
        if (!parity) {
            const int64_t rr = static_cast<int64_t>(worker) * qb + t;
            if (rr < q) rows[i][0] = Ap + rr * lda;
        } else {
            const int64_t off = (static_cast<int64_t>(worker - k) * qb + t) * r;
            const float* base = Pp + off;
            rows[i][0] = base;
            if (nplanes == 2) {
                if constexpr (LO16)
                    lo16[i] = reinterpret_cast<const uint16_t*>(Pp + plane) + off;
                else
                    rows[i][1] = base + plane;
            }
        }
    }

    double acc[T];
#pragma unroll
    for (int i = 0; i < T; ++i) acc[i] = 0.0;

    const int64_t r4 = TAIL ? r & ~int64_t{3} : r;
    for (int64_t cb = 0; cb < r4; cb += kChunk) {
        float4 xv[XR];
#pragma unroll
        for (int j = 0; j < XR; ++j) {
            const int64_t c = cb + tid * 4 + j * NT * 4;
            xv[j] = c < r4 ? load4<false>(x + c) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int i = 0; i < T; ++i) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float* row = rows[i][h];
                const bool bf = LO16 && h == 1;
                if (bf ? !lo16[i] : !row) continue;
                float4 av[XR];
#pragma unroll
                for (int j = 0; j < XR; ++j) {
                    const int64_t c = cb + tid * 4 + j * NT * 4;
                    // selects, not branches, so the loads stay in flight together
                    if constexpr (LO16) {
                        if (h == 1) continue;
                    }
                    av[j] = c < r4 ? load4<NTL>(row + c) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
                if constexpr (LO16) {
                    if (h == 1) {
                        u32x2 raw[XR];
#pragma unroll
                        for (int j = 0; j < XR; ++j) {
                            const int64_t c = cb + tid * 4 + j * NT * 4;
                            raw[j] = c < r4 ? load_bf16x4<NTL>(lo16[i] + c) : u32x2{0u, 0u};
                        }
#pragma unroll
                        for (int j = 0; j < XR; ++j) av[j] = widen_bf16x4(raw[j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < XR; ++j) {
                    acc[i] = fma(static_cast<double>(av[j].x), static_cast<double>(xv[j].x), acc[i]);
                    acc[i] = fma(static_cast<double>(av[j].y), static_cast<double>(xv[j].y), acc[i]);
                    acc[i] = fma(static_cast<double>(av[j].z), static_cast<double>(xv[j].z), acc[i]);
                    acc[i] = fma(static_cast<double>(av[j].w), static_cast<double>(xv[j].w), acc[i]);
                }
            }
        }
    }
    if constexpr (TAIL) {
        if (tid < static_cast<int>(r - r4)) {
            const double xt = x[r4 + tid];
#pragma unroll
            for (int i = 0; i < T; ++i) {
                if (rows[i][0]) acc[i] = fma(static_cast<double>(rows[i][0][r4 + tid]), xt, acc[i]);
                if (rows[i][1]) acc[i] = fma(static_cast<double>(rows[i][1][r4 + tid]), xt, acc[i]);
                if (LO16 && lo16[i]) acc[i] = fma(static_cast<double>(bf16_bits_to_f32(lo16[i][r4 + tid])), xt, acc[i]);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const double v = wave_sum(acc[i]);
        if (lane == 0) red[wv][i] = v;
    }
    __syncthreads();
    if (tid < T) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < NW; ++w) v += red[w][tid];
        const int64_t t = t0 + tid;
        if (t < a.qb) store_y(a, worker, t, 0, v);
    }
}

// s == 1, short rows (r <= 16 * LPR): LPR lanes (16 or 64) per row, so a row
// of a few hundred elements does not leave most of a workgroup idle (r = 400:
// 100 of 256 threads in the kernel above; a (10,8) code on 10000 x 400 13.6 us
// there, 5.7 here; 60000 x 256 50 and 16.5 us, 5.6 TB/s), and the sum of a row
// stays inside a wave.  A group of LPR lanes owns T consecutive rows of one worker's block,
// all their loads in flight at once; its slice of x (XR pieces of four, XR * 4
// * LPR >= r) stays in registers.  Rows past the block, or past A, read the
// last row and are not stored, or stored as the zero padding, so there is no
// branch between the loads.
template <int T, int XR, int LPR, bool LO16, bool NTL, bool TAIL>
__global__ __launch_bounds__(256) void gemv_short_kernel(WorkerArgs a) {
    constexpr int kGroups = 256 / LPR, kTile = kGroups * T;
    const int tid = threadIdx.x;
    const int l = tid % LPR;
    const int gi = LPR == 64 ? __builtin_amdgcn_readfirstlane(tid / LPR) : tid / LPR;
    const float* Ap = static_cast<const float*>(a.A);
    const float* Pp = static_cast<const float*>(a.parity);
    const float* x = static_cast<const float*>(a.X);
    int64_t q = a.q, lda = a.lda, qb = a.qb;
    int32_t r = static_cast<int32_t>(a.r), n = a.n, k = a.k, planes = a.planes, n_sys = a.n_sys, n_par = a.n_par;
    // one batch of scalar loads, as above
    asm volatile("" : "+s"(Ap), "+s"(Pp), "+s"(x), "+s"(q), "+s"(r), "+s"(lda), "+s"(qb), "+s"(n), "+s"(k),
                 "+s"(planes), "+s"(n_sys), "+s"(n_par));
    // parity workgroups (twice the bytes) first
    const uint32_t groups = static_cast<uint32_t>(ceil_div(qb, kTile));
    const uint32_t npar = groups * static_cast<uint32_t>(n_par);
    const uint32_t g = blockIdx.x;
    const bool parity = g < npar;
    const uint32_t g2 = parity ? g : g - npar;
    const uint32_t wi = g2 / groups;
    if (!parity && wi >= static_cast<uint32_t>(n_sys)) return;
    int worker;
    if (parity)
        worker = n_par == n - k ? k + static_cast<int>(wi) : a.par_ids[wi];
    else
        worker = n_sys == k ? static_cast<int>(wi) : a.sys_ids[wi];
    const int64_t t0 = static_cast<int64_t>(g2 - wi * groups) * kTile + gi * T;
    const int64_t plane = static_cast<int64_t>(n - k) * qb * r;

    const float* row[T];
    int64_t off[T];            // parity: element offset of the row in a plane
#pragma unroll
    for (int i = 0; i < T; ++i) {
        const int64_t t = min(t0 + i, qb - 1);
        off[i] = parity ? (static_cast<int64_t>(worker - k) * qb + t) * r : 0;
        row[i] = parity ? Pp + off[i] : Ap + min(static_cast<int64_t>(worker) * qb + t, q - 1) * lda;
    }
    const int r4 = TAIL ? r & ~3 : r;
    const int rem = r - r4;
    float4 xv[XR];
    float xt = 0.f;
#pragma unroll
    for (int j = 0; j < XR; ++j) {
        const int c = (l + j * LPR) * 4;
        xv[j] = c < r4 ? load4<false>(x + c) : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    if (TAIL && l < rem) xt = x[r4 + l];

    double acc[T];
#pragma unroll
    for (int i = 0; i < T; ++i) acc[i] = 0.0;
    auto add = [&](const float4 (&v)[T][XR], const float (&vt)[T]) {
#pragma unroll
        for (int i = 0; i < T; ++i) {
#pragma unroll
            for (int j = 0; j < XR; ++j) {
                acc[i] = fma(static_cast<double>(v[i][j].x), static_cast<double>(xv[j].x), acc[i]);
                acc[i] = fma(static_cast<double>(v[i][j].y), static_cast<double>(xv[j].y), acc[i]);
                acc[i] = fma(static_cast<double>(v[i][j].z), static_cast<double>(xv[j].z), acc[i]);
                acc[i] = fma(static_cast<double>(v[i][j].w), static_cast<double>(xv[j].w), acc[i]);
            }
            if (TAIL) acc[i] = fma(static_cast<double>(vt[i]), static_cast<double>(xt), acc[i]);
        }
    };
    auto sweep = [&](int64_t shift) {
        float4 v[T][XR];
        float vt[T];
#pragma unroll
        for (int j = 0; j < XR; ++j) {
            const int c = (l + j * LPR) * 4;
#pragma unroll
            for (int i = 0; i < T; ++i)
                v[i][j] = c < r4 ? load4<NTL>(row[i] + shift + c) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int i = 0; i < T; ++i) vt[i] = TAIL && l < rem ? row[i][shift + r4 + l] : 0.f;
        add(v, vt);
    };
    sweep(0);
    if (parity && planes == 2) {
        if constexpr (LO16) {
            const uint16_t* lo = reinterpret_cast<const uint16_t*>(Pp + plane);
            u32x2 raw[T][XR];
            float4 v[T][XR];
            float vt[T];
#pragma unroll
            for (int j = 0; j < XR; ++j) {
                const int c = (l + j * LPR) * 4;
#pragma unroll
                for (int i = 0; i < T; ++i) raw[i][j] = c < r4 ? load_bf16x4<NTL>(lo + off[i] + c) : u32x2{0u, 0u};
            }
#pragma unroll
            for (int i = 0; i < T; ++i) {
                vt[i] = TAIL && l < rem ? bf16_bits_to_f32(lo[off[i] + r4 + l]) : 0.f;
#pragma unroll
                for (int j = 0; j < XR; ++j) v[i][j] = widen_bf16x4(raw[i][j]);
            }
            add(v, vt);
        } else {
            sweep(plane);
        }
    }
#pragma unroll
    for (int i = 0; i < T; ++i) {
#pragma unroll
        for (int o = LPR / 2; o >= 1; o >>= 1) acc[i] += __shfl_xor(acc[i], o, 64);
    }
    if (l == 0) {
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int64_t t = t0 + i;
            if (t >= qb) break;
            const bool inside = parity || static_cast<int64_t>(worker) * qb + t < q;
            store_y(a, worker, t, 0, inside ? acc[i] : 0.0);
        }
    }
}

// General shapes (any r, s, strides): one block row per wave (all planes of a
// parity row), scalar loads, columns of X in groups of SC.  Used with several
// columns for what the matrix-core kernel does not take: rows of fewer than four
// elements or more than 2^30, and a bfloat16 lo plane.
template <int SC>
__global__ __launch_bounds__(kThreads) void gemm_small_f32_kernel(WorkerArgs a) {
    int worker;
    int64_t t;
    bool parity;
    if (!wave_task(a, a.qb, a.qb, worker, t, parity)) return;
    const int lane = threadIdx.x & 63;
    const int nplanes = parity ? a.planes : 1;
    const float* x = static_cast<const float*>(a.X);
    for (int64_t c0 = 0; c0 < a.s; c0 += SC) {
        double acc[SC];
#pragma unroll
        for (int j = 0; j < SC; ++j) acc[j] = 0.0;
        for (int h = 0; h < nplanes; ++h) {
            const RowRef rr = plane_row(a, worker, parity ? t * a.planes + h : t, parity);
            if (!rr.ptr && !rr.p16) continue;
            for (int64_t c = lane; c < a.r; c += 64) {
                const double av = rr.p16 ? bf16_bits_to_f32(rr.p16[c]) : rr.ptr[c];
                const float* xr = x + c * a.ldx + c0;
#pragma unroll
                for (int j = 0; j < SC; ++j)
                    if (c0 + j < a.s) acc[j] = fma(av, static_cast<double>(xr[j]), acc[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < SC; ++j) acc[j] = wave_sum(acc[j]);
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < SC; ++j)
                if (c0 + j < a.s) store_y(a, worker, t, c0 + j, acc[j]);
        }
    }
}

template <typename K>
hipError_t launch_waves(K kernel, const WorkerArgs& a, int64_t wsys, int64_t wpar, hipStream_t st) {
    const int64_t waves = wsys * a.n_sys + wpar * a.n_par;
    if (waves == 0) return hipSuccess;
    const int64_t blocks = ceil_div(waves, kWaves);
    if (!grid_fits(blocks, kThreads)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), 0, st, a);
    return hipGetLastError();
}

}  // namespace

template <int T, int XR, bool LO16, bool NTL, bool TAIL>
static hipError_t launch_gemv_v(const WorkerArgs& a, hipStream_t st) {
    const int64_t blocks = ceil_div(a.qb, T) * (a.n_sys + a.n_par);
    if (blocks == 0) return hipSuccess;
    if (!grid_fits(blocks, 256)) return hipErrorInvalidConfiguration;
    // Rows of 8 column slots per thread that stream from HBM: at most three
    // workgroups per compute unit (each requests 40 KB of the 160 KB of LDS,
    // which it does not use), which streams these long rows best (measured:
    // two, three and four; 65536 x 8192: 521.8 us against 524.1 without).
    // From the memory-side cache the limit costs (1472 x 7307: 12.5 us
    // against 10.7).  Rows of 6 slots want it when whole and well filled
    // ((4,2), 420 and 840 MB of A: r = 5752 452 and 909 us against 472 and 950,
    // r = 5000 449 against 467), not with a remainder (r = 5750: 519 against
    // 467) nor near 4 slots ((16,12), r = 4352: 252 against 247).
    const bool whole6 = XR == 6 && !TAIL && a.r > 4608;
    const size_t cap = NTL && (XR >= 8 || whole6) ? 40 * 1024 : 0;
    hipLaunchKernelGGL((gemv_wg_kernel<T, XR, 256, LO16, NTL, TAIL>), dim3(static_cast<unsigned>(blocks)), dim3(256),
                       cap, st, a);
    return hipGetLastError();
}

template <int T, int XR, int LPR, bool LO16, bool NTL, bool TAIL>
static hipError_t launch_short_v(const WorkerArgs& a, hipStream_t st) {
    const int64_t blocks = ceil_div(a.qb, 256 / LPR * T) * (a.n_sys + a.n_par);
    if (blocks == 0) return hipSuccess;
    if (!grid_fits(blocks, 256)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemv_short_kernel<T, XR, LPR, LO16, NTL, TAIL>), dim3(static_cast<unsigned>(blocks)), dim3(256),
                       0, st, a);
    return hipGetLastError();
}

// The plane format, the tail and the cache policy as template arguments.
// Non-temporal loads where the operands are streamed (65536 x 8192: 522 us
// against 587 with plain loads).
template <int T, int XR, int LPR>
static hipError_t launch_gemv_any(const WorkerArgs& a, hipStream_t st) {
    const bool lo16 = a.lo_bf16 && a.planes == 2, tail = a.r % 4 != 0;
    const bool ntl = a.stream;
    auto go = [&](auto lo, auto nt, auto tl) {
        constexpr bool L = decltype(lo)::value, N = decltype(nt)::value, TL = decltype(tl)::value;
        if constexpr (LPR == 256)
            return launch_gemv_v<T, XR, L, N, TL>(a, st);
        else
            return launch_short_v<T, XR, LPR, L, N, TL>(a, st);
    };
    auto go2 = [&](auto lo, auto nt) { return tail ? go(lo, nt, std::true_type{}) : go(lo, nt, std::false_type{}); };
    auto go3 = [&](auto lo) { return ntl ? go2(lo, std::true_type{}) : go2(lo, std::false_type{}); };
    return lo16 ? go3(std::true_type{}) : go3(std::false_type{});
}

template <int XR, int LPR>
static hipError_t launch_gemv_t(const WorkerArgs& a, hipStream_t st) {
    // Four rows per workgroup, or group of lanes (x is read once per four
    // rows), unless that leaves fewer than four workgroups per compute unit
    // (256 CUs); then fewer.
    const int64_t workers = a.n_sys + a.n_par;
    constexpr int G = 256 / LPR;
    if (ceil_div(a.qb, 4 * G) * workers >= 1024) return launch_gemv_any<4, XR, LPR>(a, st);
    if (ceil_div(a.qb, 2 * G) * workers >= 1024) return launch_gemv_any<2, XR, LPR>(a, st);
    return launch_gemv_any<1, XR, LPR>(a, st);
}

hipError_t launch_worker_f32(const WorkerArgs& a, hipStream_t st) {
    if (a.qb == 0) return hipSuccess;
    if (a.s == 1 && a.ldx == 1) {
        // Column slots per thread: the whole row in registers up to 8192
        // columns.  Rows of up to 1024 are short: a row per 16 or 64 lanes.
        // Six slots up to 6144 (eight leave a third of them idle: 11500 x
        // 5750 52 us against 62, 20000 x 4097 92 against 102).
        if (a.r > 6144) return launch_gemv_t<8, 256>(a, st);
        if (a.r > 4096) return launch_gemv_t<6, 256>(a, st);
        if (a.r > 2048) return launch_gemv_t<4, 256>(a, st);
        if (a.r > 1024) return launch_gemv_t<2, 256>(a, st);
        if (a.r > 512) return launch_gemv_t<4, 64>(a, st);
        if (a.r > 256) return launch_gemv_t<2, 64>(a, st);
        if (a.r > 128) return launch_gemv_t<4, 16>(a, st);
        if (a.r > 64) return launch_gemv_t<2, 16>(a, st);
        return launch_gemv_t<1, 16>(a, st);
    }
    if (gemm_f32_mfma_supported(a)) return launch_gemm_f32_mfma(a, st);
    return launch_waves(gemm_small_f32_kernel<4>, a, a.qb, a.qb, st);
}

}  // namespace coded
