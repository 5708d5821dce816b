// bf16 worker products Y_i = A'_i X (Sec. III-A: each worker multiplies its
// stored coded block by the multicast input) on the matrix cores; a vector
// kernel serves rows of fewer than eight elements.
#include "internal.h"

#include "worker_common.h"

namespace coded {
namespace {

// bf16 blocks and X, fp32 accumulation (products of two bf16 values are exact
// in fp32), same work split as gemm_small_f32_kernel.
template <int SC>
__global__ __launch_bounds__(kThreads) void gemm_small_bf16_kernel(WorkerArgs a) {
    int worker;
    int64_t t;
    bool parity;
    if (!wave_task(a, a.qb, a.qb, worker, t, parity)) return;
    const int lane = threadIdx.x & 63;
    const int nplanes = parity ? a.planes : 1;
    const uint16_t* x = static_cast<const uint16_t*>(a.X);
    const int64_t plane = static_cast<int64_t>(a.n - a.k) * a.qb * a.r;
    for (int64_t c0 = 0; c0 < a.s; c0 += SC) {
        float acc[SC];
#pragma unroll
        for (int j = 0; j < SC; ++j) acc[j] = 0.0f;
        for (int h = 0; h < nplanes; ++h) {
            const uint16_t* rowp = nullptr;
            if (!parity) {
                const int64_t row = static_cast<int64_t>(worker) * a.qb + t;
                if (row < a.q) rowp = static_cast<const uint16_t*>(a.A) + row * a.lda;
            } else {
                rowp = static_cast<const uint16_t*>(a.parity) + h * plane +
                       (static_cast<int64_t>(worker - a.k) * a.qb + t) * a.r;
            }
            if (!rowp) continue;
            for (int64_t c = lane; c < a.r; c += 64) {
                const float av = __uint_as_float(static_cast<uint32_t>(rowp[c]) << 16);
                const uint16_t* xr = x + c * a.ldx + c0;
#pragma unroll
                for (int j = 0; j < SC; ++j)
                    if (c0 + j < a.s) acc[j] = fmaf(av, __uint_as_float(static_cast<uint32_t>(xr[j]) << 16), acc[j]);
            }
        }
#pragma unroll
        for (int j = 0; j < SC; ++j) {
            float v = acc[j];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
            acc[j] = v;
        }
        if (lane == 0) {
#pragma unroll
            for (int j = 0; j < SC; ++j)
                if (c0 + j < a.s) store_y(a, worker, t, c0 + j, acc[j]);
        }
    }
}


// ---------------------------------------------------------------- bf16, matrix cores
// Worker products on v_mfma_f32_16x16x32_bf16, fp32 accumulation, for rows of
// any length >= 8, stride and alignment.  Lane layouts (checked on the
// device): A operand lane l element e = A[l%16][8*(l/16)+e], B operand lane l
// element e = B[8*(l/16)+e][l%16], result lane l item v = C[4*(l/16)+v][l%16].
//
// Bound: reading A and the parity planes from HBM once per up to 16 * NT
// columns.  A workgroup of four waves owns 16 * RT row slots of one worker.
// For a systematic worker, or one plane, slot rho is block row t0 + rho; for
// two planes a half of each wave's slots are hi rows and the other half the lo
// rows of the same block rows, whose sums are added at the end, so every
// workgroup streams the same bytes.  K is walked in chunks of KC: a chunk's
// slot rows are loaded 16 bytes per lane, KC / 8 lanes on KC * 2 contiguous
// bytes of a row (two rows x 512 bytes per wave instruction at KC = 256, the
// pattern that streams best), into a ring of PF register sets, then stored to
// a double-buffered LDS tile the A operands are read from.  Rows that start
// at any 2-byte boundary are loaded with the same instruction: 16-byte loads
// at a 4-byte boundary measured 6.7-7.0 TB/s against 7.1 aligned, at a 2-byte
// boundary 4.2-5.8.
//
// X is read straight from its rows: a thread loads eight columns of two
// consecutive k and stores them to LDS as eight k pairs, transposed, so no
// transposed copy of X and no launch for it are needed (that launch took
// 4-10 us per call).
//
// WK = 4: the waves take quarters of each chunk's K range, every wave all
// rows, and the partial sums are added through LDS (a few rows with long K).
// WK = 1: the waves take a quarter of the rows each (many rows, or wide X).
// Either way each 64 k of a wave are summed in fp32 and those sums added in
// fp64: 4.9e-8 off at any length, where one fp32 chain over the matrix
// instructions is 2.3e-7 (r = 5750) to 9e-7 (r = 15040) off.
//
// Loads never leave the operands: positions past the end of a row (or of X)
// are moved back so that the 16 bytes end with the row's last element (X's
// last element), and the tail chunk shifts the values back in place and fills
// with zeros before the LDS store, so whatever lies beyond a row never meets
// the sums.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef u32x4_t u32x4_any __attribute__((aligned(2)));   // 16 bytes at any bf16 boundary

template <int RT, int NT, int KC, int WK>
struct BfCfg {
    static constexpr int kRows = 16 * RT;                  // row slots per workgroup
    static constexpr int kStride = KC + 8;                 // bf16 per LDS row (16-byte pad spreads the banks)
    static constexpr int kABytes = 2 * kRows * kStride * 2;
    static constexpr int kXBytes = 2 * 16 * NT * kStride * 2;
    static constexpr int kRedBytes = 4 * kRows * 16 * 8;   // WK = 4: partial tiles (fp64), 16 columns at a time
    static constexpr int kLds = WK == 4 && kRedBytes > kABytes + kXBytes ? kRedBytes : kABytes + kXBytes;
    static constexpr int kALoads = kRows * (KC / 8) / kThreads;              // per thread and chunk
    static constexpr int kXTasks = (KC / 2 * 2 * NT + kThreads - 1) / kThreads;   // (k pair, 8 columns) per thread and chunk
    static constexpr int kKW = KC / WK;                    // k per wave and chunk
    static constexpr int kRW = RT * WK / 4;                // row tiles per wave
    static constexpr int kFlush = kKW >= 64 ? 1 : 64 / kKW;   // chunks per fp32 partial sum
    static_assert(kRows * (KC / 8) % kThreads == 0, "A tile must split evenly over the threads");
    static_assert(kKW % 32 == 0, "each wave takes whole steps of 32 k");
};

// v moved down by sh elements of 16 bits (0 < sh < 8), zeros above; sh >= 8: zeros; sh <= 0: v.
__device__ inline u32x4_t shift_down(u32x4_t v, int sh) {
    if (sh <= 0) return v;
    uint64_t lo = (static_cast<uint64_t>(v.y) << 32) | v.x, hi = (static_cast<uint64_t>(v.w) << 32) | v.z;
    if (sh >= 8) return u32x4_t{0u, 0u, 0u, 0u};
    if (sh & 4) {
        lo = hi;
        hi = 0;
    }
    const int bits = 16 * (sh & 3);
    if (bits) {
        lo = (lo >> bits) | (hi << (64 - bits));
        hi >>= bits;
    }
    return u32x4_t{static_cast<uint32_t>(lo), static_cast<uint32_t>(lo >> 32), static_cast<uint32_t>(hi),
                   static_cast<uint32_t>(hi >> 32)};
}

// NTL: non-temporal loads of A.
template <int RT, int NT, int KC, int PF, int WK, bool NTL>
__global__ __launch_bounds__(kThreads) void gemm_bf16_mfma_kernel(WorkerArgs a, int64_t stiles, int64_t ptiles,
                                                                  int64_t c0) {
    using C = BfCfg<RT, NT, KC, WK>;
    __shared__ __attribute__((aligned(16))) char smem[C::kLds];
    uint16_t* As = reinterpret_cast<uint16_t*>(smem);                // [2][kRows][kStride]
    uint16_t* Xs = reinterpret_cast<uint16_t*>(smem + C::kABytes);   // [2][16 NT][kStride]
    double* Red = reinterpret_cast<double*>(smem);                   // WK = 4: [4][kRows][16], after the K loop

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lk = lane >> 4;

    // Tile -> (worker, first block row); parity tiles first.
    const int64_t g = blockIdx.x;
    int worker;
    int64_t tile;
    bool parity;
    if (g < ptiles * a.n_par) {
        worker = a.par_ids[g / ptiles];
        tile = g % ptiles;
        parity = true;
    } else {
        const int64_t g2 = g - ptiles * a.n_par;
        if (g2 >= stiles * a.n_sys) return;
        worker = a.sys_ids[g2 / stiles];
        tile = g2 % stiles;
        parity = false;
    }
    const bool pair = parity && a.planes == 2;                // hi and lo rows side by side
    const int64_t t0 = tile * (pair ? C::kRows / 2 : C::kRows);
    constexpr int kSW = 16 * C::kRW;                          // slots of a wave's own rows
    const int r = static_cast<int>(a.r);
    const int nch = (r + KC - 1) / KC;

    const uint16_t* gp[C::kALoads];
    int acol[C::kALoads];
#pragma unroll
    for (int p = 0; p < C::kALoads; ++p) {
        const int f = tid + kThreads * p;
        const int rho = f / (KC / 8);
        acol[p] = (f % (KC / 8)) * 8;
        // Every slot reads a real row (rows past the block a clamped one,
        // whose result is not stored, or stored as the zero padding).
        const int in = rho % kSW, hi = kSW / 2;
        const int plane = pair && in >= hi ? 1 : 0;
        int64_t t = t0 + (pair ? rho / kSW * hi + in % hi : rho);
        t = t < a.qb ? t : a.qb - 1;
        if (parity) {
            gp[p] = static_cast<const uint16_t*>(a.parity) + plane * (static_cast<int64_t>(a.n - a.k) * a.qb * a.r) +
                    (static_cast<int64_t>(worker - a.k) * a.qb + t) * a.r;
        } else {
            int64_t row = static_cast<int64_t>(worker) * a.qb + t;
            row = row < a.q ? row : a.q - 1;
            gp[p] = static_cast<const uint16_t*>(a.A) + row * a.lda;
        }
    }
    const int ncols = static_cast<int>(min<int64_t>(16 * NT, a.s - c0));
    const int xgroups = (ncols + 7) / 8;
    const uint16_t* X = static_cast<const uint16_t*>(a.X);
    const int64_t xlast = (a.r - 1) * a.ldx + a.s - 8;    // last element eight elements can start at
    int xk[C::kXTasks], xc[C::kXTasks];
    bool xlive[C::kXTasks];
#pragma unroll
    for (int i = 0; i < C::kXTasks; ++i) {
        const int e = tid + kThreads * i;
        xk[i] = 2 * (e % (KC / 2));
        xc[i] = 8 * (e / (KC / 2));
        xlive[i] = xc[i] < ncols;                          // absent column groups read a real one, not stored
        xc[i] = xlive[i] ? xc[i] : 8 * (xgroups - 1);
    }

    struct Set {
        u32x4_t A[C::kALoads], X0[C::kXTasks], X1[C::kXTasks];
    };
    // Straight-line loads (a chunk past the last one reads the rows' last pieces).
    auto load_chunk = [&](int c, Set& s) {
#pragma unroll
        for (int p = 0; p < C::kALoads; ++p) {
            const int kk = min(c * KC + acol[p], r - 8);
            const u32x4_any* src = reinterpret_cast<const u32x4_any*>(gp[p] + kk);
            s.A[p] = NTL ? __builtin_nontemporal_load(src) : *src;
        }
#pragma unroll
        for (int i = 0; i < C::kXTasks; ++i) {
            const int64_t o = static_cast<int64_t>(c * KC + xk[i]) * a.ldx + c0 + xc[i];
            s.X0[i] = *reinterpret_cast<const u32x4_any*>(X + min(o, xlast));
            s.X1[i] = *reinterpret_cast<const u32x4_any*>(X + min(o + a.ldx, xlast));
        }
    };
    auto store_x = [&](uint16_t* Xb, int i, u32x4_t v0, u32x4_t v1) {
        uint32_t* d = reinterpret_cast<uint32_t*>(Xb + xc[i] * C::kStride + xk[i]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[(2 * j) * (C::kStride / 2)] = (v0[j] & 0xFFFFu) | (v1[j] << 16);
            d[(2 * j + 1) * (C::kStride / 2)] = (v0[j] >> 16) | (v1[j] & 0xFFFF0000u);
        }
    };
    // A chunk needs care when it reaches past the end of the rows, or when
    // one of its X reads was moved back.
    auto store_chunk = [&](int c, const Set& s) {
        uint16_t* Ab = As + (c & 1) * C::kRows * C::kStride;
        uint16_t* Xb = Xs + (c & 1) * 16 * NT * C::kStride;
        const bool tail = (c + 1) * KC > r ||
                          static_cast<int64_t>(c * KC + KC - 1) * a.ldx + c0 + 8 * (xgroups - 1) > xlast;
        if (!tail) {
#pragma unroll
            for (int p = 0; p < C::kALoads; ++p) {
                const int f = tid + kThreads * p;
                *reinterpret_cast<u32x4_t*>(Ab + (f / (KC / 8)) * C::kStride + acol[p]) = s.A[p];
            }
#pragma unroll
            for (int i = 0; i < C::kXTasks; ++i)
                if (xlive[i]) store_x(Xb, i, s.X0[i], s.X1[i]);
            return;
        }
#pragma unroll
        for (int p = 0; p < C::kALoads; ++p) {
            const int f = tid + kThreads * p;
            *reinterpret_cast<u32x4_t*>(Ab + (f / (KC / 8)) * C::kStride + acol[p]) =
                shift_down(s.A[p], c * KC + acol[p] - (r - 8));
        }
#pragma unroll
        for (int i = 0; i < C::kXTasks; ++i) {
            const int k = c * KC + xk[i];
            const int64_t o = static_cast<int64_t>(k) * a.ldx + c0 + xc[i];
            // k >= r moves everything out only when the row is far past the end: zeroed by k
            const u32x4_t z = {0u, 0u, 0u, 0u};
            const u32x4_t v0 = k < r ? shift_down(s.X0[i], static_cast<int>(min<int64_t>(o - xlast, 8))) : z;
            const u32x4_t v1 = k + 1 < r ? shift_down(s.X1[i], static_cast<int>(min<int64_t>(o + a.ldx - xlast, 8))) : z;
            if (xlive[i]) store_x(Xb, i, v0, v1);
        }
    };

    // fp32 sums of 64 k per wave (two matrix instructions), added up in fp64.
    f32x4_t acc[C::kRW][NT];
    double sum[C::kRW][NT][4];
#pragma unroll
    for (int rt = 0; rt < C::kRW; ++rt)
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            acc[rt][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < 4; ++v) sum[rt][j][v] = 0.0;
        }
    auto flush = [&]() {
#pragma unroll
        for (int rt = 0; rt < C::kRW; ++rt)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
#pragma unroll
                for (int v = 0; v < 4; ++v) sum[rt][j][v] += static_cast<double>(acc[rt][j][v]);
                acc[rt][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            }
    };
    const int kw0 = WK == 4 ? wv * C::kKW : 0;            // the wave's k range in a chunk
    const int rw0 = WK == 4 ? 0 : wv * C::kRW;            // and its row tiles
    auto multiply = [&](int buf) {
        const uint16_t* Ab = As + buf * C::kRows * C::kStride;
        const uint16_t* Xb = Xs + buf * 16 * NT * C::kStride;
#pragma unroll
        for (int ks = 0; ks < C::kKW / 32; ++ks) {
            const int koff = kw0 + 32 * ks + 8 * lk;
            bf16x8 af[C::kRW], bf[NT];
#pragma unroll
            for (int rt = 0; rt < C::kRW; ++rt)
                af[rt] = *reinterpret_cast<const bf16x8*>(Ab + (16 * (rw0 + rt) + li) * C::kStride + koff);
#pragma unroll
            for (int j = 0; j < NT; ++j)
                bf[j] = *reinterpret_cast<const bf16x8*>(Xb + (16 * j + li) * C::kStride + koff);
#pragma unroll
            for (int rt = 0; rt < C::kRW; ++rt)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[rt][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[rt], bf[j], acc[rt][j], 0, 0, 0);
            if (ks & 1) flush();
        }
    };

    Set ring[PF];
#pragma unroll
    for (int j = 0; j < PF; ++j) load_chunk(j, ring[j]);
    for (int cb = 0; cb < nch; cb += PF) {
#pragma unroll
        for (int j = 0; j < PF; ++j) {
            const int c = cb + j;
            if (c >= nch) break;
            store_chunk(c, ring[j]);
            __syncthreads();
            load_chunk(c + PF, ring[j]);
            // keep the scheduler from sinking the loads past the products
            __builtin_amdgcn_sched_barrier(0);
            multiply(c & 1);
            if (C::kFlush > 1 && (c % C::kFlush == C::kFlush - 1 || c == nch - 1)) flush();
        }
    }

    float* Y = static_cast<float*>(a.Y);
    auto put = [&](int64_t t, int col, double v) {
        if (t >= a.qb || col >= ncols) return;
        const int64_t row = static_cast<int64_t>(worker) * a.qb + t;
        // systematic rows past A are the zero padding of the last block
        Y[row * a.s + c0 + col] = parity || row < a.q ? static_cast<float>(v) : 0.0f;
    };
    if constexpr (WK == 1) {
        // Each wave holds whole sums: lane (li, lk) item v of row tile rt is
        // slot 16 rt + 4 lk + v of the wave, column li.  The lo row of a hi
        // row is half the wave's slots further: row tile rt + RW / 2, or with
        // one row tile the lane 32 further.
        constexpr int RW = C::kRW;
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int rt = 0; rt < RW; ++rt)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int slot = 16 * rt + 4 * lk + v;
                    double y = sum[rt][j][v];
                    if (!pair) {
                        put(t0 + wv * kSW + slot, 16 * j + li, y);
                    } else {
                        y += RW == 1 ? __shfl_xor(y, 32, 64) : sum[(rt + RW / 2) % RW][j][v];
                        if (slot < kSW / 2) put(t0 + wv * (kSW / 2) + slot, 16 * j + li, y);
                    }
                }
    } else {
        constexpr int w = C::kRows * 16;
        const int rows = pair ? C::kRows / 2 : C::kRows;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            __syncthreads();   // every wave is done with the tiles (or with the last pass)
#pragma unroll
            for (int rt = 0; rt < C::kRW; ++rt)
#pragma unroll
                for (int v = 0; v < 4; ++v) Red[wv * w + (16 * rt + 4 * lk + v) * 16 + li] = sum[rt][j][v];
            __syncthreads();
            for (int idx = tid; idx < rows * 16; idx += kThreads) {
                double y = (Red[idx] + Red[w + idx]) + (Red[2 * w + idx] + Red[3 * w + idx]);
                if (pair) {
                    const int o = idx + rows * 16;
                    y += (Red[o] + Red[w + o]) + (Red[2 * w + o] + Red[3 * w + o]);
                }
                put(t0 + idx / 16, 16 * j + idx % 16, y);
            }
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

// X transposed, for the single pass.
int64_t worker_workspace_bytes_bf16(int64_t r, int64_t s) { return (r * s * 2 + 255) / 256 * 256; }

// Workgroups of a launch with 16 * RT row slots each.
template <int RT>
static int64_t bf16_blocks(const WorkerArgs& a) {
    return ceil_div(a.qb, 16 * RT) * a.n_sys + ceil_div(a.qb, a.planes == 2 ? 8 * RT : 16 * RT) * a.n_par;
}

template <int RT, int NT, int KC, int PF, int WK, bool NTL>
static hipError_t launch_bf16_mm(const WorkerArgs& a, int64_t c0, hipStream_t st) {
    const int64_t stiles = ceil_div(a.qb, 16 * RT);
    const int64_t ptiles = ceil_div(a.qb, a.planes == 2 ? 8 * RT : 16 * RT);
    const int64_t blocks = stiles * a.n_sys + ptiles * a.n_par;
    if (blocks == 0) return hipSuccess;
    if (!grid_fits(blocks, kThreads)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemm_bf16_mfma_kernel<RT, NT, KC, PF, WK, NTL>), dim3(static_cast<unsigned>(blocks)),
                       dim3(kThreads), 0, st, a, stiles, ptiles, c0);
    return hipGetLastError();
}

hipError_t launch_worker_bf16(const WorkerArgs& a, hipStream_t st) {
    if (a.qb == 0 || a.s == 0) return hipSuccess;
    // rows shorter than one 16-byte piece (and empty A, or K past 32 bits)
    if (a.r < 8 || a.r > (1ll << 30) || a.q == 0) return launch_waves(gemm_small_bf16_kernel<4>, a, a.qb, a.qb, st);
    // Operands past the memory-side cache stream faster with non-temporal loads
    // (1.2 GB with 4 columns: 182 us against 200); below, plain loads find them
    // there (155 MB with 16 columns: 28 us against 35).
    const bool stream = a.stream;
    for (int64_t c0 = 0; c0 < a.s; c0 += 64) {
        const int64_t cols = std::min<int64_t>(64, a.s - c0);
        hipError_t e;
        // Tiles by columns, row length and how many workgroups come out.
        // Short rows: 64-k chunks, rows split over the waves (five-block code,
        // 300000 x 200, 16 columns: 77 us against 114 with 256-k chunks; r =
        // 1200: 20 and 20).  Long rows: a chunk of a row is 256 or 512 bytes.
        // Few workgroups: smaller tiles that split K over the waves (2000 x
        // 16000, 64 columns, 24 workgroups of 128 rows: 102 us against 185;
        // 16384 x 4096, 192 of them: 72 against 57).  Wide X keeps 64-k chunks,
        // whose 128 rows read X least often; a third chunk in flight pays from
        // r = 1024 on (131072 x 4096: 392 us against 406; r = 300: 30 and 29).
        if (cols > 32) {
            if (bf16_blocks<8>(a) < 128)
                e = launch_bf16_mm<2, 4, 128, 3, 4, false>(a, c0, st);
            else
                e = a.r <= 1024 ? launch_bf16_mm<8, 4, 64, 2, 1, false>(a, c0, st)
                                : launch_bf16_mm<8, 4, 64, 3, 1, false>(a, c0, st);
        } else if (cols > 16) {
            if (a.r <= 512)
                e = launch_bf16_mm<4, 2, 64, 2, 1, false>(a, c0, st);
            else if (bf16_blocks<4>(a) < 128)
                e = launch_bf16_mm<2, 2, 256, 2, 4, false>(a, c0, st);
            else
                e = stream ? launch_bf16_mm<4, 2, 128, 2, 1, true>(a, c0, st)
                           : launch_bf16_mm<4, 2, 128, 2, 1, false>(a, c0, st);
        } else {
            if (a.r <= 1024)
                e = launch_bf16_mm<4, 1, 64, 2, 1, false>(a, c0, st);
            else if (bf16_blocks<2>(a) < 256)
                e = launch_bf16_mm<1, 1, 512, 2, 4, false>(a, c0, st);
            else
                e = stream ? launch_bf16_mm<2, 1, 256, 2, 4, true>(a, c0, st)
                           : launch_bf16_mm<2, 1, 256, 2, 4, false>(a, c0, st);
        }
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace coded
