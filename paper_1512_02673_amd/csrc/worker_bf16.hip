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
typedef f32x4_t f32x4_any __attribute__((aligned(4)));   // 16 bytes at any fp32 boundary

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

// Results of a matrix instruction whose first operand is X^T: lane (li, lk) holds
// columns 4 lk .. 4 lk + 3 of a 16-column tile for row li of a 16-row tile.
struct TileOut {
    const WorkerArgs& a;
    int64_t c0;
    int worker, ncols;
    bool parity;

    // columns c0 + col .. of row t of the block (those below c0 + ncols)
    __device__ __forceinline__ void row(int64_t t, int col, f32x4_t o) const {
        const int64_t at = static_cast<int64_t>(worker) * a.qb + t;
        if (t >= a.qb) return;
        if (!parity && at >= a.q) o = f32x4_t{0.f, 0.f, 0.f, 0.f};   // past A: the zero padding of the last block
        float* y = static_cast<float*>(a.Y) + at * a.s + c0 + col;
        if (col + 4 <= ncols) {
            *reinterpret_cast<f32x4_any*>(y) = o;
        } else {
#pragma unroll
            for (int w = 0; w < 3; ++w)
                if (col + w < ncols) y[w] = o[w];
        }
    }
    // column tiles j and j + 1 of the rows from t: the lanes of rows 2 i and
    // 2 i + 1 trade one each, so that a store writes 32 columns (128 bytes) of
    // eight rows ((20,16), 4.9 M rows of 64, 64 columns: 442 us against 488)
    __device__ __forceinline__ void two(int64_t t, int j, f32x4_t o0, f32x4_t o1) const {
        const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
        const bool odd = li & 1;
        const f32x4_t give = odd ? o0 : o1;
        f32x4_t got;
#pragma unroll
        for (int w = 0; w < 4; ++w)
            got[w] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(give[w]), 0xB1, 0xF, 0xF, true));   // lane ^ 1
        row(t + (li & ~1), 16 * (j + odd) + 4 * lk, odd ? got : o0);
        row(t + (li | 1), 16 * (j + odd) + 4 * lk, odd ? o1 : got);
    }
    // a row tile's NT column tiles from tile j0
    template <int NT>
    __device__ __forceinline__ void tile(int64_t t, int j0, const f32x4_t (&o)[NT]) const {
        const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
#pragma unroll
        for (int j = 0; j < NT; j += 2) {
            if (NT > 1 && 16 * (j0 + j + 1) < ncols)
                two(t, j0 + j, o[j], o[NT > 1 ? j + 1 : 0]);
            else
                row(t + li, 16 * (j0 + j) + 4 * lk, o[j]);
        }
    }
};

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
                    acc[rt][j] = WK == 1 ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j], af[rt], acc[rt][j], 0, 0, 0)
                                         : __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[rt], bf[j], acc[rt][j], 0, 0, 0);
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

    if constexpr (WK == 1) {
        // Each wave holds whole sums: lane (li, lk) item v of row tile rt is
        // slot 16 rt + li of the wave, column 4 lk + v.  The lo row of a hi row
        // is half the wave's slots further: row tile rt + RW / 2, or with one
        // row tile the lane 8 further.
        constexpr int RW = C::kRW;
        const TileOut out{a, c0, worker, ncols, parity};
#pragma unroll
        for (int rt = 0; rt < RW; ++rt) {
            f32x4_t o[NT];
            if (!pair) {
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) o[j][v] = static_cast<float>(sum[rt][j][v]);
                out.tile(t0 + wv * kSW + 16 * rt, 0, o);
            } else if (RW == 1 || rt < RW / 2) {
#pragma unroll
                for (int j = 0; j < NT; ++j)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const double lo = RW == 1 ? __shfl_xor(sum[rt][j][v], 8, 64) : sum[(rt + RW / 2) % RW][j][v];
                        o[j][v] = static_cast<float>(sum[rt][j][v] + lo);
                    }
                // with one row tile, rows 8 .. 15 are the lo rows: moved past the block, so not stored
                out.tile(RW == 1 && li >= 8 ? a.qb : t0 + wv * (kSW / 2) + 16 * rt, 0, o);
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
                const int64_t t = t0 + idx / 16, row = static_cast<int64_t>(worker) * a.qb + t;
                const int col = 16 * j + idx % 16;
                // systematic rows past A are the zero padding of the last block
                if (t < a.qb && col < ncols)
                    static_cast<float*>(a.Y)[row * a.s + c0 + col] = parity || row < a.q ? static_cast<float>(y) : 0.0f;
            }
        }
    }
}

// Short rows (up to 384 elements, whole 16-byte pieces): one step of K, so a
// workgroup of the kernel above would stage X for every 64 or 128 rows and wait
// for its few loads with nothing to overlap them.  Here eight waves take two
// tiles of 16 row slots each (of a two-plane parity row: its hi and its lo
// rows).  X's pieces, then every A operand straight from memory (16 bytes a lane,
// 64 of a row per instruction, the other half of a line by the next one, which a
// non-temporal load would evict first) are in flight before anything is used; X
// goes to LDS transposed, and an operand read back serves both tiles.
//
// The operands are swapped (X^T is the first), so a lane's four results are
// consecutive columns of one row and go out in one store.  Sums as above: fp32
// over 64 k, those added in fp64, the lo plane's to the hi plane's at the end.
template <int NT, int KS>
struct ShortCfg {
    // four waves a SIMD (128 registers), three (168) where the operands need more
    static constexpr int kWaves = KS > 8 ? 3 : 4, kThreads = kWaves * 128;
    static constexpr int kSlots = kThreads / 64 * 32;          // row slots per workgroup
    // Column tiles summed and stored together: a tile's fp32 sums take 4 KS
    // registers, the A operands 8 KS.
    static constexpr int kTilesAtOnce = KS <= 4 || NT == 1 ? NT : (KS * NT > 24 ? 1 : 2);
};

template <int NT, int KS>
__global__ __launch_bounds__((ShortCfg<NT, KS>::kThreads), (ShortCfg<NT, KS>::kWaves)) void gemm_bf16_short_kernel(WorkerArgs a, int64_t stiles, int64_t ptiles,
                                                                           int64_t c0) {
    constexpr int K = 32 * KS, kStride = K + 8;               // 16-byte pad: spreads the banks
    constexpr int kThr = ShortCfg<NT, KS>::kThreads, kSlots = ShortCfg<NT, KS>::kSlots, JB = ShortCfg<NT, KS>::kTilesAtOnce;
    constexpr int kXTasks = (K / 2 * 2 * NT + kThr - 1) / kThr;   // (k pair, 8 columns) per thread
    static_assert(KS % 2 == 0, "whole sums of 64 k");
    __shared__ __attribute__((aligned(16))) uint16_t sX[16 * NT * kStride];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int li = lane & 15, lk = lane >> 4;
    const int r = static_cast<int>(a.r);

    // Tile -> (worker, first block row); parity tiles first.
    const int64_t g = blockIdx.x;
    const bool parity = g < ptiles * a.n_par;
    const int64_t g2 = parity ? g : g - ptiles * a.n_par, per = parity ? ptiles : stiles;
    const int wi = static_cast<int>(g2 / per);
    if (!parity && wi >= a.n_sys) return;
    int worker;
    if (parity)
        worker = a.n_par == a.n - a.k ? a.k + wi : a.par_ids[wi];
    else
        worker = a.n_sys == a.k ? wi : a.sys_ids[wi];
    const bool pair = parity && a.planes == 2;
    const int64_t t0 = (g2 - wi * per) * (pair ? kSlots / 2 : kSlots) + wv * (pair ? 16 : 32);

    // X: eight columns of two consecutive k per task, reads moved back to end with X
    const int ncols = static_cast<int>(min<int64_t>(16 * NT, a.s - c0));
    const int xgroups = (ncols + 7) / 8;
    const uint16_t* X = static_cast<const uint16_t*>(a.X);
    const int64_t xlast = (a.r - 1) * a.ldx + a.s - 8;        // last element eight elements can start at
    u32x4_t x0[kXTasks], x1[kXTasks];
#pragma unroll
    for (int i = 0; i < kXTasks; ++i) {
        const int e = tid + kThr * i;
        const int64_t o = static_cast<int64_t>(2 * (e % (K / 2))) * a.ldx + c0 + 8 * min(e / (K / 2), xgroups - 1);
        x0[i] = *reinterpret_cast<const u32x4_any*>(X + min(o, xlast));
        x1[i] = *reinterpret_cast<const u32x4_any*>(X + min(o + a.ldx, xlast));
    }
    // A: every slot reads a real row (one past the block, or past A, the last
    // one: its result is not stored, or stored as the zero padding), positions
    // past r its last piece
    u32x4_t f[2][KS];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int64_t t = min<int64_t>(t0 + (pair ? 0 : 16 * u) + li, a.qb - 1);
        const uint16_t* row;
        if (parity)
            row = static_cast<const uint16_t*>(a.parity) +
                  ((pair ? u * (a.n - a.k) : 0) + static_cast<int64_t>(worker - a.k)) * a.qb * a.r + t * a.r;
        else
            row = static_cast<const uint16_t*>(a.A) + min(static_cast<int64_t>(worker) * a.qb + t, a.q - 1) * a.lda;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            f[u][ks] = *reinterpret_cast<const u32x4_t*>(row + min(32 * ks + 8 * lk, r - 8));
    }
    const u32x4_t zero = {0u, 0u, 0u, 0u};
#pragma unroll
    for (int i = 0; i < kXTasks; ++i) {
        const int e = tid + kThr * i;
        const int k = 2 * (e % (K / 2)), c = 8 * (e / (K / 2));
        if (c >= ncols) continue;
        const int64_t o = static_cast<int64_t>(k) * a.ldx + c0 + c;
        const u32x4_t v0 = k < r ? shift_down(x0[i], static_cast<int>(min<int64_t>(o - xlast, 8))) : zero;
        const u32x4_t v1 = k + 1 < r ? shift_down(x1[i], static_cast<int>(min<int64_t>(o + a.ldx - xlast, 8))) : zero;
        uint32_t* d = reinterpret_cast<uint32_t*>(sX + c * kStride + k);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            d[(2 * j) * (kStride / 2)] = (v0[j] & 0xFFFFu) | (v1[j] << 16);
            d[(2 * j + 1) * (kStride / 2)] = (v0[j] >> 16) | (v1[j] & 0xFFFF0000u);
        }
    }
    __syncthreads();

    const TileOut out{a, c0, worker, ncols, parity};
#pragma unroll
    for (int j0 = 0; j0 < NT; j0 += JB) {
        f32x4_t part[2][JB][KS / 2];                          // sums of 64 k
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const int k = 32 * ks + 8 * lk;
            bf16x8 af[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) af[u] = __builtin_bit_cast(bf16x8, ks < KS - 2 || k < r ? f[u][ks] : zero);
#pragma unroll
            for (int j = 0; j < JB; ++j) {
                const bf16x8 xf = *reinterpret_cast<const bf16x8*>(sX + (16 * (j0 + j) + li) * kStride + k);
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const f32x4_t c = ks & 1 ? part[u][j][ks / 2] : f32x4_t{0.f, 0.f, 0.f, 0.f};
                    part[u][j][ks / 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, af[u], c, 0, 0, 0);
                }
            }
        }
        f32x4_t o[2][JB];
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                double sum[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    sum[u] = part[u][j][0][w];
#pragma unroll
                    for (int h = 1; h < KS / 2; ++h) sum[u] += static_cast<double>(part[u][j][h][w]);
                }
                o[0][j][w] = static_cast<float>(pair ? sum[0] + sum[1] : sum[0]);
                o[1][j][w] = static_cast<float>(sum[1]);
            }
        out.tile(t0, j0, o[0]);
        if (!pair) out.tile(t0 + 16, j0, o[1]);
        // the next columns' operands are not read from LDS before this
        asm volatile("" ::: "memory");
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

template <int NT, int KS>
static hipError_t launch_bf16_short(const WorkerArgs& a, int64_t c0, hipStream_t st) {
    using C = ShortCfg<NT, KS>;
    const int64_t stiles = ceil_div(a.qb, C::kSlots), ptiles = ceil_div(a.qb, a.planes == 2 ? C::kSlots / 2 : C::kSlots);
    const int64_t blocks = stiles * a.n_sys + ptiles * a.n_par;
    if (blocks == 0) return hipSuccess;
    if (!grid_fits(blocks, C::kThreads)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((gemm_bf16_short_kernel<NT, KS>), dim3(static_cast<unsigned>(blocks)), dim3(C::kThreads), 0, st,
                       a, stiles, ptiles, c0);
    return hipGetLastError();
}

// Where the short-row kernel is the faster one: rows of whole 16-byte pieces, up
// to 224 elements, 256 with up to 32 columns, 384 with up to 16 ((20,16), 1.2 M
// rows: r = 64, 32 columns 72 us against 124; r = 128, 64 columns 158 and 192; r
// = 264, 1 column 158 and 237; r = 256, 64 columns 146 and 142).  Small operands
// with rows of 384 or 512 bytes, the 16 of an instruction on few channels of the
// cache, are not (50000 rows of 256, 8 columns: 10.4 against 8.6; of 264: 8.0
// against 9.8), nor few rows that all wait for a wide X (4000 of 208, 64 columns:
// 7.7 against 7.2).
static bool short_rows_fit(const WorkerArgs& a, int64_t cols) {
    auto whole = [](const void* p, int64_t stride) { return reinterpret_cast<uintptr_t>(p) % 16 == 0 && stride % 8 == 0; };
    const int64_t held = operand_bytes(a.q, a.r, a.qb, a.n - a.k, 2, 2 * a.planes);
    if ((a.r == 192 || a.r == 256) && held <= (int64_t{96} << 20)) return false;
    if (cols > 32 && a.r > 192 && held <= (int64_t{4} << 20)) return false;
    return a.r <= (cols > 32 ? 224 : cols > 16 ? 256 : 384) && whole(a.A, a.lda) && whole(a.parity, a.r);
}

template <int NT>
static hipError_t launch_bf16_short_r(const WorkerArgs& a, int64_t c0, hipStream_t st) {
    if (a.r <= 64) return launch_bf16_short<NT, 2>(a, c0, st);
    if (a.r <= 128) return launch_bf16_short<NT, 4>(a, c0, st);
    if (a.r > 192 && a.r <= 256) return launch_bf16_short<NT, 8>(a, c0, st);
    if constexpr (NT == 1) {
        if (a.r > 320) return launch_bf16_short<NT, 12>(a, c0, st);
        if (a.r > 256) return launch_bf16_short<NT, 10>(a, c0, st);
    }
    return launch_bf16_short<NT, 6>(a, c0, st);
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
        if (short_rows_fit(a, cols)) {
            e = cols > 32 ? launch_bf16_short_r<4>(a, c0, st)
                : cols > 16 ? launch_bf16_short_r<2>(a, c0, st) : launch_bf16_short_r<1>(a, c0, st);
            if (e != hipSuccess) return e;
            continue;
        }
        // Tiles by columns, row length and how many workgroups come out.  Rows
        // of up to a few chunks: 64 k each, rows split over the waves; longer
        // ones 128 or 256 k.  Few workgroups: smaller tiles that split K over the
        // waves (2000 x 16000, 64 columns, 24 workgroups of 128 rows: 102 us
        // against 185; 16384 x 4096, 192 of them: 72 against 57).
        // Measured with (20,16) codes, q rows of r elements (us):
        // - more than 32 columns: 128 rows a workgroup read X least often, 64 leave
        //   no compute unit idle at the end of a launch of a few rounds (q = 50000,
        //   48 columns: r = 400 19.2 against 20.8, r = 1500 47.3 and 54.3; q =
        //   200000, r = 1100 402 and 381).  A third chunk in flight pays from r =
        //   1024 on (131072 x 4096: 392 against 406).
        // - 17 to 32: 128 rows a workgroup up to r = 768 (q = 600000: r = 264 132
        //   against 145, r = 768 285 and 316).
        // - up to 16: 128-k chunks for streamed rows past 512 (q = 600000: r = 768
        //   231 against 272, r = 1000 315 and 388; r = 512, 8 columns, no gain).
        // - non-temporal loads only where a row's part of a chunk is long: with 32
        //   columns r = 1000 took 500 with them and 409 without (the other half of
        //   a line is gone before the next row's lanes ask for it).
        if (cols > 32) {
            const int64_t blocks8 = bf16_blocks<8>(a);
            if (blocks8 < 128)
                e = launch_bf16_mm<2, 4, 128, 3, 4, false>(a, c0, st);
            else if (blocks8 < 1024 && a.r <= 1536)
                e = launch_bf16_mm<4, 4, 64, 2, 1, false>(a, c0, st);
            else if (a.r <= 1024)
                e = launch_bf16_mm<8, 4, 64, 2, 1, false>(a, c0, st);
            else
                e = launch_bf16_mm<8, 4, 64, 3, 1, false>(a, c0, st);
        } else if (cols > 16) {
            if (a.r <= 768 && (stream || a.r <= 512) && bf16_blocks<8>(a) >= 512)
                e = launch_bf16_mm<8, 2, 64, 2, 1, false>(a, c0, st);
            else if (a.r <= 512)
                e = launch_bf16_mm<4, 2, 64, 2, 1, false>(a, c0, st);
            else if (bf16_blocks<4>(a) < 128)
                e = launch_bf16_mm<2, 2, 256, 2, 4, false>(a, c0, st);
            else
                e = stream && a.r >= 2048 ? launch_bf16_mm<4, 2, 128, 2, 1, true>(a, c0, st)
                                          : launch_bf16_mm<4, 2, 128, 2, 1, false>(a, c0, st);
        } else {
            if (a.r <= 1024)
                e = a.r > 768 || (stream && a.r > (cols == 1 ? 384 : 512)) ? launch_bf16_mm<4, 1, 128, 2, 1, false>(a, c0, st)
                                                                           : launch_bf16_mm<4, 1, 64, 2, 1, false>(a, c0, st);
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
