// Decoding from any k worker results: dec(indices, results) of Sec. III-A.
//
// For a systematic generator G = [I_k; P] and a survivor set S, let M be the
// systematic blocks that did not arrive and S_par the parity survivors
// (|M| = |S_par| = m).  Every parity survivor a satisfies
//     Y_a = sum_{j in S_sys} G[a][j] Y_j + sum_{b in M} G[a][b] (A_b X),
// so the missing block products solve the m x m system
//     G[S_par, M] Z = Y_{S_par} - G[S_par, S_sys] Y_{S_sys}.
// This is exactly the LU of the k x k survivor sub-matrix G_S with the
// systematic rows (unit rows) taken as the first k-m pivots; the remaining
// m x m block is eliminated with partial pivoting (largest |entry|, lowest row
// on ties).  The kernel forms the m x k decoding matrix
//     D = G[S_par, M]^{-1} [ -G[S_par, S_sys] | I_m ]
// (columns indexed by the sorted survivor positions) in LDS, in fp64, and
// then applies it: out block M[b] = sum_c D[b][c] Y_{S[c]}, while systematic
// survivors are copied.  Survivors are canonicalised by sorting, so the
// result does not depend on the order in which they were given.
//
// Grid: (survivor set, chunk of block-row elements), flattened.  Every
// workgroup of a set rebuilds the same D (it is small next to the apply), so
// no global scratch or second launch is needed; the arithmetic is identical
// in every workgroup, so results are deterministic.
//
// E = 4 when a row's columns come in aligned groups of four or the rows lie
// one after another, so that outputs go out as 16-byte stores; E = 1
// otherwise, lanes on consecutive elements.
#include <type_traits>

#include "internal.h"
#include "decode_common.h"

namespace coded {
namespace {

constexpr int kThreads = 256;

typedef float f32x4v __attribute__((ext_vector_type(4)));
typedef f32x4v f32x4v_any __attribute__((aligned(4)));     // 16 bytes at any fp32 boundary
typedef double f64x2v __attribute__((ext_vector_type(2)));
typedef f64x2v f64x2v_any __attribute__((aligned(8)));     // 16 bytes at any fp64 boundary

// ANY: at any boundary of the type, else 16-byte aligned.
template <bool ANY>
__device__ inline f32x4v load4(const float* p) {
    if constexpr (ANY) return *reinterpret_cast<const f32x4v_any*>(p);
    return *reinterpret_cast<const f32x4v*>(p);
}
template <bool ANY>
__device__ inline f64x2v load2(const double* p) {
    if constexpr (ANY) return *reinterpret_cast<const f64x2v_any*>(p);
    return *reinterpret_cast<const f64x2v*>(p);
}

// out = v, or alpha * v + beta * c when an epilogue operand is given (c has
// out's layout; the element is read before it is written, so c may be out).
template <int E, bool ANY = true, typename T>
__device__ inline void store_out(const DecodeArgs& a, float* p, int64_t off, const T* v) {
    float w[E];
    if (a.c) {
        float cv[E];
        if constexpr (E == 4) {
            const f32x4v f = load4<ANY>(a.c + off);
            cv[0] = f.x; cv[1] = f.y; cv[2] = f.z; cv[3] = f.w;
        } else {
            cv[0] = a.c[off];
        }
#pragma unroll
        for (int i = 0; i < E; ++i)
            w[i] = static_cast<float>(fma(a.alpha, static_cast<double>(v[i]), a.beta * static_cast<double>(cv[i])));
    } else {
#pragma unroll
        for (int i = 0; i < E; ++i) w[i] = static_cast<float>(v[i]);
    }
    // decoded outputs are written once and not read again here: non-temporal
    if constexpr (E == 4) {
        const f32x4v q = {w[0], w[1], w[2], w[3]};
        if constexpr (ANY)
            __builtin_nontemporal_store(q, reinterpret_cast<f32x4v_any*>(p + off));
        else
            __builtin_nontemporal_store(q, reinterpret_cast<f32x4v*>(p + off));
    } else {
        __builtin_nontemporal_store(w[0], p + off);
    }
}

// E consecutive elements of Y as fp32 (a copied systematic block is the
// worker's result rounded to the output type).
template <int E, typename YT, bool ANY = true>
__device__ inline void load_f32(const YT* p, float* v) {
    if constexpr (E == 4 && sizeof(YT) == 4) {
        const f32x4v f = load4<ANY>(p);
        v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
    } else if constexpr (E == 4) {
        const f64x2v lo = load2<ANY>(p), hi = load2<ANY>(p + 2);
        v[0] = static_cast<float>(lo.x); v[1] = static_cast<float>(lo.y);
        v[2] = static_cast<float>(hi.x); v[3] = static_cast<float>(hi.y);
    } else {
        v[0] = static_cast<float>(p[0]);
    }
}

// The last, incomplete group of four of a block whose rows lie one after
// another: y and off belong to its first element, `left` < 4 remain.
template <typename YT>
__device__ __forceinline__ void copy_tail(const DecodeArgs& a, float* p, int64_t off, const YT* y, int left) {
    for (int i = 0; i < left; ++i) {
        const float v = static_cast<float>(y[i]);
        store_out<1>(a, p, off + i, &v);
    }
}

// Largest of a 32-bit value over the wave, in every lane.
__device__ inline uint32_t wave_max_u32(uint32_t v) {
#define CODED_MAX_DPP(CTRL, ROWS)                                                                                    \
    v = max(v, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, ROWS, 0xF, false)))
    CODED_MAX_DPP(0x111, 0xF);           // lane - 1, - 2, - 4, - 8 of a row of 16
    CODED_MAX_DPP(0x112, 0xF);
    CODED_MAX_DPP(0x114, 0xF);
    CODED_MAX_DPP(0x118, 0xF);
    CODED_MAX_DPP(0x142, 0xA);           // the row before into rows 1 and 3
    CODED_MAX_DPP(0x143, 0xC);           // the lower half into the upper
#undef CODED_MAX_DPP
    return __builtin_amdgcn_readlane(v, 63);
}

typedef double f64x4v __attribute__((ext_vector_type(4)));

// Codes wider than the register elimination below (m + k > 64, or m > 16),
// and results past 2^31 elements.
//
// Elimination: four threads hold each column of the m x (m + k) system (m + k
// <= n <= 128) in registers, every fourth row each, and mirror it in LDS.
// Gauss-Jordan without row exchanges: every wave reads column j, one row per
// lane, finds the pivot among the unused rows and divides all multipliers at
// once, so a step is one barrier and no serial search.  Bound by the latency
// of its m dependent steps.  (An LU in LDS with one thread's pivot search and
// five barriers a step took (128,96) to 210 us a call whatever its size; the
// same steps on LDS operands, two threads a column, 57; this 36.  1000 sets
// of 65536 x 1: 716 and 220 us.)
//
// Combination: out[M] += D (16 rows a tile) * Y on v_mfma_f64_16x16x4f64, 32
// elements per wave, the survivors' loads issued 32 (or all of 20) at a time and used for
// all row tiles (one sweep over Y instead of one per eight missing blocks).
// Every workgroup of a set repeats the elimination; RT row tiles hold any m
// of the launch.  Neither RT nor the chunks change a result.
//
// Threads for COLS columns: systems of up to 64 columns take half, so that four
// workgroups share a compute unit and one's elimination runs beside the others'
// combinations.
// One row tile of fp32 results: 78 registers, nothing spilled, and so three
// workgroups a compute unit instead of two (600 (66,50) sets of 1000 x 1 25.6 us
// against 30.5, 65536 x 4 240 against 278); fp64 results would spill 14.
template <int RT, int E, int COLS, typename YT>
__global__ __launch_bounds__(4 * COLS, RT == 1 && sizeof(YT) == 4 ? 6 : 1) void decode_wide_kernel(
    DecodeArgs a, DecodeSet single, int64_t chunks, uint32_t elems_per_block, int LD) {
    __shared__ SetMeta sm;
    extern __shared__ __align__(16) double sA[];     // column c at sA[c * LD], LD odd, rows 0 .. m-1
    constexpr int kParts = 4, kThreads = kParts * COLS, kWaves = kThreads / 64, HR = 16 * RT / kParts;
    static_assert(16 * RT % kParts == 0, "whole columns per part");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int k = a.k;
    const int64_t b = blockIdx.x / chunks;
    const int64_t chunk = blockIdx.x % chunks;
    const bool writer = (chunk == 0 && tid == 0);
    if (!setup_set<kThreads>(a, single, b, writer, sm)) return;
    const int m = sm.m;
    const int first_par = k - m;          // sorted: systematic survivors first, then parity

    if (m > 0) {
        // this thread's column, 0 .. m-1: G[S_par, M], then [-G[S_par, S_sys] | I],
        // and its rows part, part + kParts, ..
        const int c = tid % COLS;
        const int part = __builtin_amdgcn_readfirstlane(tid / COLS);
        const bool mine = c < m + k;
        double* mirror = sA + (mine ? c * LD : 0);
        double col[HR];
        {
            const int sc = !mine ? 0 : (c < m ? sm.miss[c] : sm.S[c - m]);
#pragma unroll
            for (int i = 0; i < HR; ++i) {
                const int row = kParts * i + part;
                col[i] = row < m && sc < k ? a.G[static_cast<int64_t>(sm.S[first_par + row]) * k + sc] : 0.0;
            }
#pragma unroll
            for (int i = 0; i < HR; ++i) {
                const int row = kParts * i + part;
                if (c >= m) col[i] = sc < k ? -col[i] : (c - m - first_par == row ? 1.0 : 0.0);
                if (mine && row < m) mirror[row] = col[i];
            }
        }
        __syncthreads();

        uint64_t unused = m == 64 ? ~uint64_t{0} : (uint64_t{1} << m) - 1;   // rows that were no pivot yet
        int place = 0;                    // of row `lane`: the column it was the pivot of, and the pivot
        double pivot = 1.0;
        int bad = 0;
        for (int j = 0; j < m; ++j) {
            const double v = lane < m ? sA[j * LD + lane] : 0.0;
            // pivot: largest |entry| of the unused rows, lowest row on ties
            // (positive doubles order like their bits, high word first)
            const bool open = (unused >> lane) & 1;
            const uint64_t u = static_cast<uint64_t>(__double_as_longlong(fabs(v)));
            const uint32_t hi = open ? static_cast<uint32_t>(u >> 32) : 0u;
            const uint32_t top = wave_max_u32(hi);
            uint64_t cand = __ballot(open && hi == top);
            if (cand & (cand - 1)) {
                const bool in = (cand >> lane) & 1;
                const uint32_t lo = in ? static_cast<uint32_t>(u) : 0u;
                const uint32_t lotop = wave_max_u32(lo);
                cand = __ballot(in && lo == lotop);
            }
            const int p = __builtin_ctzll(cand);
            const double x = mirror[p];
            const double piv = lane_value(v, p);
            if (piv == 0.0) {             // the same in every wave
                bad = first_par + j + 1;
                break;
            }
            const double l = lane == p ? 0.0 : v / piv;
            unused &= ~(uint64_t{1} << p);
            if (lane == p) {
                place = j;
                pivot = piv;
            }
            const bool live = mine && c > j;
#pragma unroll
            for (int i = 0; i < HR; ++i) {
                const int row = kParts * i + part;
                if (row < m) {
                    const double nv = fma(-lane_value(l, row), x, col[i]);
                    col[i] = row == p ? col[i] : nv;
                    if (live) mirror[row] = col[i];
                }
            }
            __syncthreads();              // this step's rows before the next column is read
        }
        if (bad != 0) {
            if (writer) a.info[b] = bad;
            return;
        }
        // the row that was column j's pivot, divided by it, is row j of D
        // (columns 0 .. m-1 are not read again)
#pragma unroll
        for (int i = 0; i < HR; ++i) {
            const int row = kParts * i + part;
            if (row < m) {
                const int j = __builtin_amdgcn_readlane(place, row);
                const double d = col[i] / lane_value(pivot, row);
                if (mine && c >= m) mirror[j] = d;
            }
        }
        __syncthreads();
    }
    if (writer) a.info[b] = 0;

    const YT* Y = static_cast<const YT*>(a.Y);
    float* out = a.out + b * a.out_stride;
    // elements below 2^31, positions past a chunk's end below 2^32
    const uint32_t s = static_cast<uint32_t>(a.s);
    const uint32_t total = static_cast<uint32_t>(a.qb * a.s);
    const uint32_t e0 = static_cast<uint32_t>(chunk) * elems_per_block;
    if (e0 >= total) return;
    const uint32_t e1 = chunk_end(e0, elems_per_block, total);

    // systematic survivors: (block, E elements) items in one sequence, U per
    // thread in flight (E == 4: four elements of one row, or of rows that lie
    // one after another, a block's last group maybe fewer)
    {
        constexpr int U = 4;
        const uint32_t nq = (e1 - e0 + E - 1) / E;
        const uint64_t items = static_cast<uint64_t>(nq) * first_par;
        const uint32_t dc = kThreads / nq, de = kThreads % nq;
        uint32_t c = static_cast<uint32_t>(tid) / nq, eq = static_cast<uint32_t>(tid) % nq;
        for (uint64_t it = tid; it < items; it += kThreads * U) {
            float v[U][E];
            int64_t off[U];
            int left[U], cs[U];          // elements of the item that lie in A
#pragma unroll
            for (int q = 0; q < U; ++q) {
                const bool live = it + kThreads * q < items;
                const uint32_t cc = live ? c : 0;
                const uint32_t e = e0 + E * (live ? eq : 0);
                const int w = sm.S[cc];
                const uint32_t t = s == 1 ? e : e / s, lim = static_cast<uint32_t>(sm.lim[w]);
                load_f32<E, YT>(Y + sm.yoff[cc] + min(e, total - E), v[q]);
                off[q] = sm.ooff[w] + static_cast<int64_t>(t) * a.ldo + (s == 1 ? 0 : e - t * s);
                left[q] = live ? (s == 1 ? static_cast<int>(min(e1, lim) - e) : (t < lim ? E : 0)) : 0;
                cs[q] = cc;
                c += dc;
                eq += de;
                if (eq >= nq) {
                    eq -= nq;
                    ++c;
                }
            }
#pragma unroll
            for (int q = 0; q < U; ++q) {
                if (left[q] >= E)
                    store_out<E>(a, out, off[q], v[q]);
                else if (E > 1 && left[q] > 0)       // s == 1: element e of a block is off - ooff
                    copy_tail(a, out, off[q], Y + sm.yoff[cs[q]] + (off[q] - sm.ooff[sm.S[cs[q]]]), left[q]);
            }
        }
    }
    if (m == 0) return;

    const int li = lane & 15, lk = lane >> 4;
    const int steps = (k + 3) / 4;
    // E == 4: Y is the first operand and its lane li takes element 4 (li % 4) +
    // li / 4 of a tile, so that lane (li, lk) gets elements 4 lk .. 4 lk + 3 of
    // block M[16 rt + li] and stores them at once.
    const int ye = E == 4 ? 4 * (li & 3) + (li >> 2) : li;
    // A store instruction writes 64 bytes of each of 16 blocks: past the caches
    // where these are whole 64-byte segments, else through them, which put the
    // pieces of a segment together (600 (36,18) sets of 65536 x 4, fp64 results:
    // 487 us past them, 259 through them; 20000 x 16, whole segments: 290 and 300).
    const bool segments = (((reinterpret_cast<uintptr_t>(out) >> 2) | static_cast<uint64_t>(a.qb * a.ldo) |
                            (s == 1 ? 0 : s | static_cast<uint64_t>(a.ldo))) & 15) == 0;
    float* ob[E == 4 ? RT : 1];
    uint32_t olim[E == 4 ? RT : 1];                  // the block's rows in A, 0 for no block
    if constexpr (E == 4) {
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int bb = 16 * rt + li, w = sm.miss[bb < m ? bb : 0];
            ob[rt] = out + sm.ooff[w];
            olim[rt] = bb < m ? static_cast<uint32_t>(sm.lim[w]) : 0u;
        }
    }
    // NB steps of four survivors' loads at a time, R row tiles.  HELD (steps ==
    // NB): D and the survivors' addresses stay in registers; the vector
    // instructions that fetch them for every tile run beside no matrix instruction
    // of their SIMD (600 (36,18) sets, fp64 results, 16384 x 8 141 us without, 116
    // so; 20000 x 16 313 and 255; (100,20), 3000 x 64 232 and 201).
    auto combine = [&](auto nb, auto tiles, auto held) __attribute__((always_inline)) {
        constexpr int NB = decltype(nb)::value, R = decltype(tiles)::value;
        constexpr bool HELD = decltype(held)::value;
        const YT* yp[HELD ? NB : 1];
        double dh[HELD ? NB : 1][R];
        if constexpr (HELD) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int c = 4 * i + lk, at = min(c, k - 1);
                yp[i] = Y + sm.yoff[at];
#pragma unroll
                for (int rt = 0; rt < R; ++rt) {
                    const int row = 16 * rt + li;
                    const double d = sA[(m + at) * LD + min(row, m - 1)];
                    dh[i][rt] = c < k && row < m ? d : 0.0;
                }
            }
        }
        for (uint32_t base = e0 + 32 * wv; base < e1; base += 32 * kWaves) {
            // past the chunk's end: its last element again (an element's products
            // depend on that element of Y only, and are not stored)
            const uint32_t last = e1 - 1, at0 = base + ye, at1 = at0 + 16;
            const uint32_t el[2] = {at0 < last ? at0 : last, at1 < last ? at1 : last};
            f64x4v acc[R][2];
#pragma unroll
            for (int rt = 0; rt < R; ++rt) acc[rt][0] = acc[rt][1] = f64x4v{0.0, 0.0, 0.0, 0.0};
            auto multiply = [&](int rt, double dv, double y0, double y1) __attribute__((always_inline)) {
                if constexpr (E == 4) {
                    acc[rt][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(y0, dv, acc[rt][0], 0, 0, 0);
                    acc[rt][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(y1, dv, acc[rt][1], 0, 0, 0);
                } else {
                    acc[rt][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(dv, y0, acc[rt][0], 0, 0, 0);
                    acc[rt][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(dv, y1, acc[rt][1], 0, 0, 0);
                }
            };
            if constexpr (HELD) {
                YT yv[NB][2];
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    yv[i][0] = yp[i][el[0]];
                    yv[i][1] = yp[i][el[1]];
                }
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const bool ok = i < NB - 1 || 4 * i + lk < k;
                    const double y0 = ok ? static_cast<double>(yv[i][0]) : 0.0;
                    const double y1 = ok ? static_cast<double>(yv[i][1]) : 0.0;
#pragma unroll
                    for (int rt = 0; rt < R; ++rt) multiply(rt, dh[i][rt], y0, y1);
                }
            } else {
                for (int st = 0; st < steps; st += NB) {
                    YT yv[NB][2];
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        const YT* y = Y + sm.yoff[min(4 * (st + i) + lk, k - 1)];
                        yv[i][0] = y[el[0]];
                        yv[i][1] = y[el[1]];
                    }
#pragma unroll
                    for (int i = 0; i < NB; ++i) {
                        const int c = 4 * (st + i) + lk;
                        const bool ok = c < k;
                        const double y0 = ok ? static_cast<double>(yv[i][0]) : 0.0;
                        const double y1 = ok ? static_cast<double>(yv[i][1]) : 0.0;
                        const double* col = sA + (m + min(c, k - 1)) * LD;
#pragma unroll
                        for (int rt = 0; rt < R; ++rt) {
                            if (16 * rt < m && st + i < steps) {
                                const int row = 16 * rt + li;
                                const double d = col[min(row, m - 1)];
                                multiply(rt, ok && row < m ? d : 0.0, y0, y1);
                            }
                        }
                    }
                }
            }
            if constexpr (E == 4) {
                uint32_t eh[2], th[2];
                int64_t oh[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    eh[h] = base + 16 * h + 4 * lk;
                    th[h] = s == 1 ? eh[h] : eh[h] / s;           // s % 4 == 0: the four share a row
                    oh[h] = static_cast<int64_t>(th[h]) * a.ldo + (s == 1 ? 0 : eh[h] - th[h] * s);
                }
#pragma unroll
                for (int rt = 0; rt < R; ++rt) {
                    if (a.c == nullptr) {
                        f32x4v w[2];
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int i = 0; i < 4; ++i) w[h][i] = static_cast<float>(acc[rt][h][i]);
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            if (eh[h] >= e1 || th[h] >= olim[rt]) continue;
                            const uint32_t left = s == 1 ? (e1 < olim[rt] ? e1 : olim[rt]) - eh[h] : 4u;
                            float* o = ob[rt] + oh[h];
                            if (left < 4) {
                                for (uint32_t i = 0; i < left; ++i) o[i] = w[h][i];
                            } else if (segments) {
                                __builtin_nontemporal_store(w[h], reinterpret_cast<f32x4v_any*>(o));
                            } else {      // between fences, or the compiler makes one plain store of the two
                                asm volatile("" ::: "memory");
                                *reinterpret_cast<f32x4v_any*>(o) = w[h];
                                asm volatile("" ::: "memory");
                            }
                        }
                    } else {
#pragma unroll
                        for (int h = 0; h < 2; ++h) {
                            if (eh[h] >= e1 || th[h] >= olim[rt]) continue;
                            const double v4[4] = {acc[rt][h][0], acc[rt][h][1], acc[rt][h][2], acc[rt][h][3]};
                            const uint32_t left = s == 1 ? (e1 < olim[rt] ? e1 : olim[rt]) - eh[h] : 4u;
                            if (left >= 4) {
                                store_out<4>(a, ob[rt], oh[h], v4);
                            } else {
                                for (uint32_t i = 0; i < left; ++i) store_out<1>(a, ob[rt], oh[h] + i, &v4[i]);
                            }
                        }
                    }
                }
                continue;
            }
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t e = base + 16 * h + li;
                if (e < e1) {
                    const uint32_t t = e / s, col = e - t * s;
#pragma unroll
                    for (int rt = 0; rt < R; ++rt) {
#pragma unroll
                        for (int v = 0; v < 4; ++v) {
                            const int bb = 16 * rt + 4 * v + lk;
                            if (bb < m) {
                                const int w = sm.miss[bb];
                                const double val = acc[rt][h][v];
                                if (t < static_cast<uint32_t>(sm.lim[w]))
                                    store_out<1>(a, out, sm.ooff[w] + static_cast<int64_t>(t) * a.ldo + col, &val);
                            }
                        }
                    }
                }
            }
        }
    };
    constexpr std::integral_constant<int, 5> five{};
    constexpr std::integral_constant<int, 8> eight{};
    constexpr std::integral_constant<int, RT> all{};
    if constexpr (COLS == 64) {
        if (steps == 5 && m <= 16) return combine(five, std::integral_constant<int, 1>{}, std::true_type{});
        if (steps == 5) return combine(five, all, std::true_type{});
    }
    combine(eight, all, std::false_type{});
}

// ---------------------------------------------------------------- fast path
// Codes with at most kFastM missing blocks per set and m + k <= 64: one wave
// eliminates the m x (m + k) system [G[S_par, M] | -G[S_par, S_sys] | I] in
// registers (Gauss-Jordan, partial pivoting: the same pivots as an LU,
// one column per lane, no workgroup barriers), and the combination of the
// survivors is one 16-row matrix-core tile:
//     out[M] (16 x 16 elements) += D (16 x 4 survivors) * Y (4 x 16 elements)
// on v_mfma_f64_16x16x4f64, with D held in registers for the whole set.

// Consecutive elements per lane in the combination's loads (E == 4 path);
// 4 needs 192 registers at k = 48 (2 waves per SIMD) and measured slower.
constexpr int kDecodePE = 2;

// PE consecutive elements of Y (16-byte aligned for fp64 pairs, PE * 4-byte
// aligned for fp32) with vector loads.
template <int PE, typename YT>
__device__ inline void load_pe(const YT* p, YT (&v)[PE]) {
    if constexpr (sizeof(YT) == 8) {
#pragma unroll
        for (int i = 0; i < PE; i += 2) {
            const double2 d = reinterpret_cast<const double2*>(p)[i / 2];
            v[i] = d.x;
            v[i + 1] = d.y;
        }
    } else if constexpr (PE == 4) {
        const float4 f = *reinterpret_cast<const float4*>(p);
        v[0] = f.x; v[1] = f.y; v[2] = f.z; v[3] = f.w;
    } else {
        const float2 f = *reinterpret_cast<const float2*>(p);
        v[0] = f.x; v[1] = f.y;
    }
}

// SIMD of the calling wave within its compute unit (hardware register
// HW_ID, bits 5:4).  The four waves of a 256-thread workgroup run on four
// different SIMDs.
__device__ inline int simd_id() {
    return static_cast<int>(__builtin_amdgcn_s_getreg(4 | (4 << 6) | ((2 - 1) << 11)) & 3);
}

// One workgroup per (set, chunk).
// E == 4: the wave on SIMD 0 of its compute unit (wave 0 if none is) forms
// D and then copies the systematic survivors; the other three waves combine
// the missing blocks on the fp64 matrix cores.  Vector instructions do not
// overlap with fp64 matrix instructions on the same SIMD, so every compute
// unit keeps the copies and the elimination on one SIMD and the matrix work
// on the other three.  Which wave takes which role changes only the timing.
// E == 1: wave 0 eliminates while the others start copying; then all four
// combine.
// FLAT (E == 4, YBUF, s == ldo == 1): Y and the output at any alignment, blocks
// of any number of elements; the tails and odd ends cost the others' 80
// registers (1000 (64,48) sets of 16384 x 8: 185 us against 135).
// KS: matrix-core K steps (4 survivors each) the kernel is built for, k <= 4 KS;
// FULL: k == 4 KS (no padding steps).
// Raw buffer over `bytes` bytes (gfx9 dword-3 value: no stride, no format).
__device__ inline __amdgpu_buffer_rsrc_t y_buffer(const void* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0), static_cast<int>(bytes),
                                             0x00020000);
}

// YBUF (E == 4, Y's byte offsets below 2^31): the combining waves read Y as a
// raw buffer, each lane's offset per survivor fixed for the set and the
// group's offset in a scalar register, so the loads need no vector address
// arithmetic.
// Six waves per SIMD (80 registers, six workgroups per compute unit) for the
// variants with whole survivor groups and buffer-addressed Y up to 12 groups,
// which then spill one word in the elimination; the others keep the default
// register budget.
template <int KS, bool FULL, bool YBUF, bool FLAT>
constexpr int decode_min_waves() {
    return FULL && YBUF && !FLAT && KS <= 12 ? 6 : 1;
}

template <int KS, int E, typename YT, bool FULL, bool YBUF, bool FLAT>
__global__ __launch_bounds__(kThreads, (decode_min_waves<KS, FULL, YBUF, FLAT>())) void decode_mfma_kernel(
    DecodeArgs args, DecodeSet single, int64_t chunks, int elems_per_block) {
    __shared__ SetMeta sm;
    __shared__ double sD[64 * kFastLd];
    __shared__ double sOut[E == 4 ? kThreads / 64 - 1 : 1][E == 4 ? 256 * kDecodePE : 1];   // per combining wave output tile
    __shared__ int32_t sSimd[kThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    DecodeArgs a = args;
    if constexpr (E == 1) {
        // Short chunks, latency bound: the sizes the set-up and the first
        // loads depend on are fetched in one batch and held in scalar
        // registers (left alone, the compiler fetches them one dependent
        // round trip after another).
        asm volatile("" : "+s"(a.q), "+s"(a.qb), "+s"(a.s), "+s"(a.ldo), "+s"(a.n), "+s"(a.k), "+s"(chunks),
                     "+s"(elems_per_block));
    }
    const int k = a.k;
    // fewer than 2^31 workgroups (checked at launch): 32-bit division
    const uint32_t bid = blockIdx.x, nch = static_cast<uint32_t>(chunks);
    const int64_t b = bid / nch;
    const int64_t chunk = bid - static_cast<uint32_t>(b) * nch;
    const bool writer = (chunk == 0 && tid == 0);
    if (lane == 0) sSimd[wv] = simd_id();             // read after setup_set's barriers
    if (!setup_set<kThreads>(a, single, b, writer, sm)) return;
    const int m = sm.m;
    const int first_par = k - m;
    const YT* Y = static_cast<const YT*>(a.Y);
    float* out = a.out + b * a.out_stride;
    const int s = static_cast<int>(a.s);
    const int total = static_cast<int>(a.qb * a.s);
    const int e0 = static_cast<int>(chunk) * elems_per_block;
    const int e1 = min(total, e0 + elems_per_block);
    constexpr int kWaves = kThreads / 64;

    // E == 1 (chunks of single elements, often short): the systematic
    // survivors are copied as (element, survivor) items spread over the
    // waves that do not eliminate, and the first CI items of each thread are
    // loaded before the barrier that publishes the elimination's status (and
    // stored only after it: a singular set writes nothing).
    constexpr int CI = 4;
    const int len = e1 - e0, items = len * first_par;
    const int cw = m > 0 ? 1 : 0, nthr = kThreads - 64 * cw, ctid = tid - 64 * cw;
    YT cy[CI];
    int64_t co[CI];                      // output offset of item i, -1 for none
    if constexpr (E == 1) {
#pragma unroll
        for (int i = 0; i < CI; ++i) {
            const int it = ctid + i * nthr;
            co[i] = -1;
            cy[i] = YT(0);
            if (ctid >= 0 && it < items) {
                const int c = it / len, e = e0 + (it - c * len);
                const int t = e / s, col = e - t * s;
                const int w = sm.S[c];
                if (t < sm.lim[w]) {
                    cy[i] = Y[sm.yoff[c] + e];
                    co[i] = sm.ooff[w] + static_cast<int64_t>(t) * a.ldo + col;
                }
            }
        }
    }

    // E == 1: each wave's first tile of Y (Y_{S[4 st + lk]} at element li of
    // the tile, as the tile loop below reads it) is requested before the
    // barrier that publishes D, so its latency overlaps the elimination.
    const int ntiles1 = (e1 - e0 + 15) / 16;
    YT yfirst[E == 1 ? KS : 1];
    if constexpr (E == 1) {
        if (m > 0 && wv < ntiles1) {
            const int li = lane & 15, lk = lane >> 4;
            const int el = min(e0 + wv * 16 + li, e1 - 1);
#pragma unroll
            for (int st = 0; st < KS; ++st) {
                const int c = 4 * st + lk;
                yfirst[st] = Y[(c < k ? static_cast<int32_t>(sm.yoff[c]) : 0) + el];
            }
        }
    }

    // the eliminating wave (E == 4: also the copying wave)
    int ew = 0;
    if constexpr (E == 4) {
#pragma unroll
        for (int w = kWaves - 1; w >= 0; --w) ew = sSimd[w] == 0 ? w : ew;
    }
    if (m > 0 && wv == ew) eliminate_set(a, sm, m, first_par, lane, sD);
    __syncthreads();
    if (sm.status != 0) {
        if (writer) a.info[b] = sm.status;
        return;
    }
    if (writer) a.info[b] = 0;

    if constexpr (E == 1) {
#pragma unroll
        for (int i = 0; i < CI; ++i) {
            if (co[i] >= 0) {
                const float fv = static_cast<float>(cy[i]);   // the worker's result in the output type
                store_out<1>(a, out, co[i], &fv);
            }
        }
        for (int it = ctid + CI * nthr; ctid >= 0 && it < items; it += nthr) {
            const int c = it / len, e = e0 + (it - c * len);
            const int t = e / s, col = e - t * s;
            const int w = sm.S[c];
            if (t < sm.lim[w]) {
                const float fv = static_cast<float>(Y[sm.yoff[c] + e]);
                store_out<1>(a, out, sm.ooff[w] + static_cast<int64_t>(t) * a.ldo + col, &fv);
            }
        }
    }

    // E == 4: the copying wave takes the systematic survivors.  Long chunks go
    // block by block, U four-element items per lane in flight (an item past
    // the block's end re-reads its last elements and stores nothing), the
    // block's addresses in scalar registers.  Chunks of up to 128 such items go as one
    // sequence of (block, four elements) items: block by block, a chunk of 64
    // elements leaves three quarters of the lanes idle and waits for memory
    // once per block ((25,23), 16 columns: 13.2 us against 5.7).  With dense
    // output rows (ldo == s) element e of a block is at offset e from its
    // first row.
    if constexpr (E == 4) {
        if (wv == ew) {
            constexpr int U = sizeof(YT) == 8 ? 4 : 8;
            const bool dense = FLAT || a.ldo == a.s;
            const uint32_t nq = static_cast<uint32_t>(e1 - e0 + 3) / 4;
            const uint32_t citems = nq * static_cast<uint32_t>(first_par);   // nq k < 2^31 / 4
            if (e0 >= e1) return;
            if (nq > 128) {
                for (int c = 0; c < first_par; ++c) {
                    const int w = __builtin_amdgcn_readfirstlane(sm.S[c]);
                    const YT* yr = Y + static_cast<int64_t>(w) * total;
                    float* ob = out + static_cast<int64_t>(w) * a.qb * a.ldo;
                    const int elim = min(e1, __builtin_amdgcn_readfirstlane(sm.lim[w]) * s);   // inside A
                    for (int e = e0 + 4 * lane; e < elim; e += 1024) {
                        float v[4][4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) load_f32<4, YT, FLAT>(yr + min(e + 256 * u, (FLAT ? total : elim) - 4), v[u]);
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            const int ee = e + 256 * u;
                            if (ee + (FLAT ? 4 : 1) <= elim) {
                                const int64_t off = dense ? ee : static_cast<int64_t>(ee / s) * a.ldo + ee % s;
                                store_out<4, FLAT>(a, ob, off, v[u]);
                            } else if (FLAT && ee < elim) {
                                copy_tail(a, ob, ee, yr + ee, elim - ee);
                            }
                        }
                    }
                }
                return;
            }
            const uint32_t dc = 64 / nq, de = 64 % nq;
            uint32_t c = static_cast<uint32_t>(lane) / nq, eq = static_cast<uint32_t>(lane) % nq;
            for (uint32_t it = lane; it < citems; it += 64 * U) {
                float v[U][4];
                int32_t we[U];         // block of item u, -1 for none, its element and the elements from it on
                int ee[U], left[FLAT ? U : 1];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const bool live = it + 64 * u < citems;
                    const uint32_t cc = live ? c : 0;
                    const int w = sm.S[cc];
                    const int e = e0 + 4 * static_cast<int>(live ? eq : 0);
                    load_f32<4, YT, FLAT>(Y + sm.yoff[cc] + (FLAT ? min(e, total - 4) : e), v[u]);
                    ee[u] = e;
                    we[u] = live && e < sm.lim[w] * s ? w : -1;
                    if constexpr (FLAT) left[u] = min(e1, sm.lim[w]) - e;
                    c += dc;
                    eq += de;
                    if (eq >= nq) {
                        eq -= nq;
                        ++c;
                    }
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (we[u] < 0) continue;
                    if (FLAT && left[FLAT ? u : 0] < 4) {
                        copy_tail(a, out, sm.ooff[we[u]] + ee[u], Y + static_cast<int64_t>(we[u]) * total + ee[u],
                                  left[FLAT ? u : 0]);
                    } else {
                        const int64_t off = dense ? ee[u] : static_cast<int64_t>(ee[u] / s) * a.ldo + ee[u] % s;
                        store_out<4, FLAT>(a, out, sm.ooff[we[u]] + off, v[u]);
                    }
                }
            }
            return;
        }
    }
    if (m == 0) return;

    // Missing blocks: 16-element tiles, one wave per tile.  Lane (li, lk)
    // holds D[li][4 st + lk] (A operand) and loads Y_{S[4 st + lk]}[e] (B);
    // accumulator item v is out block M[4 v + lk], element li of the tile.
    const int li = lane & 15, lk = lane >> 4;
    double af[KS];
    int32_t yo[KS];
    uint32_t valid = 0;                   // bit st: survivor 4 st + lk exists
#pragma unroll
    for (int st = 0; st < KS; ++st) {
        const int c = 4 * st + lk;
        af[st] = c < k ? sD[c * kFastLd + li] : 0.0;
        yo[st] = c < k ? static_cast<int32_t>(sm.yoff[c]) : 0;
        valid |= (c < k ? 1u : 0u) << st;
    }
    if constexpr (E == 4) {
        // Tiles in groups of PE: lane (li, lk) loads elements PE li .. PE li +
        // PE - 1 of a 16 PE-element group at once, and PE matrix-core
        // products take the elements in each phase.  The results go through
        // this wave's LDS tile (16 blocks x 16 PE elements, fp64) back into
        // element order, and each lane writes 4 consecutive elements of one
        // block per 16-byte store, or fewer at the end of a block (E == 4:
        // s % 4 == 0, or s == 1 with a dense output, read and written at any
        // alignment).
        constexpr int PE = kDecodePE;
        constexpr int W = 16 * PE;
        const int ngroups = (e1 - e0 + W - 1) / W;
        const int crank = __builtin_amdgcn_readfirstlane(wv < ew ? wv : wv - 1);   // rank among the combining waves
        double* buf = sOut[crank];
        // each store instruction covers 16 / PE blocks, 4 PE lanes (W
        // elements, whole 128-byte lines for PE = 2) per block; this lane's
        // block, its first row in out and its element limit are fixed for the set
        constexpr int QPB = 4 * PE;
        const int g4 = lane % QPB;
        float* obase[PE];
        int elim[PE];
#pragma unroll
        for (int h = 0; h < PE; ++h) {
            const int bb = lane / QPB + (16 / PE) * h;
            const int w = sm.miss[bb < m ? bb : 0];
            obase[h] = out + sm.ooff[w];
            elim[h] = bb < m ? min(e1, sm.lim[w] * s) : 0;   // 0: no block for this lane
        }
        const bool dense = FLAT || a.ldo == a.s;
        // YBUF: byte offset of this lane's elements of survivor 4 st + lk (a
        // group's elements past the block's end read the next result or zeros
        // past the buffer; those columns are not stored)
        uint32_t yb[YBUF ? KS : 1];
        const __amdgpu_buffer_rsrc_t yrs =
            y_buffer(Y, static_cast<uint32_t>(YBUF ? static_cast<int64_t>(a.n) * total * sizeof(YT) : 0));
        if constexpr (YBUF) {
#pragma unroll
            for (int st = 0; st < KS; ++st) yb[st] = static_cast<uint32_t>((yo[st] + PE * li) * sizeof(YT));
        }
        for (int gp = crank; gp < ngroups; gp += kWaves - 1) {
            const int base = e0 + gp * W;
            YT yv[KS][PE];
            if constexpr (YBUF) {
                static_assert(PE == 2, "one 2-element load per survivor");
                const uint32_t so = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(base) * sizeof(YT));
                auto load = [&](uint32_t add, uint32_t so) __attribute__((always_inline)) {
#pragma unroll
                    for (int st = 0; st < KS; ++st) {
                        if constexpr (sizeof(YT) == 8) {
                            const double2 d = __builtin_bit_cast(
                                double2, __builtin_amdgcn_raw_buffer_load_b128(yrs, yb[st] + add, so, 0));
                            yv[st][0] = d.x;
                            yv[st][1] = d.y;
                        } else {
                            const float2 f = __builtin_bit_cast(
                                float2, __builtin_amdgcn_raw_buffer_load_b64(yrs, yb[st] + add, so, 0));
                            yv[st][0] = f.x;
                            yv[st][1] = f.y;
                        }
                    }
                };
                if (FLAT && (total & 1) && base + W > total) {
                    // an odd block's last element has no second one, at the
                    // end of Y not even in memory: its lane reads the pair
                    // before and takes the second (no offset falls below zero:
                    // lane 0 is the last one only when base > 0)
                    const bool last = base + PE * li == total - 1;
                    const uint32_t d = base > 0 ? sizeof(YT) : 0;
                    load(d - (last ? static_cast<uint32_t>(sizeof(YT)) : 0u), so - d);
#pragma unroll
                    for (int st = 0; st < KS; ++st) yv[st][0] = last ? yv[st][1] : yv[st][0];
                } else {
                    load(0, so);
                }
            } else {
                // a group past the chunk's end reads the block's last PE elements
                // instead (in bounds; those columns are not stored)
                const int el = min(base + PE * li, total - PE);
#pragma unroll
                for (int st = 0; st < KS; ++st) load_pe<PE>(Y + yo[st] + el, yv[st]);
            }
            f64x4v acc[PE];
#pragma unroll
            for (int q = 0; q < PE; ++q) acc[q] = f64x4v{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int st = 0; st < KS; ++st) {
                // padding steps (k not a multiple of 4) contribute exact zeros
                const bool ok = FULL || ((valid >> st) & 1u);
#pragma unroll
                for (int q = 0; q < PE; ++q)
                    acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(af[st], ok ? static_cast<double>(yv[st][q]) : 0.0,
                                                                  acc[q], 0, 0, 0);
            }
            // item v of lane (li, lk): block 4 v + lk, element PE li + q of acc[q],
            // kept in the tile at [block][q][li] (one 8-byte write per item, no
            // register moves)
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int q = 0; q < PE; ++q) buf[(4 * v + lk) * W + 16 * q + li] = acc[q][v];
#pragma unroll
            for (int h = 0; h < PE; ++h) {
                const int bb = lane / QPB + (16 / PE) * h, eg = base + 4 * g4;
                if (eg < elim[h]) {
                    // elements 4 g4 .. 4 g4 + 3: (li, q) = (2 g4, 0), (2 g4, 1), (2 g4 + 1, 0), (2 g4 + 1, 1)
                    static_assert(PE == 2, "tile order");
                    const double2 r0 = *reinterpret_cast<const double2*>(&buf[bb * W + 2 * g4]);
                    const double2 r1 = *reinterpret_cast<const double2*>(&buf[bb * W + 16 + 2 * g4]);
                    const double v4[4] = {r0.x, r1.x, r0.y, r1.y};
                    // s % 4 == 0: the four share one row; dense rows (ldo == s) need no division
                    const int64_t off = dense ? eg : static_cast<int64_t>(eg / s) * a.ldo + eg % s;
                    if (!FLAT || eg + 4 <= elim[h]) {
                        store_out<4, FLAT>(a, obase[h], off, v4);
                    } else {
                        for (int i = 0; i < elim[h] - eg; ++i) store_out<1>(a, obase[h], off + i, &v4[i]);
                    }
                }
            }
        }
    } else {
        for (int tile = wv; tile < ntiles1; tile += kWaves) {
            const int e = e0 + tile * 16 + li;
            // Straight-line loads, all issued before the first is used (the
            // first tile's before the barrier).  A lane past the chunk's end
            // reads its last element instead: column li of the product
            // depends on column li of Y only, and is not stored.
            const int el = min(e, e1 - 1);
            YT yv[KS];
#pragma unroll
            for (int st = 0; st < KS; ++st) yv[st] = tile == wv ? yfirst[st] : Y[yo[st] + el];
            f64x4v acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int st = 0; st < KS; ++st) {
                const double bv = (FULL || ((valid >> st) & 1u)) ? static_cast<double>(yv[st]) : 0.0;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(af[st], bv, acc, 0, 0, 0);
            }
            if (e < e1) {
                const int t = e / s, col = e - t * s;
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int bb = 4 * v + lk;
                    if (bb < m) {
                        const int w = sm.miss[bb];
                        const double val = acc[v];
                        if (t < sm.lim[w]) store_out<1>(a, out, sm.ooff[w] + static_cast<int64_t>(t) * a.ldo + col, &val);
                    }
                }
            }
        }
    }
}

// The fast path takes codes (not sets) by their largest possible m, so a set
// decodes with the same arithmetic alone or in a batch.  Its positions are
// signed 32-bit, some of them past a block's end: blocks of up to 2^30
// elements (one worker alone may have twice that).
bool fast_path_ok(const DecodeArgs& a) {
    const int mmax = std::min(a.k, a.n - a.k);
    return mmax <= kFastM && a.k + mmax <= 64 && static_cast<int64_t>(a.n) * a.qb * a.s <= 0x7FFFFFFF &&
           a.qb * a.s <= (int64_t(1) << 30);
}

template <int E, bool FLAT>
hipError_t launch_fast(const DecodeArgs& a, const DecodeSet& single, hipStream_t st) {
    // About 1024 workgroups when the batch is small: a set is cut into chunks
    // of at least 64 elements (each workgroup repeats the small elimination),
    // which keeps the per-wave tile chains of a single decode short while the
    // repeated eliminations, one per workgroup on its first SIMD, stay few
    // (one (32,24) set of 64 columns: 23.0 us with 1024 workgroups, 23.5 with
    // 512, 29 with 2048).  About 512 for a batch whose sets may miss more than
    // four blocks, where the elimination weighs more (1000 (64,48) sets of
    // 16384 x 8: 139 us with 512, 150 with 1024; 100 (16,12) sets of 2000 x
    // 64: 28.7 and 26.1).
    const int64_t total = a.qb * a.s;
    const int64_t target = a.batch > 1 && std::min(a.k, a.n - a.k) > 4 ? 512 : 1024;
    const Chunks cut = split_chunks(total, ceil_div(target, a.batch), 16);
    const int64_t chunks = cut.count, blocks = chunks * a.batch;
    if (!grid_fits(blocks, kThreads)) return hipErrorInvalidConfiguration;
    const int ksteps = (a.k + 3) / 4;
    const dim3 grid(static_cast<unsigned>(blocks));
    const int per32 = static_cast<int>(cut.per);
    // Y read as a raw buffer (E == 4) when its byte offsets fit in 31 bits
    const bool ybuf = E == 4 && static_cast<int64_t>(a.n) * total * (a.y_f64 ? 8 : 4) < (int64_t(1) << 31);
#define CODED_FAST_Y(KS, FULL, YB)                                                                             \
    do {                                                                                                       \
        if (a.y_f64)                                                                                           \
            hipLaunchKernelGGL((decode_mfma_kernel<KS, E, double, FULL, YB, FLAT>), grid, dim3(kThreads), 0, st, a,  \
                               single, chunks, per32);                                                         \
        else                                                                                                   \
            hipLaunchKernelGGL((decode_mfma_kernel<KS, E, float, FULL, YB, FLAT>), grid, dim3(kThreads), 0, st, a,   \
                               single, chunks, per32);                                                         \
    } while (0)
#define CODED_FAST_F(KS, FULL)                       \
    do {                                             \
        if (FLAT || ybuf)                            \
            CODED_FAST_Y(KS, FULL, E == 4);          \
        else                                         \
            CODED_FAST_Y(KS, FULL, FLAT);            \
    } while (0)
#define CODED_FAST(KS)                          \
    do {                                        \
        if (a.k == 4 * (KS))                    \
            CODED_FAST_F(KS, true);             \
        else                                    \
            CODED_FAST_F(KS, false);            \
    } while (0)
    if (ksteps <= 4) CODED_FAST(4);
    else if (ksteps <= 8) CODED_FAST(8);
    else if (ksteps <= 12) CODED_FAST(12);
    else CODED_FAST(16);
#undef CODED_FAST
#undef CODED_FAST_F
#undef CODED_FAST_Y
    return hipGetLastError();
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) % 16) == 0; }

template <int RT, int E, int COLS>
hipError_t launch_wide_cols(const DecodeArgs& a, const DecodeSet& single, int mmax, hipStream_t st) {
    // Whole rounds of the workgroups that run at once: two a compute unit, four
    // of the small ones, one with the registers of four row tiles.  (600 sets
    // in one 512-thread workgroup each ran two rounds, the second with 88.)
    constexpr int kThreads = 4 * COLS;
    const int64_t total = a.qb * a.s;
    const Chunks cut = split_chunks(total, chunks_per_set(total, a.batch, RT == 4 ? 256 : 256 * 1024 / kThreads), 32);
    const int64_t blocks = cut.count * a.batch;
    if (!grid_fits(blocks, kThreads)) return hipErrorInvalidConfiguration;
    const int LD = std::max(mmax, 1) | 1;            // odd: columns start in different banks
    const size_t shmem = static_cast<size_t>(a.k + mmax) * LD * sizeof(double);
    const dim3 grid(static_cast<unsigned>(blocks));
    if (a.y_f64)
        hipLaunchKernelGGL((decode_wide_kernel<RT, E, COLS, double>), grid, dim3(kThreads), shmem, st, a, single, cut.count,
                           static_cast<uint32_t>(cut.per), LD);
    else
        hipLaunchKernelGGL((decode_wide_kernel<RT, E, COLS, float>), grid, dim3(kThreads), shmem, st, a, single, cut.count,
                           static_cast<uint32_t>(cut.per), LD);
    return hipGetLastError();
}

// By the code, as the arithmetic does not depend on it but a set's chunks do.
template <int RT, int E>
hipError_t launch_wide(const DecodeArgs& a, const DecodeSet& single, int mmax, hipStream_t st) {
    if constexpr (RT == 2) {
        if (a.k + std::min(a.k, a.n - a.k) <= 64) return launch_wide_cols<RT, E, 64>(a, single, mmax, st);
    }
    return launch_wide_cols<RT, E, kMaxN>(a, single, mmax, st);
}

}  // namespace

// The bound callers check, k st + st^2 + st doubles (st: mmax rounded up to an
// even number), is at most 128 doubles short of decode_wide_kernel's
// (k + mmax) (mmax | 1): 63 KB with the kernel's static LDS at the callers' 56.
size_t decode_lds_bytes(int k, int mmax) {
    const int st = (std::max(mmax, 1) + 1) / 2 * 2;
    return static_cast<size_t>(k * st + st * st + st) * sizeof(double);
}

// many: the sets are (part of) a batch of more than one.
static hipError_t launch_sets(const DecodeArgs& a, bool many, const DecodeSet& s, int mmax, hipStream_t st) {
    const bool vec4 = a.s % 4 == 0 && a.ldo % 4 == 0 && aligned16(a.out) && aligned16(a.Y) &&
                      (!many || a.out_stride % 4 == 0) && (a.c == nullptr || aligned16(a.c));
    // Outputs whose rows lie one after another are one column of q s elements,
    // taken four at a time at any alignment: 1000 (16,12) sets of 65536 x 1
    // 206 us one by one, 115 so; (32,24), 5000 x 5, 900 sets 85 and 48.  A single
    // set, bound by latency, spreads better over the waves one by one.
    DecodeArgs flat = a;
    flat.qb = a.qb * a.s;
    flat.q = a.q * a.s;
    flat.s = flat.ldo = 1;
    const bool dense = a.ldo == a.s && many && flat.qb >= 4;
    if (fast_path_ok(a)) {
        if (vec4) return launch_fast<4, false>(a, s, st);
        // read as a raw buffer: see ybuf in launch_fast
        if (dense && static_cast<int64_t>(a.n) * flat.qb * (a.y_f64 ? 8 : 4) < (int64_t(1) << 31))
            return launch_fast<4, true>(flat, s, st);
        return launch_fast<1, false>(a, s, st);
    }
    if (mmax > 64) return hipErrorInvalidValue;      // n <= 128: cannot be
    const DecodeArgs& w = dense ? flat : a;
    const bool four = vec4 || dense;
    if (mmax <= 16) return four ? launch_wide<1, 4>(w, s, mmax, st) : launch_wide<1, 1>(a, s, mmax, st);
    if (mmax <= 32) return four ? launch_wide<2, 4>(w, s, mmax, st) : launch_wide<2, 1>(a, s, mmax, st);
    return four ? launch_wide<4, 4>(w, s, mmax, st) : launch_wide<4, 1>(a, s, mmax, st);
}

hipError_t launch_decode(const DecodeArgs& a, const DecodeSet* single, int mmax, hipStream_t st) {
    if (a.qb * a.s > 0x7FFFFFFF) return hipErrorInvalidValue;
    DecodeSet s{};
    if (single) s = *single;
    for (int64_t b = 0; b < a.batch; b += kSetsPerLaunch) {
        DecodeArgs part = a;
        part.batch = static_cast<int32_t>(std::min(a.batch - b, kSetsPerLaunch));
        part.info = a.info + b;
        part.out = a.out + b * a.out_stride;
        if (a.sets) part.sets = a.sets + b * a.k;
        const hipError_t e = launch_sets(part, a.batch > 1, s, mmax, st);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace coded
