// Monte-Carlo of the runtime model (Sec. III-B to III-D): for each draw the
// n worker samples T0_i = shift - ln(U_i) / rate come from the counter-based
// SplitMix64 word of (draw, worker), as in the survivor draw, and the job's
// overall runtime is formed for three schemes from the same samples:
//   uncoded      n subtasks of T0/n, the slowest one (eq. uncoded);
//   repetition   k subtasks of T0/k, each on n/k consecutive workers, the
//                slowest task's fastest replica (eq. rep_coded);
//   MDS (n,k)    subtasks of T0/k, the k-th finisher (eq. mds_coded).
// T0 falls as the word grows, so every order statistic is taken on the words'
// top 53 bits (U's bits) and only the selected one goes through the logarithm.
//
// Bound by vector issue: about 19 instructions per word, then the order
// statistics.  One thread per draw, the words in registers, sorted by a
// network of compare-exchanges (Batcher's merge exchange, Knuth vol. 3,
// Algorithm 5.2.2M, which takes any n): n log^2 n / 4 exchanges of two
// instructions, where counting ranks takes n (n - 1) compares of three.  A
// value below 2^53 read as the bits of a double is zero, subnormal or small
// and normal, and doubles of one sign order as their bits do, so an exchange
// is one v_min_f64 and one v_max_f64 (full rate, as every instruction here).
// (10,5), 2^24 draws, three schemes: 266 us, 420 by ranks; (64,48), 2^20 draws:
// 85 us, 2430 by ranks over words formed again for every compare.
// Past 64 workers 53-bit values no longer fit the registers: there the network
// sorts 32-bit keys, the words' top 25 bits with the worker's index below, and
// the selected worker's word is formed again; when a neighbour shares the 25
// bits (about 1e-5 of the draws) the lane ranks those few words exactly.
#include <type_traits>
#include <utility>

#include "internal.h"

namespace coded {
namespace {

constexpr uint64_t kGamma = 0x9E3779B97F4A7C15ull;
constexpr uint64_t kRuntimeStream = 4;

// SplitMix64 output of counter c is mix(seed + (c + 1) * gamma).  With the
// counter 4 << 56 | draw << 16 | worker (worker < 2^16, so the OR is a sum)
// the state is base(draw) + worker * gamma, modulo 2^64.
__device__ inline uint64_t mix(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ inline uint64_t base_of(uint64_t seed, uint64_t draw) {
    return seed + (((kRuntimeStream << 56) | (draw << 16)) + 1) * kGamma;
}

__device__ inline uint64_t word_of(uint64_t base, int worker) {
    return mix(base + static_cast<uint64_t>(worker) * kGamma);
}

// Constants of a launch: division by rate, n and k as a product with the
// reciprocal and one exact-residual correction (Markstein's step, which rounds
// as the division does), unless rate is so far from one that the steps could
// overflow (`plain`).
struct SimConst {
    double shift, rate, inv_rate, nn, inv_n, kk, inv_k;
    int32_t plain;
};
__device__ inline double divide(double x, double d, double inv) {
    const double q = x * inv;
    return fma(fma(-q, d, x), inv, q);
}
// T0 of a word's top 53 bits.
__device__ inline double mother(uint64_t top, const SimConst& c) {
    const double u = (static_cast<double>(top) + 0.5) * 0x1.0p-53;
    const double l = log(u);
    return c.shift - (c.plain ? l / c.rate : divide(l, c.rate, c.inv_rate));
}

// "a finishes no later than b": larger word, then lower index.
__device__ inline bool before(uint64_t ua, int a, uint64_t ub, int b) { return ua > ub || (ua == ub && a < b); }

__device__ inline double as_key(uint64_t top) { return __longlong_as_double(static_cast<long long>(top)); }
__device__ inline uint64_t key_bits(double v) { return static_cast<uint64_t>(__double_as_longlong(v)); }
// v_min / v_max without the compiler's quieting of possible signalling NaNs
// (there are none), which would add an instruction per word.
__device__ inline double kmin(double a, double b) {
    double r;
    asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline double kmax(double a, double b) {
    double r;
    asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ inline void exchange(double& a, double& b) {
    const double lo = kmin(a, b), hi = kmax(a, b);
    a = lo;
    b = hi;
}
__device__ inline void exchange(uint32_t& a, uint32_t& b) {
    const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
    a = lo;
    b = hi;
}

// The exchanges (i, j), i < j, of the network for N values, ascending.
template <int N>
struct Network {
    struct Pair {
        int16_t a, b;
    };
    template <typename F>
    static constexpr void each(F f) {
        int t = 0;
        while ((1 << t) < N) ++t;
        if (t == 0) return;
        for (int p = 1 << (t - 1); p > 0; p >>= 1) {
            int q = 1 << (t - 1), r = 0, d = p;
            while (true) {
                for (int i = 0; i < N - d; ++i)
                    if ((i & p) == r) f(i, i + d);
                if (q == p) break;
                d = q - p;
                q >>= 1;
                r = p;
            }
        }
    }
    static constexpr int count() {
        int c = 0;
        each([&](int, int) { ++c; });
        return c;
    }
    struct Table {
        Pair at[count() > 0 ? count() : 1];
    };
    static constexpr Table make() {
        Table tb{};
        int c = 0;
        each([&](int i, int j) {
            tb.at[c].a = static_cast<int16_t>(i);
            tb.at[c].b = static_cast<int16_t>(j);
            ++c;
        });
        return tb;
    }
};
template <int N>
constexpr auto kTable = Network<N>::make();
template <int A, int B, int N, typename T>
__device__ __forceinline__ int step(T (&v)[N]) {
    exchange(v[A], v[B]);
    return 0;
}
template <int N, typename T, int... I>
__device__ __forceinline__ void sort_steps(T (&v)[N], std::integer_sequence<int, I...>) {
    const int done[] = {0, step<kTable<N>.at[I].a, kTable<N>.at[I].b>(v)...};
    (void)done;
}
template <int N, typename T>
__device__ __forceinline__ void sort_network(T (&v)[N]) {
    sort_steps(v, std::make_integer_sequence<int, Network<N>::count()>{});
}

// v[idx], idx the same in every lane, by halving (every register index constant).
template <int N, typename T>
__device__ __forceinline__ T pick(const T (&v)[N], int idx) {
    if constexpr (N == 1) {
        return v[0];
    } else {
        T h[(N + 1) / 2];
        const bool odd = idx & 1;
#pragma unroll
        for (int i = 0; i < (N + 1) / 2; ++i) {
            const T even = v[2 * i], next = v[2 * i + 1 < N ? 2 * i + 1 : 2 * i];
            h[i] = odd ? next : even;
        }
        return pick(h, idx >> 1);
    }
}

// The k-th largest word by exact ranks among the words that share the top 25
// bits `tk`; the words with larger ones come first.
__device__ inline uint64_t ranked_word(uint64_t base, int n, int k, uint32_t tk) {
    int above = 0;
    for (int i = 0; i < n; ++i) above += static_cast<uint32_t>(word_of(base, i) >> 39) > tk;
    uint64_t got = 0;
    for (int i = 0; i < n; ++i) {
        const uint64_t ui = word_of(base, i);
        if (static_cast<uint32_t>(ui >> 39) != tk) continue;
        int rank = above;
        for (int j = 0; j < n; ++j) {
            const uint64_t uj = word_of(base, j);
            rank += j != i && static_cast<uint32_t>(uj >> 39) == tk && before(uj, j, ui, i);
        }
        if (rank == k - 1) got = ui;
    }
    return got;
}

// N >= n values per draw; more than LOW of them are real.
template <int N, int LOW>
__global__ __launch_bounds__(256) void runtime_sim_kernel(int n, int k, uint64_t seed, uint64_t first_draw, int64_t count,
                                                          SimConst c, double* t_unc, double* t_rep, double* t_mds) {
    const int64_t d = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
    if (d >= count) return;
    const uint64_t base = base_of(seed, first_draw + static_cast<uint64_t>(d));
    constexpr bool kWide = N > 64;
    constexpr int kBlock = kWide ? 8 : N;              // words formed together
    using V = std::conditional_t<kWide, uint32_t, double>;
    V v[N];
    // slowest worker: the smallest word; repetition: per task (n/k consecutive
    // workers) the largest word, then the smallest of those
    const double top = as_key((1ull << 53) - 1);
    double slow = top, worst = top, best = 0.0;
    const int g = n / k;
    int pos = 0;
    uint64_t state = base;
#pragma unroll
    for (int b = 0; b < N; b += kBlock) {
        // no branches between the words' chains, so they overlap
        double key[kBlock];
#pragma unroll
        for (int i = b; i < b + kBlock && i < N; ++i) {
            const uint64_t w = mix(state);
            // the next state by one addition (left alone it is multiplied out again)
            asm volatile("" : "+v"(state));
            state += kGamma;
            key[i - b] = as_key(w >> 11);
            // values past n sort below every real one (or equal to it)
            const bool real = i <= LOW || i < n;
            if constexpr (kWide)
                v[i] = real ? (static_cast<uint32_t>(w >> 32) & ~127u) | i : 0u;
            else
                v[i] = real ? key[i - b] : 0.0;
        }
        if (t_unc) {
#pragma unroll
            for (int i = b; i < b + kBlock && i < N; ++i)
                if (i <= LOW || i < n) slow = kmin(slow, key[i - b]);
        }
        if (t_rep) {
#pragma unroll
            for (int i = b; i < b + kBlock && i < N; ++i) {
                if (i <= LOW || i < n) {
                    best = kmax(best, key[i - b]);
                    if (++pos == g) {
                        worst = kmin(worst, best);
                        best = 0.0;
                        pos = 0;
                    }
                }
            }
        }
    }
    if (t_unc) {
        const double t0 = mother(key_bits(slow), c);
        t_unc[d] = c.plain ? t0 / c.nn : divide(t0, c.nn, c.inv_n);
    }
    if (t_rep) {
        const double t0 = mother(key_bits(worst), c);
        t_rep[d] = c.plain ? t0 / c.kk : divide(t0, c.kk, c.inv_k);
    }
    if (t_mds) {
        // the k-th finisher: the k-th largest word
        sort_network(v);
        uint64_t sel;
        if constexpr (kWide) {
            const uint32_t s = pick(v, N - k);
            const uint32_t up = k > 1 ? pick(v, N - k + 1) : ~s, down = k < n ? pick(v, N - k - 1) : ~s;
            uint64_t w = word_of(base, static_cast<int>(s & 127u));
            if ((up ^ s) < 128u || (down ^ s) < 128u) w = ranked_word(base, n, k, s >> 7);
            sel = w >> 11;
        } else {
            sel = key_bits(pick(v, N - k));
        }
        const double t0 = mother(sel, c);
        t_mds[d] = c.plain ? t0 / c.kk : divide(t0, c.kk, c.inv_k);
    }
}

template <int N, int LOW>
hipError_t launch_sim(int n, int k, uint64_t seed, uint64_t first, int64_t count, const SimConst& c, double* tu,
                      double* tr, double* tm, hipStream_t st) {
    // a grid takes fewer than 2^32 draws
    constexpr int64_t kMost = int64_t(1) << 31;
    for (int64_t d = 0; d < count; d += kMost) {
        const int64_t part = count - d < kMost ? count - d : kMost, blocks = ceil_div(part, 256);
        if (!grid_fits(blocks, 256)) return hipErrorInvalidConfiguration;
        hipLaunchKernelGGL((runtime_sim_kernel<N, LOW>), dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, n, k, seed,
                           first + static_cast<uint64_t>(d), part, c, tu ? tu + d : nullptr, tr ? tr + d : nullptr,
                           tm ? tm + d : nullptr);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// The smallest instance of N, ... that holds n.
template <int PREV, int N, int... MORE>
hipError_t launch_fit(int n, int k, uint64_t seed, uint64_t first, int64_t count, const SimConst& c, double* tu,
                      double* tr, double* tm, hipStream_t st) {
    if constexpr (sizeof...(MORE) > 0) {
        if (n > N) return launch_fit<N, MORE...>(n, k, seed, first, count, c, tu, tr, tm, st);
    }
    return launch_sim<N, PREV>(n, k, seed, first, count, c, tu, tr, tm, st);
}

}  // namespace

hipError_t launch_runtime_sim(int n, int k, uint64_t seed, uint64_t first, int64_t count, double shift, double rate,
                              double* tu, double* tr, double* tm, hipStream_t st) {
    static_assert(kMaxN <= 128, "worker indices take 7 bits of the sorting keys");
    if (count == 0) return hipSuccess;
    SimConst c{};
    c.shift = shift;
    c.rate = rate;
    c.inv_rate = 1.0 / rate;
    c.nn = n;
    c.inv_n = 1.0 / n;
    c.kk = k;
    c.inv_k = 1.0 / k;
    c.plain = !(rate > 1e-100 && rate < 1e100 && shift > -1e100 && shift < 1e100);
    // Exact sizes while a padding value costs most of an exchange layer, then
    // steps of at most a seventh.
    return launch_fit<0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16, 18, 20, 22, 24, 28, 32, 36, 40, 48, 56, 64,
                      72, 84, 96, 112, 128>(n, k, seed, first, count, c, tu, tr, tm, st);
}

}  // namespace coded
