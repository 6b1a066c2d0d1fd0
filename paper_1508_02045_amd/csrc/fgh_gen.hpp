// fgh_gen.hpp -- passes for any odd length L = q p with q <= 17, chosen at run time.
//
// Index split (n = n1 + q n2, k = k2 + p k1), as in the size-specialised passes:
//   step A: per n1 < q a p-point DFT of the stride-q subsequence, times W_L^{n1 k2};
//   step B: per k2 < p a q-point DFT.
// Step B and, when p <= 17, step A run in registers (one DFT per thread, radix picked by a uniform
// branch).  A longer p -- a large prime factor, or a product that does not split into two radices
// -- is a dense product with the p x p DFT matrix on the matrix cores: with the sums and
// differences a_m = x_m + x_{p-m}, b_m = x_m - x_{p-m} (m <= h = (p - 1) / 2) it is two real
// (h + 1) x (h + 1) products,
//   X_k, X_{p-k} = sum_m cos(2 pi k m / p) a_m -+ i sum_m sin(2 pi k m / p) b_m,
// p multiply-adds per point instead of 4 p.  One wavefront computes 16 rows k by 16 columns
// (subsequences) in four accumulator tiles.  Those of a composite p are summed in two chains (SPLIT,
// even and odd steps): one rounds more than the short butterflies of its factors.  FP64 application
// at 441 x 441: error 5.3e-16 in one chain, 4.9e-16 in two, 4.9e-16 on the mixed-radix passes.  For a
// prime p one chain rounds less than the direct sums it replaces (511 x 509: 8.5e-16, 1.2e-15), and
// two would be up to 5 % slower (89 x 89 FP32: 22.7 -> 23.8 us).  The factors come from the length's own
// twiddle table in LDS (W_p^m = W_L^{q m}).  The direct sums ran p^2 dependent table reads per
// subsequence on one thread.  FP64 application of 201 x 151 x 101 points: 40.2 ms -> 0.406 ms, of
// 1023 x 767 points: 1.49 ms -> 0.057 ms; a CG body at 85 x 85: 262 -> 32 us.
//
// Every pass keeps its tile in one LDS buffer: a step whose outputs go to other slots than its
// inputs came from holds the outputs in registers across a barrier (a thread has one step-A
// subsequence, a wavefront up to NI products).
#pragma once
#include "fgh_v2.hpp"

namespace fgh {

constexpr int kGenRadix = 17;       // largest register radix
constexpr int kGenMaxThreads = 512;
constexpr int kGenMaxItems = 4;     // products per wavefront
constexpr int kGenSplit = 8;        // added to a kernel's NI: dense sums in two chains

#define FGH_GEN_RADICES(X) X(1) X(3) X(5) X(7) X(9) X(11) X(13) X(15) X(17)

template <typename T>
struct Mfma;
template <>
struct Mfma<double> {
    typedef double V __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V mac(double a, double b, V c)
    {
        return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return (lane >> 4) + 4 * r; }
};
template <>
struct Mfma<float> {
    typedef float V __attribute__((ext_vector_type(4)));
    static __device__ __forceinline__ V mac(float a, float b, V c)
    {
        return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
    }
    static __device__ __forceinline__ int row(int lane, int r) { return 4 * (lane >> 4) + r; }
};

// Where a tile's lines lie in LDS: element n of line l at l * PS + n * NS (complex elements).
struct Lines {
    int n;       // lines in the tile
    int PS, NS;
    float inv;   // 1 / n
};

// ------------------------------------------------------------------------------------------
// Step A in place: per (n1, line) the p-point DFT of x[n1 i1 + m im] -> slots n1 o1 + k ok, times
// W_L^{n1 k} (TW).  Forward: i1 = 1, im = q, o1 = p, ok = 1; the middle pass's way back from the
// [n1][k2] order to the natural one: i1 = p, im = 1, o1 = 1, ok = q.  All threads call it,
// synchronised; it returns synchronised.
// ------------------------------------------------------------------------------------------
template <typename T, int R, bool INV, bool TW>
__device__ __forceinline__ void step_a_reg(const cpx<T>* src, cpx<T>* dst, int is, int os, int n1, bool act,
                                           const cpx<T>* tw)
{
    cpx<T> v[R];
    if (act) {
#pragma unroll
        for (int m = 0; m < R; m++) v[m] = src[m * is];
        reg_dft<T, R, INV, true>(v);
    }
    lds_barrier();
    if (act) {
#pragma unroll
        for (int k = 0; k < R; k++) dst[k * os] = (TW && k) ? cmul(v[k], twiddle<T, INV>(tw, n1 * k)) : v[k];
    }
    lds_barrier();
}

template <typename T, bool INV, bool TW, int NI, bool SPLIT>
__device__ __forceinline__ void step_a_dense(cpx<T>* X, const Lines& ln, int i1, int im, int o1, int ok, int q, int p,
                                             const cpx<T>* tw)
{
    using V = typename Mfma<T>::V;
    const int h = (p - 1) >> 1, L = q * p;
    const int nrt = (h + 16) >> 4, ncol = q * ln.n, nct = (ncol + 15) >> 4, items = nrt * nct;
    const int wid = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, nw = (int)(blockDim.x >> 6);
    const int g = lane >> 4, j = lane & 15;
    const int is = im * ln.NS;
    V acc[NI][4];
#pragma unroll
    for (int i = 0; i < NI; i++) {
        const int it = wid + i * nw;
#pragma unroll
        for (int u = 0; u < 4; u++) acc[i][u] = V{T(0), T(0), T(0), T(0)};
        if (it < items) {
            const int ct = it / nrt, rt = it - ct * nrt;
            const int c = ct * 16 + j < ncol ? ct * 16 + j : 0;
            const int n1 = fdiv(c, ln.inv), l = c - n1 * ln.n;
            const cpx<T>* x = X + l * ln.PS + n1 * i1 * ln.NS;
            // factor index q (k m mod p) along m = g, g + 4, ...; k m <= 4 k < 4 p here
            const int k = rt * 16 + j;
            int w = k * g, st = 4 * k;
#pragma unroll
            for (int u = 0; u < 3; u++) {
                if (w >= p) w -= p;
                if (st >= p) st -= p;
            }
            w *= q;
            st *= q;
            int lo = g * is, hi = (p - g) * is;
            auto mac = [&](V* s, cpx<T> f, cpx<T> a, cpx<T> b) {
                s[0] = Mfma<T>::mac(f.x, a.x, s[0]);
                s[1] = Mfma<T>::mac(f.x, a.y, s[1]);
                s[2] = Mfma<T>::mac(f.y, b.x, s[2]);
                s[3] = Mfma<T>::mac(f.y, b.y, s[3]);
                w += st;
                if (w >= L) w -= L;
                lo += 4 * is;
                hi -= 4 * is;
            };
            auto step = [&](V* s) {
                const cpx<T> a = x[lo], b = x[hi];
                mac(s, tw[w], a + b, a - b);
            };
            const cpx<T> zero = {T(0), T(0)};
            {   // m = 0 has no mirror (its sine factor is 0)
                const cpx<T> a = x[lo], b = g ? x[hi] : zero;
                mac(acc[i], tw[w], a + b, a - b);
            }
            const int full = (h + 1) >> 2;  // steps whose four m are all <= h
            V odd[4] = {};
            if constexpr (SPLIT) {
                int s = 1;
                for (; s + 1 < full; s += 2) {
                    step(odd);
                    step(acc[i]);
                }
                if (s < full) step(odd);
            } else {
#pragma unroll 2
                for (int s = 1; s < full; s++) step(acc[i]);
            }
            if ((h + 1) & 3) {
                const bool in = 4 * full + g <= h;
                const cpx<T> a = in ? x[lo] : zero, b = in ? x[hi] : zero;
                mac(acc[i], tw[w], a + b, a - b);
            }
            if constexpr (SPLIT) {
#pragma unroll
                for (int u = 0; u < 4; u++) acc[i][u] += odd[u];
            }
        }
    }
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NI; i++) {
        const int it = wid + i * nw;
        if (it < items) {
            const int ct = it / nrt, rt = it - ct * nrt;
            const int c = ct * 16 + j;
            const int n1 = fdiv(c, ln.inv), l = c - n1 * ln.n;
            cpx<T>* y = X + l * ln.PS + n1 * o1 * ln.NS;
            if (c < ncol) {
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int k = rt * 16 + Mfma<T>::row(lane, r);
                    if (k <= h) {
                        const T cx = acc[i][0][r], cy = acc[i][1][r], sx = acc[i][2][r], sy = acc[i][3][r];
                        const cpx<T> up = {cx - sy, cy + sx}, dn = {cx + sy, cy - sx};
                        const cpx<T> v = INV ? dn : up, u = INV ? up : dn;
                        y[k * ok * ln.NS] = TW ? cmul(v, twiddle<T, INV>(tw, n1 * k)) : v;
                        if (k) y[(p - k) * ok * ln.NS] = TW ? cmul(u, twiddle<T, INV>(tw, n1 * (p - k))) : u;
                    }
                }
            }
        }
    }
    lds_barrier();
}

// LINEFAST: consecutive threads take consecutive lines (lines interleaved, PS = 1); otherwise
// consecutive n1 (lines contiguous, NS = 1).
template <typename T, bool INV, bool TW, bool LINEFAST, int NI>
__device__ __forceinline__ void step_a(cpx<T>* X, const Lines& ln, int i1, int im, int o1, int ok, const Axis& ax,
                                       const cpx<T>* tw)
{
    const int q = ax.q, p = ax.p;
    if constexpr (NI > 0) {
        step_a_dense<T, INV, TW, (NI & 7), (NI & kGenSplit) != 0>(X, ln, i1, im, o1, ok, q, p, tw);
    } else {
        const int job = threadIdx.x;
        int n1, l;
        if (LINEFAST) {
            n1 = fdiv(job, ln.inv);
            l = job - n1 * ln.n;
        } else {
            l = job / q;
            n1 = job - l * q;
        }
        const bool act = job < q * ln.n;
        if (!act) l = n1 = 0;
        const cpx<T>* src = X + l * ln.PS + n1 * i1 * ln.NS;
        cpx<T>* dst = X + l * ln.PS + n1 * o1 * ln.NS;
        switch (p) {
#define C(R) \
    case R: step_a_reg<T, R, INV, TW>(src, dst, im * ln.NS, ok * ln.NS, n1, act, tw); break;
            FGH_GEN_RADICES(C)
#undef C
        }
    }
}

// Step B in place: per (k2, line) the q-point DFT over n1 (slots n1 p + k2), which leaves the
// natural order.  The caller synchronises afterwards.
template <typename T, int R, bool INV, bool LINEFAST>
__device__ __forceinline__ void step_b_reg(cpx<T>* X, const Lines& ln, int p)
{
    const float ip = 1.0f / (float)p;
    for (int job = threadIdx.x; job < p * ln.n; job += blockDim.x) {
        const int a = fdiv(job, LINEFAST ? ln.inv : ip);
        const int b = job - a * (LINEFAST ? ln.n : p);
        const int l = LINEFAST ? b : a, k2 = LINEFAST ? a : b;
        cpx<T>* y = X + l * ln.PS + k2 * ln.NS;
        cpx<T> v[R];
#pragma unroll
        for (int n1 = 0; n1 < R; n1++) v[n1] = y[n1 * p * ln.NS];
        reg_dft<T, R, INV, true>(v);
#pragma unroll
        for (int k1 = 0; k1 < R; k1++) y[k1 * p * ln.NS] = v[k1];
    }
}
template <typename T, bool INV, bool LINEFAST>
__device__ __forceinline__ void step_b(cpx<T>* X, const Lines& ln, const Axis& ax)
{
    if (ax.q == 1) return;
    switch (ax.q) {
#define C(R) \
    case R: if constexpr (R > 1) step_b_reg<T, R, INV, LINEFAST>(X, ln, ax.p); break;
        FGH_GEN_RADICES(C)
#undef C
    }
    lds_barrier();
}

// ------------------------------------------------------------------------------------------
// Row passes.  LDS: twiddles | npen packed complex rows of L slots | phase tables.  L is odd, so
// the 16-byte slots of consecutive rows lie on different banks.
// ------------------------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ Lines row_lines(const Axis& ax, int npen)
{
    return {npen, ax.L, 1, 1.0f / (float)npen};
}

template <typename T, bool INV, int NI>
__device__ __forceinline__ void row_transform(cpx<T>* Z, const Axis& ax, int npen, const cpx<T>* tw)
{
    const Lines ln = row_lines<T>(ax, npen);
    step_a<T, INV, true, false, NI>(Z, ln, 1, ax.q, ax.p, 1, ax, tw);
    step_b<T, INV, false>(Z, ln, ax);
}

// Splits the packed spectra into the two real rows' half spectra and stores them.
template <typename T, int D>
__device__ __forceinline__ void store_half_spectra(const Geo& g, int L, cpx<T>* out, long long row0, int nrows,
                                                   const cpx<T>* Z)
{
    const int Hb = g.Hb;
    const float ih = 1.0f / (float)Hb;
    const unsigned s1 = (unsigned)g.s1;
    cpx<T>* outb = out + row0 * Hb;
    for (int idx = threadIdx.x; idx < nrows * D * Hb; idx += blockDim.x) {
        const int q = fdiv(idx, ih);
        const int k = idx - q * Hb;
        const int r = q / D, c = q - r * D;
        const cpx<T>* x = Z + (q >> 1) * L;
        const cpx<T> a = x[k], b = x[k ? L - k : 0];
        const cpx<T> v = (q & 1) ? cpx<T>{T(0.5) * (a.y + b.y), T(-0.5) * (a.x - b.x)}
                                 : cpx<T>{T(0.5) * (a.x + b.x), T(0.5) * (a.y - b.y)};
        outb[(unsigned)c * s1 + (unsigned)(r * Hb + k)] = v;
    }
}

// Loads the half spectra of a tile of rows as packed complex rows Z = A + iB with the Hermitian
// completion A(L - k) = conj A(k) (zero outside the band).
template <typename T, int D>
__device__ __forceinline__ void load_half_spectra(const Geo& g, int L, const cpx<T>* in, long long row0, int nrows,
                                                  int npen, cpx<T>* Z)
{
    constexpr int UN = 4;
    const int Hb = g.Hb, qend = nrows * D;
    const float ih = 1.0f / (float)Hb;
    const unsigned s1 = (unsigned)g.s1;
    const cpx<T>* inb = in + row0 * Hb;
    const int tot = npen * Hb;
    for (int base = threadIdx.x; base < tot; base += UN * blockDim.x) {
        cpx<T> A[UN], B[UN];
        int m[UN], k[UN];
#pragma unroll
        for (int u = 0; u < UN; u++) {
            int idx = base + u * (int)blockDim.x;
            if (idx >= tot) idx = 0;
            m[u] = fdiv(idx, ih);
            k[u] = idx - m[u] * Hb;
            const int q0 = 2 * m[u], q1 = q0 + 1;
            const int r0 = q0 / D, r1 = q1 / D;
            const unsigned o0 = q0 < qend ? (unsigned)(q0 - r0 * D) * s1 + (unsigned)(r0 * Hb + k[u]) : (unsigned)k[u];
            const unsigned o1 = q1 < qend ? (unsigned)(q1 - r1 * D) * s1 + (unsigned)(r1 * Hb + k[u]) : (unsigned)k[u];
            A[u] = inb[o0];
            B[u] = inb[o1];
            if (q0 >= qend) A[u] = {T(0), T(0)};
            if (q1 >= qend) B[u] = {T(0), T(0)};
        }
#pragma unroll
        for (int u = 0; u < UN; u++)
            if (base + u * (int)blockDim.x < tot) {
                cpx<T>* z = Z + m[u] * L;
                z[k[u]] = {A[u].x - B[u].y, A[u].y + B[u].x};
                if (k[u]) z[L - k[u]] = {A[u].x + B[u].y, B[u].x - A[u].y};
            }
    }
    const int gap = L - 2 * Hb + 1;  // positions Hb .. L - Hb outside the band
    for (int idx = threadIdx.x; idx < npen * gap; idx += blockDim.x) {
        const int m = idx / gap;
        Z[m * L + Hb + idx - m * gap] = {T(0), T(0)};
    }
}

template <typename T, int D, int NI>
__global__ __launch_bounds__(kGenMaxThreads) void kg_first(FirstArgs<T> a, int op)
{
    static_assert(kGenMaxThreads >= 2 * kThreads, "first_beta's sums share the block sum's doubles");
    __shared__ double red[kGenMaxThreads / 64];
    T beta = T(0);
    if (!(op == OP_AP_CG && a.end_part) && a.done && *a.done) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int L = a.ax.L, npen = a.npen;
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* Z = tw + L;
    T* tab = reinterpret_cast<T*>(Z + npen * L);
    const long long row0 = xcd_tile(blockIdx.x, gridDim.x) * a.rpb;
    const int nrows = (int)(a.g.rows - row0 < a.rpb ? a.g.rows - row0 : a.rpb);
    for (int m = threadIdx.x; m < L; m += blockDim.x) tw[m] = a.twg[m];
    if (a.A.kind == AK_PHASE)
        for (int m = threadIdx.x; m < kMaxPhases * 6; m += blockDim.x) tab[m] = T(a.A.tab[m / 6][m % 6]);
    if ((a.rpb * D) & 1)  // the imaginary half of the last packed row is a zero row
        for (int i = threadIdx.x; i < L; i += blockDim.x) Z[(npen - 1) * L + i].y = T(0);
    if (op == OP_AP_CG && !first_beta(a, red, &beta)) return;
    lds_barrier();
    double acc = 0.0;
    const int total = a.rpb * L, lim = nrows * L;
    const RowLen<0> rl{L, 1.0f / (float)L};
    constexpr int KU = 3;
    T* Zr = reinterpret_cast<T*>(Z);
    if (op == OP_AP_CG && a.xd) {
        for (int base = 0; base < total; base += KU * blockDim.x)
            first_stage0_chunk<T, D, 0, KU, true>(a, op, tab, beta, base, total, lim, row0 * L, Zr, rl, L, acc);
    } else {
        for (int base = 0; base < total; base += KU * blockDim.x)
            first_stage0_chunk<T, D, 0, KU>(a, op, tab, beta, base, total, lim, row0 * L, Zr, rl, L, acc);
    }
    if (sizeof(T) == 8 && op == OP_AP_CG && a.pq_part) {
        const double tot = block_sum(acc, red);
        if (threadIdx.x == 0) a.pq_part[blockIdx.x] = tot;
    }
    lds_barrier();
    row_transform<T, false, NI>(Z, a.ax, npen, tw);
    store_half_spectra<T, D>(a.g, L, a.out, row0, nrows, Z);
}

template <typename T, int D, int epi, int NI>
__global__ __launch_bounds__(kGenMaxThreads) void kg_last(LastArgs<T> a)
{
    if (a.done && *a.done) return;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kGenMaxThreads / 64];
    const int L = a.ax.L, npen = a.npen;
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* Z = tw + L;
    T* tab = reinterpret_cast<T*>(Z + npen * L);
    for (int m = threadIdx.x; m < L; m += blockDim.x) tw[m] = a.twg[m];
    if (epi == EPI_EM && a.A.kind == AK_PHASE)
        for (int m = threadIdx.x; m < kMaxPhases * 6; m += blockDim.x) tab[m] = T(a.A.tab_inv[m / 6][m % 6]);
    const long long row0 = xcd_tile(blockIdx.x, gridDim.x) * a.rpb;
    const int nrows = (int)(a.g.rows - row0 < a.rpb ? a.g.rows - row0 : a.rpb);
    load_half_spectra<T, D>(a.g, L, a.in, row0, nrows, npen, Z);
    lds_barrier();
    row_transform<T, true, NI>(Z, a.ax, npen, tw);
    const RowLen<0> rl{L, 1.0f / (float)L};
    constexpr int KU = (epi == EPI_CHEB || epi == EPI_EM || epi == EPI_CGRX) ? 2 : 3;
    double acc = 0.0;
    for (int base = 0; base < a.rpb * L; base += KU * blockDim.x)
        acc = last_epilogue_chunk<T, D, 0, epi, KU>(a, tab, base, a.rpb * L, nrows * L, row0 * L,
                                                    reinterpret_cast<const T*>(Z), rl, L, acc);
    const double tot = block_sum(acc, red);
    if (threadIdx.x == 0) {
        a.partials[blockIdx.x] = tot;
        if (a.defer_sc && blockIdx.x == 0) {
            a.defer_sc->pend = 1;
            a.defer_sc->pend_op = a.redop;
        }
    }
}

// The last pass of one loop body with the first pass of the next (Richardson, Chebyshev, Eyre-Milton),
// as k2_lastfirst: a point's update and its next z = A u are one thread's, which writes z into the
// slot its y came from; the rows are then transformed forward in place.
template <typename T, int D, int epi, int NI>
__global__ __launch_bounds__(kGenMaxThreads) void kg_lastfirst(LastArgs<T> a)
{
    if (a.done && *a.done) return;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[kGenMaxThreads / 64];
    const int L = a.ax.L, npen = a.npen;
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* Z = tw + L;
    T* tab = reinterpret_cast<T*>(Z + npen * L);
    T* tabinv = tab + kMaxPhases * 6;
    for (int m = threadIdx.x; m < L; m += blockDim.x) tw[m] = a.twg[m];
    if (a.A.kind == AK_PHASE)
        for (int m = threadIdx.x; m < kMaxPhases * 6; m += blockDim.x) {
            tab[m] = T(a.A.tab[m / 6][m % 6]);
            tabinv[m] = T(a.A.tab_inv[m / 6][m % 6]);
        }
    const long long row0 = xcd_tile(blockIdx.x, gridDim.x) * a.rpb;
    const int nrows = (int)(a.g.rows - row0 < a.rpb ? a.g.rows - row0 : a.rpb);
    load_half_spectra<T, D>(a.g, L, a.in, row0, nrows, npen, Z);
    lds_barrier();
    row_transform<T, true, NI>(Z, a.ax, npen, tw);
    const RowLen<0> rl{L, 1.0f / (float)L};
    constexpr int KU = 2;
    double acc = 0.0;
    for (int base = 0; base < a.rpb * L; base += KU * blockDim.x)
        acc += lastfirst_chunk<T, D, 0, epi, KU>(a, tab, tabinv, base, a.rpb * L, nrows * L, row0 * L,
                                                 reinterpret_cast<T*>(Z), rl, L);
    if ((a.rpb * D) & 1)  // the imaginary half of the last packed row is a zero row
        for (int i = threadIdx.x; i < L; i += blockDim.x) Z[(npen - 1) * L + i].y = T(0);
    lds_barrier();
    row_transform<T, false, NI>(Z, a.ax, npen, tw);
    store_half_spectra<T, D>(a.g, L, a.out, row0, nrows, Z);
    const double tot = block_sum(acc, red);
    if (threadIdx.x == 0) {
        a.partials[blockIdx.x] = tot;
        if (a.defer_sc && blockIdx.x == 0) {
            a.defer_sc->pend = 1;
            a.defer_sc->pend_op = a.redop;
        }
    }
}

// ------------------------------------------------------------------------------------------
// Strided axis pass (3D axis 1), one component per workgroup, tile of P columns kept column
// fastest.  NI = 0 loads the step-A subsequences from global memory straight into registers.
// ------------------------------------------------------------------------------------------
template <typename T, int R, bool INV>
__device__ __forceinline__ void axis_a_reg(const AxisArgs<T>& a, const cpx<T>* in, int B, int j0, float iP,
                                           const cpx<T>* tw, cpx<T>* X)
{
    const int P = a.P, q = a.ax.q, L = a.ax.L;
    const bool banded = a.bin && B != L;
    for (int job = threadIdx.x; job < q * P; job += blockDim.x) {
        const int n1 = fdiv(job, iP), col = job - n1 * P;
        const bool inr = j0 + col < a.inner;
        const int j = inr ? j0 + col : j0;
        cpx<T> v[R];
#pragma unroll
        for (int m = 0; m < R; m++) {
            int s = n1 + q * m;
            const bool ok = banded ? band_index(s, L, B, &s) : true;
            v[m] = ok ? in[(unsigned)(s * a.inner + j)] : cpx<T>{T(0), T(0)};
        }
        reg_dft<T, R, INV, true>(v);
        cpx<T>* y = X + n1 * R * P + col;
#pragma unroll
        for (int k = 0; k < R; k++) y[k * P] = k ? cmul(v[k], twiddle<T, INV>(tw, n1 * k)) : v[k];
    }
}

template <typename T, int R, bool INV>
__device__ __forceinline__ void axis_b_reg(const AxisArgs<T>& a, cpx<T>* out, int B, int j0, float iP,
                                           const cpx<T>* X)
{
    const int P = a.P, p = a.ax.p, L = a.ax.L;
    const bool banded = a.bout && B != L;
    for (int job = threadIdx.x; job < p * P; job += blockDim.x) {
        const int k2 = fdiv(job, iP), col = job - k2 * P;
        const int j = j0 + col;
        const cpx<T>* y = X + job;  // slot k2 P + col
        cpx<T> v[R];
#pragma unroll
        for (int n1 = 0; n1 < R; n1++) v[n1] = y[n1 * p * P];
        reg_dft<T, R, INV, true>(v);
        if (j < a.inner) {
#pragma unroll
            for (int k1 = 0; k1 < R; k1++) {
                int s = k2 + p * k1;
                if (banded && !band_index(s, L, B, &s)) continue;
                out[(unsigned)(s * a.inner + j)] = v[k1];
            }
        }
    }
}

template <typename T, bool INV, int NI>
__global__ __launch_bounds__(kGenMaxThreads) void kg_axis(AxisArgs<T> a, int B)
{
    int b = blockIdx.x;
    if (!INV && a.pending && (b -= Pending::kBlocks) < 0) return finish_pending(a.pend, b + Pending::kBlocks);
    if (stopped(a.done)) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int L = a.ax.L, P = a.P, q = a.ax.q, p = a.ax.p;
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* X = tw + L;
    const int gx = a.ntiles, gy = a.outer;
    const long long lin = xcd_tile(b, (long long)gx * gy * a.comps);
    const int tile = (int)(lin % gx);
    const int o = (int)((lin / gx) % gy);
    const int c = (int)(lin / ((long long)gx * gy));
    for (int m = threadIdx.x; m < L; m += blockDim.x) tw[m] = a.twg[m];
    const cpx<T>* in = a.in + c * a.in_cs + o * a.in_os;
    cpx<T>* out = a.out + c * a.out_cs + o * a.out_os;
    const int j0 = tile * P;
    const float iP = 1.0f / (float)P;
    if constexpr (NI == 0) {
        lds_barrier();
        switch (p) {
#define C(R) \
    case R: axis_a_reg<T, R, INV>(a, in, B, j0, iP, tw, X); break;
            FGH_GEN_RADICES(C)
#undef C
        }
        lds_barrier();
    } else {
        constexpr int UN = 8;
        const bool banded = a.bin && B != L;
        const int tot = L * P;
        for (int base = threadIdx.x; base < tot; base += UN * blockDim.x) {
            cpx<T> v[UN];
#pragma unroll
            for (int u = 0; u < UN; u++) {
                const int idx = base + u * (int)blockDim.x;
                int s = fdiv(idx, iP);
                const int col = idx - s * P;
                bool ok = idx < tot && j0 + col < a.inner;
                if (banded && ok) ok = band_index(s, L, B, &s);
                v[u] = in[ok ? (unsigned)(s * a.inner + j0 + col) : 0u];
                if (!ok) v[u] = {T(0), T(0)};
            }
#pragma unroll
            for (int u = 0; u < UN; u++)
                if (base + u * (int)blockDim.x < tot) X[base + u * (int)blockDim.x] = v[u];
        }
        lds_barrier();
        step_a<T, INV, true, true, NI>(X, Lines{P, 1, P, iP}, 1, q, p, 1, a.ax, tw);
    }
    switch (q) {
#define C(R) \
    case R: axis_b_reg<T, R, INV>(a, out, B, j0, iP, X); break;
        FGH_GEN_RADICES(C)
#undef C
    }
}

// ------------------------------------------------------------------------------------------
// Middle pass along axis 0, in place on the spectrum.  G^ is rank one per frequency, G^ z = k t
// with t = k.z / |k|^2, and only k_0 varies along a column: two lines per column are enough, z_0 and
// z' = sum_{c>=1} k_c z_c, combined while loading; they leave as z_0' = IDFT(k_0 t) and
// t' = IDFT(t), the components c >= 1 being k_c t' (in 2D the second line is z_1 itself, and k_1 is
// applied with the multiplier).  Eyre-Milton's I - 2 G^ is the input times the
// transform pair's factor minus twice that, the input being read again when storing.
// Lines: column col of line pair member s at s P + col (column fastest).
// ------------------------------------------------------------------------------------------
// 1 / v for a positive integer v, rounded about once (a last Newton step on the exact remainder; a
// float holds v in two parts, since |k|^2 has up to 26 bits).  The bare hardware reciprocal of the
// rounded |k|^2 is as fast; FP32 errors of whole applications with it and with this one: 441 x 441
// 2.42e-7 and 2.41e-7, 1023 x 767 2.51e-7 both.
__device__ __forceinline__ void recip_exact(int v, double* r)
{
    const double x = (double)v, r0 = recip_int(x);
    *r = fma(fma(-x, r0, 1.0), r0, r0);
}
__device__ __forceinline__ void recip_exact(int v, float* r)
{
    const float hi = (float)v, lo = (float)(v - (int)hi), r0 = recip_int(hi);
    *r = fmaf(fmaf(-lo, r0, fmaf(-hi, r0, 1.0f)), r0, r0);
}

// Column j of the middle pass: |k|^2 without k_0.
template <typename T, int D>
__device__ __forceinline__ int column_kperp(const MidArgs<T>& a, int j)
{
    int kv1 = j, kv2 = 0;
    if (D == 3) {
        const int kb1 = j / a.Hb;
        kv1 = signed_index(kb1, a.B1);
        kv2 = j - kb1 * a.Hb;
    }
    return kv1 * kv1 + kv2 * kv2;
}

// scale / |k|^2 of frequency k_0: 0 at k = 0 (G^ vanishes there) and outside the band (Ga).
template <typename T>
__device__ __forceinline__ T mid_weight(const MidArgs<T>& a, int k0, int kperp, bool colok)
{
    const bool inband = colok && (2 * (k0 < 0 ? -k0 : k0) < a.B0);
    const int kk = k0 * k0 + kperp;
    T r;
    recip_exact(kk, &r);
    return (inband && kk > 0) ? T(a.scale) * r : T(0);
}

// Step B, the multiplier and the inverse step B in one thread: the two lines of a (k2, column) take
// 2 q complex registers, which fits three wavefronts per SIMD in double precision up to q = 9.
constexpr int kMidFusedRadix = 9;
template <typename T, int D, int R>
__device__ __forceinline__ void mid_b_reg(const MidArgs<T>& a, int j0, float iP, const cpx<T>* tw, cpx<T>* X)
{
    const int P = a.P, p = a.ax.p, L = a.ax.L, NS = 2 * P;
    for (int job = threadIdx.x; job < p * P; job += blockDim.x) {
        const int k2 = fdiv(job, iP), col = job - k2 * P;
        const int j = j0 + col;
        const int kperp = column_kperp<T, D>(a, j);
        const T kl = D == 2 ? T(j) : T(1);
        cpx<T>* y = X + k2 * NS + col;
        cpx<T> z0[R], zp[R];
#pragma unroll
        for (int n1 = 0; n1 < R; n1++) {
            z0[n1] = y[n1 * p * NS];
            zp[n1] = y[n1 * p * NS + P];
        }
        reg_dft<T, R, false, true>(z0);
        reg_dft<T, R, false, true>(zp);
#pragma unroll
        for (int k1 = 0; k1 < R; k1++) {
            const int k0 = signed_index(k2 + p * k1, L);
            const cpx<T> t = mid_weight<T>(a, k0, kperp, j < a.cols) * (T(k0) * z0[k1] + kl * zp[k1]);
            zp[k1] = kl * t;
            z0[k1] = T(k0) * t;
        }
        reg_dft<T, R, true, true>(z0);
        reg_dft<T, R, true, true>(zp);
#pragma unroll
        for (int n1 = 0; n1 < R; n1++) {
            const cpx<T> w = conj(tw[n1 * k2]);
            y[n1 * p * NS] = n1 ? cmul(z0[n1], w) : z0[n1];
            y[n1 * p * NS + P] = n1 ? cmul(zp[n1], w) : zp[n1];
        }
    }
}

// The same in three steps through LDS, one line per thread at a time, for larger q.
template <typename T, int R>
__device__ __forceinline__ void mid_binv_reg(cpx<T>* X, const Lines& ln, int p, const cpx<T>* tw)
{
    for (int job = threadIdx.x; job < p * ln.n; job += blockDim.x) {
        const int k2 = fdiv(job, ln.inv);
        cpx<T>* y = X + job;  // slot k2 NS + line, NS = lines
        cpx<T> v[R];
#pragma unroll
        for (int k1 = 0; k1 < R; k1++) v[k1] = y[k1 * p * ln.NS];
        reg_dft<T, R, true, true>(v);
#pragma unroll
        for (int n1 = 0; n1 < R; n1++) y[n1 * p * ln.NS] = n1 ? cmul(v[n1], conj(tw[n1 * k2])) : v[n1];
    }
}

template <typename T, int D>
__device__ __forceinline__ void mid_b_split(const MidArgs<T>& a, int j0, float iP, const Lines& ln, const cpx<T>* tw,
                                            cpx<T>* X)
{
    step_b<T, false, true>(X, ln, a.ax);
    const int P = a.P, L = a.ax.L;
    for (int idx = threadIdx.x; idx < L * P; idx += blockDim.x) {
        const int pos = fdiv(idx, iP), col = idx - pos * P;
        const int j = j0 + col;
        const int k0 = signed_index(pos, L);
        cpx<T>* y = X + pos * ln.NS + col;
        const T kl = D == 2 ? T(j) : T(1);
        const cpx<T> t = mid_weight<T>(a, k0, column_kperp<T, D>(a, j), j < a.cols) * (T(k0) * y[0] + kl * y[P]);
        y[0] = T(k0) * t;
        y[P] = kl * t;
    }
    lds_barrier();
    switch (a.ax.q) {
#define C(R)     case R: if constexpr (R > kMidFusedRadix) mid_binv_reg<T, R>(X, ln, a.ax.p, tw); break;
        FGH_GEN_RADICES(C)
#undef C
    }
}

template <typename T, int D, int MULT, int NI>
__global__ __launch_bounds__(kGenMaxThreads) void kg_middle(MidArgs<T> a)
{
    int b = blockIdx.x;
    if (D == 2 && a.pending && (b -= Pending::kBlocks) < 0) return finish_pending(a.pend, b + Pending::kBlocks);
    if (stopped(a.done)) return;
    extern __shared__ __align__(16) unsigned char smem[];
    const int L = a.ax.L, P = a.P, q = a.ax.q, p = a.ax.p, NS = 2 * P;
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* X = tw + L;
    const int j0 = (int)xcd_tile(b, a.ntiles) * P;
    for (int m = threadIdx.x; m < L; m += blockDim.x) tw[m] = a.twg[m];
    const float iP = 1.0f / (float)P;
    const int tot = L * P;
    // 3D: wave numbers k_1, k_2 of a column
    auto kc = [&](int j, T* k) {
        const int kb1 = j / a.Hb;
        k[0] = T(signed_index(kb1, a.B1));
        k[1] = T(j - kb1 * a.Hb);
    };
    constexpr int UN = 4;
    for (int base = threadIdx.x; base < tot; base += UN * blockDim.x) {
        cpx<T> z[UN][D];
#pragma unroll
        for (int u = 0; u < UN; u++) {
            const int idx = base + u * (int)blockDim.x;
            const int s = fdiv(idx, iP);
            const int j = j0 + idx - s * P;
            const bool ok = idx < tot && j < a.cols;
#pragma unroll
            for (int c = 0; c < D; c++) {
                z[u][c] = (a.buf + c * a.cs)[ok ? (unsigned)(s * a.cols + j) : 0u];
                if (!ok) z[u][c] = {T(0), T(0)};
            }
        }
#pragma unroll
        for (int u = 0; u < UN; u++) {
            const int idx = base + u * (int)blockDim.x;
            if (idx < tot) {
                const int s = fdiv(idx, iP);
                const int col = idx - s * P;
                cpx<T> zp = z[u][1];
                if (D == 3) {
                    T k[2];
                    kc(j0 + col, k);
                    zp = k[0] * zp + k[1] * z[u][D - 1];
                }
                X[s * NS + col] = z[u][0];
                X[s * NS + P + col] = zp;
            }
        }
    }
    lds_barrier();
    const Lines ln{2 * P, 1, NS, 1.0f / (float)(2 * P)};
    step_a<T, false, true, true, NI>(X, ln, 1, q, p, 1, a.ax, tw);
    if (q > kMidFusedRadix) {
        mid_b_split<T, D>(a, j0, iP, ln, tw, X);
    } else {
        switch (q) {
#define C(R) \
    case R: if constexpr (R <= kMidFusedRadix) mid_b_reg<T, D, R>(a, j0, iP, tw, X); break;
            FGH_GEN_RADICES(C)
#undef C
        }
    }
    lds_barrier();
    step_a<T, true, false, true, NI>(X, ln, p, 1, 1, q, a.ax, tw);
    const T keep = T(a.scale) * T(L);  // Eyre-Milton: the factor of the input
    for (int idx = threadIdx.x; idx < tot; idx += blockDim.x) {
        const int s = fdiv(idx, iP);
        const int col = idx - s * P;
        const int j = j0 + col;
        if (j < a.cols) {
            cpx<T> v[3];
            v[0] = X[s * NS + col];
            v[1] = X[s * NS + P + col];
            if (D == 3) {
                T k[2];
                kc(j, k);
                v[D - 1] = k[1] * v[1];
                v[1] = k[0] * v[1];
            }
#pragma unroll
            for (int c = 0; c < D; c++) {
                cpx<T>* o = a.buf + c * a.cs + (unsigned)(s * a.cols + j);
                *o = MULT == MULT_EM ? keep * *o - T(2) * v[c] : v[c];
            }
        }
    }
}

}  // namespace fgh
