// fgh_v2.hpp -- size-specialised passes: compile-time length L = L1 * L2, register-resident DFTs.
//
// Index split (n = n1 + L1 n2, k = k2 + L2 k1):
//   X[k2 + L2 k1] = sum_{n1} W_L1^{n1 k1} W_L^{n1 k2} sum_{n2} W_L2^{n2 k2} x[n1 + L1 n2]
// Step A: per n1, an L2-point DFT of the stride-L1 subsequence, times W_L^{n1 k2}; step B: per
// k2, an L1-point DFT.  Both DFTs run in registers (compound sizes recurse on the same split with
// compile-time roots), so a pass moves its tile global -> registers -> LDS -> registers -> global:
// one LDS exchange and one barrier per pass (two in the middle pass, whose forward step B, the
// Fourier multiplier and the inverse step B all stay in registers).
#pragma once
#include <hip/hip_runtime.h>

#include "fgh_args.hpp"

namespace fgh {

// 1 / v for an exact positive integer v: the hardware reciprocal, refined by one Newton step in
// double precision (relative error a few units in the last place).
__device__ __forceinline__ float recip_int(float v) { return __builtin_amdgcn_rcpf(v); }
__device__ __forceinline__ double recip_int(double v)
{
    const double r = __builtin_amdgcn_rcp(v);
    return fma(fma(-v, r, 1.0), r, r);
}

// Workgroup barrier that orders LDS accesses only.  Threads of one launch exchange data through
// LDS alone, so global loads issued before the barrier (prefetches of the next tile) stay in
// flight across it, and global stores are not waited for.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The loop's stop flag, for the passes that may run beside the workgroup that sets it (Pending).  A
// relaxed atomic, and so a vector load: a scalar load in every workgroup cost 1 % of the strided
// passes (243^3 FP64 141.2 -> 142.6 us, a CG body 1111 -> 1116 us).
__device__ __forceinline__ bool stopped(const int* done)
{
    return done && __hip_atomic_load(done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// What ends a loop whose stopping-test value (raw sum) is v after its next body: 0 nothing, else
// Scalars::done.
__device__ __forceinline__ int end_state(const Scalars* s, double v)
{
    const double q = sqrt(v / s->npts);
    if (!(v == v) || v > 1.0e300 || (s->blowup > 0.0 && q > s->blowup)) return 3;
    if (s->thr >= 0.0 && q <= s->thr) return 1;
    return s->m + 1 >= s->limit ? 2 : 0;
}

__device__ __forceinline__ void end_body(Scalars* s, double v)
{
    const int d = end_state(s, v);
    s->m += 1;
    s->last = sqrt(v / s->npts);
    if (d) s->done = d;
}

// The scalar update that ends a loop reduction (RedOp) from its total.
__device__ __forceinline__ void apply_redop(Scalars* s, int op, double tot)
{
    s->total = tot;
    if (op == RED_CG_ALPHA) {
        s->qp = tot;
        s->alpha = s->rr / tot;
    } else if (op == RED_CG_END) {
        s->rr_new = tot;
        s->beta = tot / s->rr;
        s->rr = tot;
        end_body(s, tot);
    } else if (op == RED_SET_RR) {
        s->rr = tot;
    } else if (op == RED_STEP_END) {
        end_body(s, tot);
    } else if (op == RED_CHEB_END) {
        end_body(s, tot);
        // Algorithm 3: alpha, beta of the next body
        const double al = 1.0 / (s->cheb_delta + s->beta / s->alpha);
        s->alpha = al;
        s->beta = -(s->cheb_c * al * 0.5) * (s->cheb_c * al * 0.5);
    }
}

// Sums of two arrays of partial sums (na and nb of them, 0 allowed), the same in every thread and
// whatever the workgroup's size: the order is that of kThreads threads (thread t sums t,
// t + kThreads, ...), each wavefront's shuffle tree, then the wavefronts in turn.  Loads are issued
// eight at a time, and both arrays' first ones together, so that one memory latency covers them.
// All threads of the workgroup call it; red: 2 kThreads / 64 doubles of LDS that are free on entry.
__device__ __forceinline__ double partial_share(const double* p, int n, int i)
{
    double v = 0.0;
    for (; i + 7 * kThreads < n; i += 8 * kThreads) {
        double t[8];
#pragma unroll
        for (int u = 0; u < 8; u++) t[u] = p[i + u * kThreads];
#pragma unroll
        for (int u = 0; u < 8; u++) v += t[u];
    }
    if (i < n) {
        double t[7];
#pragma unroll
        for (int u = 0; u < 7; u++) t[u] = i + u * kThreads < n ? p[i + u * kThreads] : 0.0;
#pragma unroll
        for (int u = 0; u < 7; u++)
            if (i + u * kThreads < n) v += t[u];
    }
    return v;
}
__device__ __forceinline__ void sum_partials2(const double* a, int na, const double* b, int nb, double* red,
                                              double* sa, double* sb)
{
    constexpr int W = kThreads / 64;
    const int lane = threadIdx.x & 63, nw = (int)blockDim.x >> 6;
    for (int w = (int)threadIdx.x >> 6; w < W; w += nw) {
        double va = partial_share(a, na, w * 64 + lane), vb = partial_share(b, nb, w * 64 + lane);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            va += __shfl_down(va, off, 64);
            vb += __shfl_down(vb, off, 64);
        }
        if (lane == 0) {
            red[w] = va;
            red[W + w] = vb;
        }
    }
    __syncthreads();
    *sa = *sb = 0.0;
#pragma unroll
    for (int w = 0; w < W; w++) {
        *sa += red[w];
        *sb += red[W + w];
    }
}
__device__ __forceinline__ double sum_partials(const double* p, int n, double* red)
{
    double s, none;
    sum_partials2(p, n, p, 0, red, &s, &none);
    return s;
}

// Completes the pending loop reductions in their own workgroup (b < Pending::kBlocks of the launch;
// the first does it).  The partial sums were written by
// earlier kernels, so no fence or counter is needed.  Same summation order and scalar update as
// the separate reduction kernel.  The sums are taken whether or not an end is pending, so that their
// loads do not wait for the flag.  The sums use the tile's LDS (Pending::kLds bytes of it at least),
// so that the tiles' workgroups declare none beside it.
__device__ __forceinline__ void finish_pending(const Pending& p, int b)
{
    if (b) return;
    extern __shared__ __align__(16) unsigned char smem[];
    double* red = reinterpret_cast<double*>(smem);
    Scalars* s = p.sc;
    double end, pq;
    sum_partials2(p.end, p.nend, p.pq, p.npq, red, &end, &pq);
    if (threadIdx.x == 0) {
        if (s->pend) {
            apply_redop(s, s->pend_op, end);
            s->pend = 0;
        }
        if (p.npq && !s->done) apply_redop(s, RED_CG_ALPHA, pq);
    }
}

// CG's beta for the first pass: from the scalar block, or, while the previous body's end is
// pending, from the partial sums of its (r, r), which every workgroup adds up for itself.  Returns
// false where the loop has stopped or that end stops it (the next kernel records it): nothing is
// to be done then.
template <typename T>
__device__ __forceinline__ bool first_beta(const FirstArgs<T>& a, double* red, T* beta)
{
    const Scalars* s = a.sc;
    double b = s->beta;
    if (a.end_part) {  // the sums' loads do not wait for the flags
        const double tot = sum_partials(a.end_part, a.nend, red);
        if (*a.done) return false;
        if (s->pend) {
            if (end_state(s, tot)) return false;
            b = tot / s->rr;
        }
    }
    *beta = T(b);
    return true;
}

constexpr int smallest_factor(int n)
{
    for (int p = 2; p * p <= n; p++)
        if (n % p == 0) return p;
    return n;
}

// cos and sin of 2 pi m / R for 0 < m <= (R - 1) / 2, rounded once.
template <int R>
__device__ __forceinline__ constexpr double exact_cos(int m)
{
    constexpr double t[][8] = {
        {0.766044443118978035202393, 0.173648177666930348851717, -0.5, -0.939692620785908384054109},
        {0.841253532831181168861812, 0.415415013001886425529274, -0.142314838273285140443793, -0.654860733945285064056925,
         -0.959492973614497389890368},
        {0.885456025653209895900376, 0.568064746731155802511808, 0.120536680255323053349068, -0.354604887042535625969638,
         -0.748510748171101098634631, -0.970941817426052027156982},
        {0.913545457642600895502128, 0.669130606358858213826273, 0.309016994374947424102293, -0.104528463267653471399834,
         -0.5, -0.809016994374947424102293, -0.978147600733805637928567},
        {0.932472229404355804573116, 0.739008917220659115924534, 0.445738355776538267396458, 0.092268359463301995239651,
         -0.273662990072082863539078, -0.602634636379256389178588, -0.850217135729614152134144,
         -0.982973099683901778281949}};
    return t[(R - 9) / 2][m - 1];
}
template <int R>
__device__ __forceinline__ constexpr double exact_sin(int m)
{
    constexpr double t[][8] = {
        {0.642787609686539326322643, 0.984807753012208059366743, 0.866025403784438646763723, 0.342020143325668733044100},
        {0.540640817455597582107636, 0.909631995354518371411715, 0.989821441880932732376092, 0.755749574354258283774036,
         0.281732556841429697711418},
        {0.464723172043768545656015, 0.822983865893656394579617, 0.992708874098053992800752, 0.935016242685414823439785,
         0.663122658240795202376785, 0.239315664287557767148754},
        {0.406736643075800207753986, 0.743144825477394235014697, 0.951056516295153572116439, 0.994521895368273336922692,
         0.866025403784438646763723, 0.587785252292473129168706, 0.207911690817759337101742},
        {0.361241666187152948744715, 0.673695643646557211712692, 0.895163291355062322067016, 0.995734176295034521871191,
         0.961825643172819070408796, 0.798017227280239503332805, 0.526432162877355800244608,
         0.183749517816570331574409}};
    return t[(R - 9) / 2][m - 1];
}

// The index below r1 r2 with remainders k1 and k2 (r1, r2 coprime).
__device__ __forceinline__ constexpr int crt_index(int r1, int r2, int k1, int k2)
{
    int k = k1;
    while (k % r2 != k2) k += r1;
    return k;
}

// exp(-+2 pi i m / R) with m, R compile-time after unrolling (the compiler folds the trig).  EXACT: from
// the correctly rounded values above (9 <= R <= 17).  The folded trig rounds its argument, which
// leaves the root up to 9 units of 2^-53 off; the size-specialised kernels have those values in
// every result of a refined solve and keep them.  Relative error of an FP64 application at 85 x 85:
// 7.1e-16 with folded roots, 3.6e-16 with exact ones (mixed-radix passes: 4.1e-16).
template <typename T, int R, bool INV, bool EXACT = false>
__device__ __forceinline__ cpx<T> croot(int m)
{
    if constexpr (EXACT) {
        const int k = m % R;
        if (k == 0) return {T(1), T(0)};
        const bool mirror = 2 * k > R;
        const int j = mirror ? R - k : k;
        const double s = exact_sin<R>(j);
        return {T(exact_cos<R>(j)), T(INV != mirror ? s : -s)};
    }
    const double a = 6.283185307179586476925286766559 * double(m % R) / double(R);
    return {T(cos(a)), T(INV ? sin(a) : -sin(a))};
}

template <typename T, int R, bool INV, bool EXACT = false>
__device__ __forceinline__ void reg_dft(cpx<T>* v);

// DFT of an odd prime R > 7 from the sums and differences of mirrored inputs: (R - 1)^2 / 4 real
// factors on complex values for the cosine and the sine half each.
template <typename T, int R, bool INV>
__device__ __forceinline__ void dft_prime(cpx<T>* v)
{
    constexpr int H = (R - 1) / 2;
    cpx<T> a[H], b[H], y0 = v[0];
    const cpx<T> x0 = v[0];
#pragma unroll
    for (int m = 1; m <= H; m++) {
        a[m - 1] = v[m] + v[R - m];
        b[m - 1] = v[m] - v[R - m];
        y0 = y0 + a[m - 1];
    }
    v[0] = y0;
#pragma unroll
    for (int k = 1; k <= H; k++) {
        cpx<T> re = x0, im = {T(0), T(0)};
#pragma unroll
        for (int m = 1; m <= H; m++) {
            const cpx<T> w = croot<T, R, false, true>(m * k);  // (cos, -sin)
            re = re + w.x * a[m - 1];
            im = im + w.y * b[m - 1];
        }
        // X_k = re + i im and X_{R-k} = re - i im with im = -sum sin b (forward; swapped inverse)
        const cpx<T> p = {re.x - im.y, re.y + im.x}, q = {re.x + im.y, re.y - im.x};
        v[k] = INV ? q : p;
        v[R - k] = INV ? p : q;
    }
}

template <typename T, int R, bool INV, bool EXACT>
__device__ __forceinline__ void reg_dft(cpx<T>* v)
{
    if constexpr (R == 1) {
        return;
    } else if constexpr (R == 3 || R == 5 || R == 7) {
        dft_small<T, R, INV>(v);
    } else if constexpr (smallest_factor(R) == R) {
        dft_prime<T, R, INV>(v);
    } else {
        constexpr int R1 = smallest_factor(R);
        constexpr int R2 = R / R1;
        // EXACT, coprime factors (15): n = R2 n1 + R1 n2 and k by its remainders need no twiddles.  FP64
        // application at 225 x 225: error 4.5e-16 -> 4.3e-16 (mixed-radix passes: 4.3e-16), 25.0 -> 24.2 us.
        constexpr bool pfa = EXACT && R2 % R1 != 0;
        cpx<T> y[R];
#pragma unroll
        for (int n1 = 0; n1 < R1; n1++) {
            cpx<T> s[R2];
#pragma unroll
            for (int n2 = 0; n2 < R2; n2++) s[n2] = v[pfa ? (R2 * n1 + R1 * n2) % R : n1 + R1 * n2];
            reg_dft<T, R2, INV, EXACT>(s);
#pragma unroll
            for (int k2 = 0; k2 < R2; k2++)
                y[n1 * R2 + k2] = (pfa || n1 * k2 == 0) ? s[k2] : cmul(s[k2], croot<T, R, INV, EXACT>(n1 * k2));
        }
#pragma unroll
        for (int k2 = 0; k2 < R2; k2++) {
            cpx<T> s[R1];
#pragma unroll
            for (int n1 = 0; n1 < R1; n1++) s[n1] = y[n1 * R2 + k2];
            reg_dft<T, R1, INV, EXACT>(s);
#pragma unroll
            for (int k1 = 0; k1 < R1; k1++) v[pfa ? crt_index(R1, R2, k1, k2) : k2 + R2 * k1] = s[k1];
        }
    }
}

// ------------------------------------------------------------------------------------------
// Runtime-kind coefficient helpers (the kind is uniform across the launch).
// ------------------------------------------------------------------------------------------
template <typename T, int D>
__device__ __forceinline__ void coef_mul_rt(const CoefArgs& A, const T* tab, long long pt, long long npts,
                                            const T* u, T* z)
{
    if (A.kind == AK_ISO) {
        const T a = static_cast<const T*>(A.coef)[pt];
#pragma unroll
        for (int c = 0; c < D; c++) z[c] = a * u[c];
    } else if (A.kind == AK_PHASE) {
        sym_mul<T, D>(tab + 6 * A.phase[pt], u, z);
    } else {
        T co[6];
        const T* cc = static_cast<const T*>(A.coef);
#pragma unroll
        for (int q = 0; q < ncoef_of<D>(); q++) co[q] = cc[q * npts + pt];
        sym_mul<T, D>(co, u, z);
    }
}

// (A + w I)^{-1} v at one point.
template <typename T, int D>
__device__ __forceinline__ void coef_shift_solve_rt(const CoefArgs& A, const T* tabinv, T w, long long pt,
                                                    long long npts, const T* v, T* xn)
{
    if (A.kind == AK_ISO) {
        const T av = static_cast<const T*>(A.coef)[pt];
#pragma unroll
        for (int c = 0; c < D; c++) xn[c] = v[c] / (av + w);
    } else if (A.kind == AK_PHASE) {
        sym_mul<T, D>(tabinv + 6 * A.phase[pt], v, xn);
    } else {
        T co[6];
        const T* cc = static_cast<const T*>(A.coef);
#pragma unroll
        for (int q = 0; q < ncoef_of<D>(); q++) co[q] = cc[q * npts + pt];
        sym_shift_solve<T, D>(co, w, v, xn);
    }
}

// Component c of a [d][n] vector: a uniform base address, so that a point's access is that base
// plus a 32-bit per-lane offset (no 64-bit address arithmetic per access).
template <typename P>
__device__ __forceinline__ P* comp(P* base, int c, unsigned n)
{
    return base + (size_t)c * n;
}

// Batched point processing: the loads of kU points per thread are all issued before any of them
// is used, so one memory latency covers kU points (a loop with a runtime trip count would wait
// once per point).  The operation and coefficient kind are uniform across the launch, so their
// branches sit outside the unrolled point loops; out-of-range points load from point 0 and are
// discarded.
constexpr int kU = 4;

// Points per thread and chunk for a row length L: one chunk covers a tile of up to 8 rows.
constexpr int ku_for(int L)
{
    const int k = (8 * L + kThreads - 1) / kThreads;
    return k < 2 ? 2 : (k > 8 ? 8 : k);
}

// A row length: compile-time (LT > 0, the size-specialised kernels) or run-time (LT = 0), and the
// row of a tile's point index.  The run-time form divides by multiplying with the reciprocal: the
// error of (i + 0.5) / L stays below half of 1 / L for indices below 2^21, so the floor is exact.
template <int LT>
struct RowLen {
    int l;
    float inv;
    __device__ __forceinline__ int len() const { return LT ? LT : l; }
    __device__ __forceinline__ int row(int i) const
    {
        return LT ? i / (LT ? LT : 1) : (int)(((float)i + 0.5f) * inv);
    }
};

// Stage 0 of the first pass for KU points starting at this thread's index base + threadIdx.x:
// z = A(pt) u with u per FirstOp.  Real rows 2m and 2m + 1 of the tile (row r, component c:
// r D + c) are written as the real and imaginary parts of complex row m (RS slots apart).
// For CG's operand in double precision this thread's part of (A p, p) is added to acc (point by point,
// so that it does not depend on KU).
template <typename T, int D, int LT, int KU, bool XD = false>
__device__ __forceinline__ void first_stage0_chunk(const FirstArgs<T>& a, int op, const T* tab, T beta, int base,
                                                   int total, int lim, long long pt0, T* Zr, RowLen<LT> rl, int RS,
                                                   double& acc)
{
    const unsigned npts = (unsigned)a.g.npts;  // 32-bit offsets: d |grid| < 2^31 here
    unsigned pt[KU];
    bool ok[KU];
#pragma unroll
    for (int u = 0; u < KU; u++) {
        const int idx = base + u * (int)blockDim.x + (int)threadIdx.x;
        ok[u] = idx < lim;
        pt[u] = ok[u] ? (unsigned)(pt0 + idx) : 0u;
    }
    T uu[KU][D];
    if (op == OP_E) {
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) uu[u][c] = T(a.E[c]);
    } else if (op == OP_AP_CG) {
        T rr[KU][D], pp[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                rr[u][c] = comp(a.r, c, npts)[pt[u]];
                pp[u][c] = comp(a.p, c, npts)[pt[u]];
            }
        if (XD) {  // the previous body's x += alpha p, with p as it was on entry
            const T al = T(a.sc->alpha);
            T xx[KU][D];
#pragma unroll
            for (int u = 0; u < KU; u++)
#pragma unroll
                for (int c = 0; c < D; c++) xx[u][c] = comp(a.xd, c, npts)[pt[u]];
#pragma unroll
            for (int u = 0; u < KU; u++)
#pragma unroll
                for (int c = 0; c < D; c++)
                    if (ok[u]) comp(a.xd, c, npts)[pt[u]] = fma(al, pp[u][c], xx[u][c]);
        }
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                uu[u][c] = rr[u][c] + beta * pp[u][c];
                if (ok[u]) comp(a.p, c, npts)[pt[u]] = uu[u][c];
            }
    } else {
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) uu[u][c] = comp(a.x, c, npts)[pt[u]];
        if (op == OP_AX) {
#pragma unroll
            for (int u = 0; u < KU; u++)
#pragma unroll
                for (int c = 0; c < D; c++) uu[u][c] += T(a.E[c]);
        }
    }
    T z[KU][D];
    if (op == OP_ID) {
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) z[u][c] = uu[u][c];
    } else if (a.A.kind == AK_PHASE) {
        int ph[KU];
#pragma unroll
        for (int u = 0; u < KU; u++) ph[u] = a.A.phase[pt[u]];
#pragma unroll
        for (int u = 0; u < KU; u++) sym_mul<T, D>(tab + 6 * ph[u], uu[u], z[u]);
    } else if (a.A.kind == AK_ISO) {
        const T* cc = static_cast<const T*>(a.A.coef);
        T co[KU];
#pragma unroll
        for (int u = 0; u < KU; u++) co[u] = cc[pt[u]];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) z[u][c] = co[u] * uu[u][c];
    } else {
        const T* cc = static_cast<const T*>(a.A.coef);
        T co[KU][6];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int q = 0; q < ncoef_of<D>(); q++) co[u][q] = comp(cc, q, npts)[pt[u]];
#pragma unroll
        for (int u = 0; u < KU; u++) sym_mul<T, D>(co[u], uu[u], z[u]);
    }
    if (op == OP_EM) {
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) z[u][c] -= T(a.omega) * uu[u][c];
    }
    if (sizeof(T) == 8 && op == OP_AP_CG) {
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++)
                if (ok[u]) acc += double(z[u][c]) * double(uu[u][c]);
    }
#pragma unroll
    for (int u = 0; u < KU; u++) {
        const int idx = base + u * (int)blockDim.x + (int)threadIdx.x;
        if (idx < total) {
            const int r = rl.row(idx);
            const int i = idx - r * rl.len();
#pragma unroll
            for (int c = 0; c < D; c++) {
                const int q = r * D + c;
                Zr[((q >> 1) * RS + i) * 2 + (q & 1)] = ok[u] ? z[u][c] : T(0);
            }
        }
    }
}

// The twiddle table of a length on its way to LDS: load() early, store() once other loads are under
// way, so that the two share one memory latency.  (kThreads threads.)
template <typename T, int L>
struct TwiddleCopy {
    static constexpr int N = (L + kThreads - 1) / kThreads;
    cpx<T> v[N];
    __device__ __forceinline__ void load(const cpx<T>* g)
    {
#pragma unroll
        for (int u = 0; u < N; u++) {
            const int m = (int)threadIdx.x + u * kThreads;
            v[u] = g[m < L ? m : 0];
        }
    }
    __device__ __forceinline__ void store(cpx<T>* tw) const
    {
#pragma unroll
        for (int u = 0; u < N; u++) {
            const int m = (int)threadIdx.x + u * kThreads;
            if (m < L) tw[m] = v[u];
        }
    }
};

// Epilogue of the last pass for kU points: y from the real rows Zr, the solver update per Epi.
template <typename T, int D, int LT, int epi, int KU>
__device__ __forceinline__ double last_epilogue_chunk(const LastArgs<T>& a, const T* tabinv, int base, int total,
                                                      int lim, long long pt0, const T* Zr, RowLen<LT> rl, int RS,
                                                      double acc = 0.0)
{
    const unsigned npts = (unsigned)a.g.npts;  // 32-bit offsets: d |grid| < 2^31 here
    unsigned pt[KU];
    bool ok[KU];
    T y[KU][D];
#pragma unroll
    for (int u = 0; u < KU; u++) {
        const int idx = base + u * (int)blockDim.x + (int)threadIdx.x;
        ok[u] = idx < lim;
        pt[u] = ok[u] ? (unsigned)(pt0 + idx) : 0u;
        const int ii = ok[u] ? idx : 0;
        const int r = rl.row(ii);
        const int i = ii - r * rl.len();
#pragma unroll
        for (int c = 0; c < D; c++) {
            // real rows 2m, 2m+1 are the real and imaginary parts of packed row m (RS slots apart)
            const int q = r * D + c;
            y[u][c] = Zr[((q >> 1) * RS + i) * 2 + (q & 1)];
        }
    }
    if constexpr (epi == EPI_STORE) {
        const T sg = T(a.sgn);
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const T v = sg * y[u][c];
                if (ok[u]) {
                    comp(a.y, c, npts)[pt[u]] = v;
                    acc += double(v) * double(v);
                }
            }
    } else if constexpr (epi == EPI_RICH) {
        T xv[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) xv[u][c] = comp(a.x, c, npts)[pt[u]];
        const T w = T(-a.omega);
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const T st = w * y[u][c];
                if (ok[u]) {
                    comp(a.x, c, npts)[pt[u]] = xv[u][c] + st;
                    acc += double(st) * double(st);
                }
            }
    } else if constexpr (epi == EPI_CG) {
        T pv[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) pv[u][c] = comp(a.p, c, npts)[pt[u]];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++)
                if (ok[u]) {
                    comp(a.q, c, npts)[pt[u]] = y[u][c];
                    acc += double(y[u][c]) * double(pv[u][c]);
                }
    } else if constexpr (epi == EPI_CGR || epi == EPI_CGRX) {
        T rv[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) rv[u][c] = comp(a.r, c, npts)[pt[u]];
        const T al = T(a.sc->alpha);
        if constexpr (epi == EPI_CGRX) {
            T xv[KU][D], pv[KU][D];
#pragma unroll
            for (int u = 0; u < KU; u++)
#pragma unroll
                for (int c = 0; c < D; c++) {
                    xv[u][c] = comp(a.x, c, npts)[pt[u]];
                    pv[u][c] = comp(a.p, c, npts)[pt[u]];
                }
#pragma unroll
            for (int u = 0; u < KU; u++)
#pragma unroll
                for (int c = 0; c < D; c++)
                    if (ok[u]) comp(a.x, c, npts)[pt[u]] = fma(al, pv[u][c], xv[u][c]);
        }
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const T rn = rv[u][c] - al * y[u][c];
                if (ok[u]) {
                    comp(a.r, c, npts)[pt[u]] = rn;
                    acc += double(rn) * double(rn);
                }
            }
    } else if constexpr (epi == EPI_CHEB) {
        T xv[KU][D], rv[KU][D], pv[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const unsigned o = pt[u];
                xv[u][c] = comp(a.x, c, npts)[o];
                rv[u][c] = comp(a.r, c, npts)[o];
                pv[u][c] = comp(a.p, c, npts)[o];
            }
        const T al = T(a.sc ? a.sc->alpha : a.alpha), be = T(a.sc ? a.sc->beta : a.beta);
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const T rn = rv[u][c] - al * y[u][c];
                if (ok[u]) {
                    const unsigned o = pt[u];
                    comp(a.r, c, npts)[o] = rn;
                    comp(a.x, c, npts)[o] = xv[u][c] + al * pv[u][c];
                    comp(a.p, c, npts)[o] = rn - be * pv[u][c];
                    acc += double(rn) * double(rn);
                }
            }
    } else {  // EPI_EM
        T xv[KU][D], sv[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const unsigned o = pt[u];
                xv[u][c] = comp(a.x, c, npts)[o];
                sv[u][c] = a.src ? comp(a.src, c, npts)[o] : T(2.0 * a.omega * a.E[c]);
            }
        const T w = T(a.omega);
        T xn[KU][D];
        if (a.A.kind == AK_PHASE) {
            int ph[KU];
#pragma unroll
            for (int u = 0; u < KU; u++) ph[u] = a.A.phase[pt[u]];
#pragma unroll
            for (int u = 0; u < KU; u++) {
                T v[D];
#pragma unroll
                for (int c = 0; c < D; c++) v[c] = a.src ? y[u][c] : y[u][c] + sv[u][c];
                sym_mul<T, D>(tabinv + 6 * ph[u], v, xn[u]);
            }
        } else if (a.A.kind == AK_ISO) {
            const T* cc = static_cast<const T*>(a.A.coef);
            T co[KU];
#pragma unroll
            for (int u = 0; u < KU; u++) co[u] = cc[pt[u]];
#pragma unroll
            for (int u = 0; u < KU; u++)
#pragma unroll
                for (int c = 0; c < D; c++) xn[u][c] = (a.src ? y[u][c] : y[u][c] + sv[u][c]) / (co[u] + w);
        } else {
            const T* cc = static_cast<const T*>(a.A.coef);
            T co[KU][6];
#pragma unroll
            for (int u = 0; u < KU; u++)
#pragma unroll
                for (int q = 0; q < ncoef_of<D>(); q++) co[u][q] = comp(cc, q, npts)[pt[u]];
#pragma unroll
            for (int u = 0; u < KU; u++) {
                T v[D];
#pragma unroll
                for (int c = 0; c < D; c++) v[c] = a.src ? y[u][c] : y[u][c] + sv[u][c];
                sym_shift_solve<T, D>(co[u], w, v, xn[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                T xnew = xn[u][c];
                if (a.src) xnew += sv[u][c];
                const T st = xnew - xv[u][c];
                if (ok[u]) {
                    comp(a.x, c, npts)[pt[u]] = xnew;
                    acc += double(st) * double(st);
                }
            }
    }
    return acc;
}

// Frequency position pos of an FFT of length L in the band of B frequencies?  Band index out.
__device__ __forceinline__ bool band_index(int pos, int L, int B, int* s)
{
    const int k = signed_index(pos, L);
    const int ak = k < 0 ? -k : k;
    if (2 * ak >= B) return false;
    *s = k < 0 ? k + B : k;
    return true;
}

// ------------------------------------------------------------------------------------------
// Workgroup -> tile mapping.  Workgroups are dispatched round-robin over the 8 XCDs (each with
// its own L2); giving every XCD a contiguous range of tiles keeps neighbouring tiles, which share
// cache lines at their edges, on the same L2.
// ------------------------------------------------------------------------------------------
__device__ __forceinline__ long long xcd_tile(long long b, long long nb)
{
    const long long q = nb >> 3, r = nb & 7;
    const long long x = b & 7, slot = b >> 3;
    return x * q + (x < r ? x : r) + slot;
}

// ------------------------------------------------------------------------------------------
// Pass 1 (rows of the last axis), all global accesses whole-row contiguous:
//   stage 0  coalesced loads, z = A(x) op x per point -> LDS (real rows)
//   stage A  two real rows (pencils 2m, 2m+1) packed as one complex row, L2-point DFTs -> Y
//   stage B  L1-point DFTs -> the full complex spectrum X of the packed row (LDS)
//   stage S  split into the two real spectra, A(k) = (X(k) + conj X(L-k)) / 2,
//            B(k) = (X(k) - conj X(L-k)) / 2i, and store k < Hb row by row.
// LDS: twiddles | Y (npairs rows) | Zr reals (2 npairs rows), reused as X (npairs rows).
// ------------------------------------------------------------------------------------------
// Points per lane and chunk of stage 0 of the first pass, per precision and length, from timings
// of the pass alone: a tile of about two whole chunks keeps the most loads in flight.  Otherwise
// FP32 chunks of at most 4 points keep four waves per SIMD at the longer rows.
// kx: the same for CG's first pass with the deferred iterate update (three vectors per point).
template <typename T, int L>
struct FirstTune {
    static constexpr int ku = (sizeof(T) == 4 && ku_for(L) > 4) ? 4 : ku_for(L);
    static constexpr int kx = ku > 2 ? ku / 2 : ku;
};
template <>
struct FirstTune<float, 243> {
    static constexpr int ku = 6, kx = 4;  // kx = 6 is as fast but costs a wave per SIMD in every op
};
template <>
struct FirstTune<double, 243> {
    static constexpr int ku = 6, kx = 6;
};

// Stages A, B and S of the first pass in place on the packed complex rows Zc (row m holds real
// rows 2m and 2m+1 as its real and imaginary parts).  Stage A maps all L1 jobs of one row to lanes
// of one wavefront: the wavefront's lanes read all their inputs before any lane writes (one
// instruction stream), so a row can be transformed in its own storage; rows of different waves
// are disjoint.  Stage B is in place per job (it reads and writes the slots k2 + L2 j).
template <typename T, int D, int L1, int L2, int RS = L1 * L2, typename Args>
__device__ __forceinline__ void first_transform_store_ip(const Args& a, long long row0, const cpx<T>* tw, cpx<T>* Zc)
{
    constexpr int L = L1 * L2;
    constexpr int PPW = 64 / L1;  // rows per wavefront in stage A
    static_assert(PPW >= 1, "a row's stage-A jobs must fit one wavefront");
    const int npairs = (a.rpb * D + 1) / 2;
    const int wid = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63;
    const int nw = (npairs + PPW - 1) / PPW;
    for (int w = wid; w < nw; w += (int)(blockDim.x >> 6)) {
        const int m = w * PPW + lane / L1;
        const int n1 = lane - (lane / L1) * L1;
        const bool act = lane < PPW * L1 && m < npairs;
        if (act) {
            // every store below depends on every load of this lane, and the lanes share one
            // instruction stream: all reads of the wavefront precede its writes
            cpx<T> sv[L2];
            const cpx<T>* z = Zc + m * RS + n1;
#pragma unroll
            for (int n2 = 0; n2 < L2; n2++) sv[n2] = z[L1 * n2];
            reg_dft<T, L2, false>(sv);
            cpx<T>* y = Zc + m * RS + n1 * L2;
            int t = 0;
#pragma unroll
            for (int k2 = 0; k2 < L2; k2++) {
                y[k2] = k2 ? cmul(sv[k2], tw[t]) : sv[k2];
                t += n1;
                if (t >= L) t -= L;
            }
        }
    }
    lds_barrier();
    for (int job = threadIdx.x; job < npairs * L2; job += blockDim.x) {
        const int m = job / L2;
        const int k2 = job - m * L2;
        cpx<T> sv[L1];
        cpx<T>* y = Zc + m * RS + k2;
#pragma unroll
        for (int n1 = 0; n1 < L1; n1++) sv[n1] = y[n1 * L2];
        reg_dft<T, L1, false>(sv);
#pragma unroll
        for (int k1 = 0; k1 < L1; k1++) y[L2 * k1] = sv[k1];
    }
    lds_barrier();
    // stage S: thread (tq, k) stores frequency k of the real rows q = tq, tq + qstep, ...
    // (32-bit element offsets: the plan keeps d |spectrum| below 2^31 for these kernels)
    const int Hb = a.g.Hb;
    const int qstep = (int)blockDim.x / Hb;
    const int tq = (int)threadIdx.x / Hb;
    const int k = (int)threadIdx.x - tq * Hb;
    const int nrows = (int)(a.g.rows - row0 < a.rpb ? a.g.rows - row0 : a.rpb);
    const int qend = nrows * D;
    const unsigned s1 = (unsigned)a.g.s1;
    cpx<T>* outb = a.out + row0 * Hb;  // uniform base, 32-bit per-lane offsets
    if (tq < qstep)
        for (int q = tq; q < qend; q += qstep) {
            const int r = q / D;
            const int c = q - r * D;
            const cpx<T>* x = Zc + (q >> 1) * RS;
            const cpx<T> Z = x[k];
            const cpx<T> Zm = x[k ? L - k : 0];
            const cpx<T> v = (q & 1) ? cpx<T>{T(0.5) * (Z.y + Zm.y), T(-0.5) * (Z.x - Zm.x)}
                                     : cpx<T>{T(0.5) * (Z.x + Zm.x), T(0.5) * (Z.y - Zm.y)};
            outb[(unsigned)c * s1 + (unsigned)(r * Hb + k)] = v;
        }
}

// First pass with one LDS buffer of npairs packed rows (the stages run in place).
// LDS: twiddles | Zc (npairs complex rows) | phase table.
// CG: op is OP_AP_CG.  A first pass of its own: the tests for beta, the pending end and the sums are
// a chain of scalar loads that a plain application's pass would wait for (FP32 applications of 63^2 and
// 45^3 points with a pass for both and one for each: 15.12 and 15.00, 25.91 and 25.72 us).
template <typename T, int D, int L1, int L2, bool CG, int KU = FirstTune<T, L1 * L2>::ku,
          int KX = FirstTune<T, L1 * L2>::kx>
__device__ __forceinline__ void first_body(const FirstArgs<T>& a, int op, int b, int nb)
{
    __builtin_assume(CG == (op == OP_AP_CG));
    if (!(CG && a.end_part) && a.done && *a.done) return;
    constexpr int L = L1 * L2;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double red[2 * kThreads / 64];
    const int npairs = (a.rpb * D + 1) / 2;
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* Zc = tw + L;
    T* tab = reinterpret_cast<T*>(Zc + npairs * L);
    // in two parts for CG (1 us of 415 at 243^3 FP64); a plain pass on a small grid waits for the loads
    // that the other lanes make there (63^2 FP32 application 14.95 -> 14.79 us with one part)
    TwiddleCopy<T, L> tc;
    if (CG)
        tc.load(a.twg);
    else
        for (int m = threadIdx.x; m < L; m += blockDim.x) tw[m] = a.twg[m];
    if (a.A.kind == AK_PHASE)
        for (int m = threadIdx.x; m < kMaxPhases * 6; m += blockDim.x) tab[m] = T(a.A.tab[m / 6][m % 6]);
    if (CG) tc.store(tw);
    if ((a.rpb * D) & 1)  // the imaginary half of the last packed row is a zero row
        for (int i = threadIdx.x; i < L; i += blockDim.x) Zc[(npairs - 1) * L + i].y = T(0);
    T beta = T(0);
    if (CG && !first_beta(a, red, &beta)) return;
    lds_barrier();
    const long long row0 = xcd_tile(b, nb) * a.rpb;
    double acc = 0.0;
    {
        const int total = a.rpb * L;
        const long long pt0 = row0 * L;
        const long long left = a.g.rows * (long long)L - pt0;
        const int lim = left < total ? (int)left : total;
        T* Zr = reinterpret_cast<T*>(Zc);
        if (CG && a.xd) {
            for (int base = 0; base < total; base += KX * blockDim.x)
                first_stage0_chunk<T, D, L, KX, true>(a, op, tab, beta, base, total, lim, pt0, Zr, RowLen<L>{}, L, acc);
        } else {
            for (int base = 0; base < total; base += KU * blockDim.x)
                first_stage0_chunk<T, D, L, KU>(a, op, tab, beta, base, total, lim, pt0, Zr, RowLen<L>{}, L, acc);
        }
    }
    if (CG && sizeof(T) == 8 && a.pq_part) {
        const double tot = block_sum(acc, red);
        if (threadIdx.x == 0) a.pq_part[b] = tot;
    }
    lds_barrier();
    first_transform_store_ip<T, D, L1, L2>(a, row0, tw, Zc);
}

template <typename T, int D, int L1, int L2, bool CG>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k2_first(FirstArgs<T> a, int op)
{
    first_body<T, D, L1, L2, CG>(a, op, blockIdx.x, gridDim.x);
}

// Several plans of one shape in one launch: member blockIdx.y with its own argument block; the
// member's workgroups see the block ids and tile mapping of the single-plan launch.
template <typename T, int D, int L1, int L2, bool CG>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2, 8))) void k2_first_b(
    const FirstArgs<T>* __restrict__ tab, int op)
{
    first_body<T, D, L1, L2, CG>(tab[blockIdx.y], op, blockIdx.x, gridDim.x);
}

// Step-A jobs of the strided pass: load a subsequence and transform it, then write it to LDS times its
// twiddles; table() puts those there.  EARLY: a thread's first job runs up to its twiddles ahead of
// the table's barrier, so that the pass starts with one memory latency instead of two.  That pays
// for the long subsequences (243^3 FP64: 173 and 157 -> 158 and 140 us, 125^3 FP32: 15.1 -> 12.4 us);
// at 135^3 FP64 the registers held across the barrier cost more (22.6 -> 23.6 us).  The loads stay
// in one block with the transform: apart from it the compiler contracts other products, and refined
// solves keep their rounding.
template <bool EARLY, typename FT, typename FL, typename FX>
__device__ __forceinline__ void run_jobs(int n, FT table, FL load_transform, FX write)
{
    int job = threadIdx.x;
    if (EARLY && job < n) load_transform(job);
    table();
    lds_barrier();
    if (EARLY) {
        while (job < n) {
            write();
            job += blockDim.x;
            if (job < n) load_transform(job);
        }
    } else {
        for (; job < n; job += blockDim.x) {
            load_transform(job);
            write();
        }
    }
}

// ------------------------------------------------------------------------------------------
// Strided axis pass (3D axis 1), one component per workgroup, tile of P columns.
// ------------------------------------------------------------------------------------------
// b: the workgroup's linear id over the (tile, outer, component) grid of one plan, after that of the
// pending loop reductions (forward passes).
template <typename T, int L1, int L2, bool INV>
__device__ __forceinline__ void axis_body(const AxisArgs<T>& a, int B, int b)
{
    if (!INV && a.pending && (b -= Pending::kBlocks) < 0) return finish_pending(a.pend, b + Pending::kBlocks);
    if (stopped(a.done)) return;
    const int gx = a.ntiles, gy = a.outer;
    constexpr int L = L1 * L2;
    extern __shared__ __align__(16) unsigned char smem[];
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* Y = tw + L;
    const int P = a.P;
    TwiddleCopy<T, L> tc;
    tc.load(a.twg);
    const unsigned lin = (unsigned)xcd_tile(b, gx * gy * a.comps);
    const int tile = (int)(lin % gx);
    const int o = (int)((lin / gx) % gy);
    const int c = (int)(lin / gx / gy);
    const cpx<T>* in = a.in + c * a.in_cs + o * a.in_os;
    cpx<T>* out = a.out + c * a.out_cs + o * a.out_os;
    // a band as long as the axis (GaNi) maps every position to itself: no band test then
    const bool banded = B != L;
    {
        // step A
        cpx<T> s[L2];
        int n1 = 0, p = 0;
        auto load = [&](int job) {
            n1 = job / P;
            p = job - n1 * P;
            const int j = tile * P + p;
#pragma unroll
            for (int n2 = 0; n2 < L2; n2++) {
                const int pos = n1 + L1 * n2;
                int si = pos;
                bool ok = j < a.inner;
                if (a.bin && banded) ok = ok && band_index(pos, L, B, &si);
                s[n2] = ok ? in[(unsigned)(si * a.inner + j)] : cpx<T>{T(0), T(0)};
            }
            reg_dft<T, L2, INV>(s);
        };
        auto write = [&]() {
            cpx<T>* y = Y + p * L + n1 * L2;
            int m = 0;
#pragma unroll
            for (int k2 = 0; k2 < L2; k2++) {
                y[k2] = k2 ? cmul(s[k2], INV ? conj(tw[m]) : tw[m]) : s[k2];
                m += n1;
                if (m >= L) m -= L;
            }
        };
        run_jobs<(L2 >= 25)>(P * L1, [&]() { tc.store(tw); }, load, write);
    }
    lds_barrier();
    for (int job = threadIdx.x; job < P * L2; job += blockDim.x) {
        const int k2 = job / P;
        const int p = job - k2 * P;
        const int j = tile * P + p;
        cpx<T> s[L1];
        const cpx<T>* y = Y + p * L + k2;
#pragma unroll
        for (int n1 = 0; n1 < L1; n1++) s[n1] = y[n1 * L2];
        reg_dft<T, L1, INV>(s);
        if (j < a.inner) {
#pragma unroll
            for (int k1 = 0; k1 < L1; k1++) {
                const int pos = k2 + L2 * k1;
                int so = pos;
                if (a.bout && banded && !band_index(pos, L, B, &so)) continue;
                out[(unsigned)(so * a.inner + j)] = s[k1];
            }
        }
    }
}

template <typename T, int L1, int L2, bool INV>
__global__ __launch_bounds__(kThreads) void k2_axis(AxisArgs<T> a, int B)
{
    axis_body<T, L1, L2, INV>(a, B, blockIdx.x);
}

// Several plans of one shape: member blockIdx.y.
template <typename T, int L1, int L2, bool INV>
__global__ __launch_bounds__(kThreads) void k2_axis_b(const AxisArgs<T>* __restrict__ tab, int B)
{
    axis_body<T, L1, L2, INV>(tab[blockIdx.y], B, blockIdx.x);
}

// ------------------------------------------------------------------------------------------
// Middle pass along axis 0 (all components, in place): forward step A -> LDS -> forward step B,
// multiplier and inverse step B in registers -> LDS -> inverse step A.
// ------------------------------------------------------------------------------------------
template <typename T, int D, int L1, int L2, int MULT, bool PEND>
__device__ __forceinline__ void middle_body(const MidArgs<T>& a, int b)
{
    if (PEND && (b -= Pending::kBlocks) < 0) return finish_pending(a.pend, b + Pending::kBlocks);
    if (stopped(a.done)) return;
    constexpr int L = L1 * L2;
    extern __shared__ __align__(16) unsigned char smem[];
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* Y = tw + L;
    const int P = a.P;
    const int YS = a.ys;      // LDS stride of a column (L, or L + 1 to spread the banks)
    const int PL = P * YS;
    const int tile = (int)xcd_tile(b, a.ntiles);
    for (int m = threadIdx.x; m < L; m += blockDim.x) tw[m] = a.twg[m];
    lds_barrier();
    // forward step A: jobs (c, n1, p), p fastest
    for (int job = threadIdx.x; job < D * P * L1; job += blockDim.x) {
        const int cn = job / P;
        const int p = job - cn * P;
        const int c = cn / L1;
        const int n1 = cn - c * L1;
        const int j = tile * P + p;
        const cpx<T>* in = a.buf + c * a.cs + j;
        cpx<T> s[L2];
#pragma unroll
        for (int n2 = 0; n2 < L2; n2++)
            s[n2] = (j < a.cols) ? in[(unsigned)((n1 + L1 * n2) * a.cols)] : cpx<T>{T(0), T(0)};
        reg_dft<T, L2, false>(s);
        cpx<T>* y = Y + c * PL + p * YS + n1 * L2;
        int m = 0;
#pragma unroll
        for (int k2 = 0; k2 < L2; k2++) {
            y[k2] = k2 ? cmul(s[k2], tw[m]) : s[k2];
            m += n1;
            if (m >= L) m -= L;
        }
    }
    lds_barrier();
    // forward step B, multiplier, inverse step B: jobs (k2, p)
    const T scale = T(a.scale);
    for (int job = threadIdx.x; job < P * L2; job += blockDim.x) {
        const int k2 = job / P;
        const int p = job - k2 * P;
        const int j = tile * P + p;
        int kv1 = 0, kv2 = 0;
        if (D == 2) {
            kv1 = j;
        } else {
            const int kb1 = j / a.Hb;
            kv1 = signed_index(kb1, a.B1);
            kv2 = j - kb1 * a.Hb;
        }
        const bool colok = j < a.cols;
        // |k|^2 is an integer below 2^24 at these lengths, exact in T
        const T kperp = T(kv1 * kv1 + kv2 * kv2);
        if constexpr (MULT == MULT_G) {
            // G^ is rank one per frequency, (G^ z)_c = k_c t with t = k.z / |k|^2, and along this
            // column only k_0 varies: the components c >= 1 enter through sum_c k_c z_c on the way
            // in and leave as k_c times one inverse transform of t.  Two forward and two inverse
            // L1-point DFTs instead of D of each.
            cpx<T> z0[L1], zp[L1];
            {
                const cpx<T>* y = Y + p * YS + k2;
#pragma unroll
                for (int n1 = 0; n1 < L1; n1++) z0[n1] = y[n1 * L2];
            }
#pragma unroll
            for (int n1 = 0; n1 < L1; n1++) zp[n1] = {T(0), T(0)};
#pragma unroll
            for (int c = 1; c < D; c++) {
                const T kc = T(c == 1 ? kv1 : kv2);
                const cpx<T>* y = Y + c * PL + p * YS + k2;
#pragma unroll
                for (int n1 = 0; n1 < L1; n1++) zp[n1] = zp[n1] + kc * y[n1 * L2];
            }
            reg_dft<T, L1, false>(z0);
            reg_dft<T, L1, false>(zp);
#pragma unroll
            for (int k1 = 0; k1 < L1; k1++) {
                const int pos = k2 + L2 * k1;
                const int k0 = signed_index(pos, L);
                const bool inband = colok && (2 * (k0 < 0 ? -k0 : k0) < a.B0);
                const T kk = T(k0 * k0) + kperp;
                // w = scale / |k|^2, and 0 at k = 0 (G^ vanishes there) and outside the band (Ga)
                const T w = (inband && kk > T(0)) ? scale * recip_int(kk) : T(0);
                const cpx<T> t = w * (T(k0) * z0[k1] + zp[k1]);
                zp[k1] = t;
                z0[k1] = T(k0) * t;
            }
            reg_dft<T, L1, true>(z0);
            reg_dft<T, L1, true>(zp);
            cpx<T>* y = Y + p * YS + k2;
            int m = 0;
#pragma unroll
            for (int n1 = 0; n1 < L1; n1++) {
                const cpx<T> tw_n = conj(tw[m]);
                const cpx<T> v0 = n1 ? cmul(z0[n1], tw_n) : z0[n1];
                const cpx<T> vt = n1 ? cmul(zp[n1], tw_n) : zp[n1];
                y[n1 * L2] = v0;
                y[PL + n1 * L2] = T(kv1) * vt;
                if (D == 3) y[2 * PL + n1 * L2] = T(kv2) * vt;
                m += k2;
                if (m >= L) m -= L;
            }
        } else {
            cpx<T> s[D][L1];
#pragma unroll
            for (int c = 0; c < D; c++) {
                const cpx<T>* y = Y + c * PL + p * YS + k2;
#pragma unroll
                for (int n1 = 0; n1 < L1; n1++) s[c][n1] = y[n1 * L2];
                reg_dft<T, L1, false>(s[c]);
            }
#pragma unroll
            for (int k1 = 0; k1 < L1; k1++) {
                const int pos = k2 + L2 * k1;
                const int k0 = signed_index(pos, L);
                const bool inband = colok && (2 * (k0 < 0 ? -k0 : k0) < a.B0);
                const T kk = T(k0 * k0) + kperp;
                // w = scale / |k|^2, and 0 at k = 0 (I - 2G^ is the identity there); Eyre-Milton
                // runs on the GaNi grid only, where every k is in the band
                const T w = (inband && kk > T(0)) ? scale * recip_int(kk) : T(0);
                const T kvec[3] = {T(k0), T(kv1), T(kv2)};
                cpx<T> kz = {T(0), T(0)};
#pragma unroll
                for (int c = 0; c < D; c++) kz = kz + kvec[c] * s[c][k1];
                const cpx<T> wkz = w * kz;
#pragma unroll
                for (int c = 0; c < D; c++) s[c][k1] = scale * s[c][k1] - T(2) * (kvec[c] * wkz);
            }
#pragma unroll
            for (int c = 0; c < D; c++) {
                reg_dft<T, L1, true>(s[c]);
                cpx<T>* y = Y + c * PL + p * YS + k2;
                int m = 0;
#pragma unroll
                for (int n1 = 0; n1 < L1; n1++) {
                    y[n1 * L2] = n1 ? cmul(s[c][n1], conj(tw[m])) : s[c][n1];
                    m += k2;
                    if (m >= L) m -= L;
                }
            }
        }
    }
    lds_barrier();
    // inverse step A: jobs (c, n1, p)
    for (int job = threadIdx.x; job < D * P * L1; job += blockDim.x) {
        const int cn = job / P;
        const int p = job - cn * P;
        const int c = cn / L1;
        const int n1 = cn - c * L1;
        const int j = tile * P + p;
        cpx<T> s[L2];
        const cpx<T>* y = Y + c * PL + p * YS + n1 * L2;
#pragma unroll
        for (int k2 = 0; k2 < L2; k2++) s[k2] = y[k2];
        reg_dft<T, L2, true>(s);
        if (j < a.cols) {
            cpx<T>* outp = a.buf + c * a.cs + j;
#pragma unroll
            for (int n2 = 0; n2 < L2; n2++) outp[(unsigned)((n1 + L1 * n2) * a.cols)] = s[n2];
        }
    }
}

template <typename T, int D, int L1, int L2, int MULT, bool PEND>
__global__ __launch_bounds__(kThreads) void k2_middle(MidArgs<T> a)
{
    middle_body<T, D, L1, L2, MULT, PEND>(a, blockIdx.x);
}

template <typename T, int D, int L1, int L2, int MULT, bool PEND>
__global__ __launch_bounds__(kThreads) void k2_middle_b(const MidArgs<T>* __restrict__ tab)
{
    middle_body<T, D, L1, L2, MULT, PEND>(tab[blockIdx.y], blockIdx.x);
}

// ------------------------------------------------------------------------------------------
// Last pass, all global accesses whole-row contiguous:
//   stage L   coalesced loads of the half spectra of the rows -> LDS (Sx)
//   stage B'  packed row Z = A + iB of pencils 2m, 2m+1 with Hermitian completion
//             (A(L-k) = conj A(k)), inverse L1-point DFTs -> Y
//   stage A'  inverse L2-point DFTs; real and imaginary parts are the two real rows (Zr)
//   stage E   solver epilogue per point, the d components together.
// LDS: twiddles | npairs packed rows of L + 1 slots (half spectra in, real rows out) | table.
// ------------------------------------------------------------------------------------------
// Stages B' and A' of the last pass in place.  Packed row m has its own region of L + 1 complex
// slots: it enters holding the half spectra of real rows 2m and 2m+1 (slots [0, Hb) and
// [Hb, 2Hb)) and leaves holding the two real rows interleaved as one complex row.  Both stages
// map the jobs of one row to lanes of one wavefront, whose lanes read all their inputs before any
// lane writes (one instruction stream); rows of different waves are disjoint.  The caller has
// synchronised after filling S; returns synchronised.
template <typename T, int D, int L1, int L2>
__device__ __forceinline__ void last_transform(const LastArgs<T>& a, const cpx<T>* tw, cpx<T>* S)
{
    constexpr int L = L1 * L2;
    constexpr int LP = L + 1;
    constexpr int PB = 64 / L2, PA = 64 / L1;  // rows per wavefront in stages B' and A'
    static_assert(PB >= 1 && PA >= 1, "a row's jobs must fit one wavefront");
    const int npairs = (a.rpb * D + 1) / 2;
    const int Hb = a.g.Hb;
    const int wid = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, nwaves = (int)(blockDim.x >> 6);
    for (int w = wid; w < (npairs + PB - 1) / PB; w += nwaves) {
        const int m = w * PB + lane / L2;
        const int k2 = lane - (lane / L2) * L2;
        if (lane < PB * L2 && m < npairs) {
            const cpx<T>* s0 = S + m * LP;
            const cpx<T>* s1 = s0 + Hb;
            cpx<T> sv[L1];
#pragma unroll
            for (int k1 = 0; k1 < L1; k1++) {
                const int k = k2 + L2 * k1;
                cpx<T> A = {T(0), T(0)}, B = {T(0), T(0)};
                if (k < Hb) {
                    A = s0[k];
                    B = s1[k];
                } else if (L - k < Hb) {
                    A = conj(s0[L - k]);
                    B = conj(s1[L - k]);
                }
                sv[k1] = {A.x - B.y, A.y + B.x};
            }
            reg_dft<T, L1, true>(sv);
            cpx<T>* y = S + m * LP + k2;
            int t = 0;
#pragma unroll
            for (int n1 = 0; n1 < L1; n1++) {
                y[n1 * L2] = n1 ? cmul(sv[n1], conj(tw[t])) : sv[n1];
                t += k2;
                if (t >= L) t -= L;
            }
        }
    }
    lds_barrier();
    for (int w = wid; w < (npairs + PA - 1) / PA; w += nwaves) {
        const int m = w * PA + lane / L1;
        const int n1 = lane - (lane / L1) * L1;
        if (lane < PA * L1 && m < npairs) {
            cpx<T> sv[L2];
            cpx<T>* y = S + m * LP;
#pragma unroll
            for (int k2 = 0; k2 < L2; k2++) sv[k2] = y[n1 * L2 + k2];
            reg_dft<T, L2, true>(sv);
#pragma unroll
            for (int n2 = 0; n2 < L2; n2++) y[n1 + L1 * n2] = sv[n2];
        }
    }
    lds_barrier();
}

// Epilogue of the last pass over the tile of rows starting at row0; returns this thread's sum.
template <typename T, int D, int L, int epi, int KUH = 2>  // KUH: points per chunk of the heavy epilogues
__device__ __forceinline__ double last_epilogue_tile(const LastArgs<T>& a, const T* tab, long long row0, const T* Zr)
{
    double acc = 0.0;
    const int total = a.rpb * L;
    const long long pt0 = row0 * L;
    const long long left = a.g.rows * (long long)L - pt0;
    const int lim = left < total ? (int)left : total;
    // the Chebyshev, Eyre-Milton and CGRX epilogues hold two or three more vectors per point: smaller chunks
    constexpr int KU = (epi == EPI_CHEB || epi == EPI_EM || epi == EPI_CGRX) && ku_for(L) > KUH ? KUH : ku_for(L);
    for (int base = 0; base < total; base += KU * blockDim.x) {
        if (epi == EPI_CGR || epi == EPI_CGRX)  // point by point: the two have different chunks
            acc = last_epilogue_chunk<T, D, L, epi, KU>(a, tab, base, total, lim, pt0, Zr, RowLen<L>{}, L + 1, acc);
        else
            acc += last_epilogue_chunk<T, D, L, epi, KU>(a, tab, base, total, lim, pt0, Zr, RowLen<L>{}, L + 1);
    }
    return acc;
}

template <typename T, int D, int L1, int L2, int epi>
__device__ __forceinline__ void last_body(const LastArgs<T>& a, int b, int nb)
{
    if (a.done && *a.done) return;
    constexpr int L = L1 * L2;
    extern __shared__ __align__(16) unsigned char smem[];
    const int npairs = (a.rpb * D + 1) / 2;
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* Sx = tw + L;  // npairs packed rows of L + 1 slots
    const T* Zr = reinterpret_cast<const T*>(Sx);
    T* tab = reinterpret_cast<T*>(Sx + npairs * (L + 1));
    __shared__ double red[kThreads / 64];
    // the twiddles share the spectra's memory latency in single precision (243^3: 81 -> 77 us); in
    // double the registers they wait in cost more (125^3: 26.4 -> 27.8 us), and on the few rows of a 2D
    // grid there is nothing to gain (63^2 FP32 application 15.06 -> 14.95 us without)
    constexpr bool late = sizeof(T) == 4 && D == 3;
    TwiddleCopy<T, L> tc;
    tc.load(a.twg);
    if (!late) tc.store(tw);
    if (epi == EPI_EM && a.A.kind == AK_PHASE)
        for (int m = threadIdx.x; m < kMaxPhases * 6; m += blockDim.x) tab[m] = T(a.A.tab_inv[m / 6][m % 6]);
    const long long row0 = xcd_tile(b, nb) * a.rpb;
    const int Hb = a.g.Hb;
    {
        // stage L: thread (tq, k) loads frequency k of the real rows q = tq, tq + qstep, ...,
        // kQ rows per batch with all loads issued before the LDS stores (32-bit offsets)
        constexpr int kQ = 6;
        const int qstep = (int)blockDim.x / Hb;
        const int tq = (int)threadIdx.x / Hb;
        const int k = (int)threadIdx.x - tq * Hb;
        const int nrows = (int)(a.g.rows - row0 < a.rpb ? a.g.rows - row0 : a.rpb);
        const int qend = nrows * D;
        const unsigned s1 = (unsigned)a.g.s1;
        const cpx<T>* inb = a.in + row0 * Hb;  // uniform base, 32-bit per-lane offsets
        if (tq < qstep)
            for (int q0 = tq; q0 < 2 * npairs; q0 += kQ * qstep) {
                cpx<T> v[kQ];
#pragma unroll
                for (int u = 0; u < kQ; u++) {
                    const int q = q0 + u * qstep;
                    const int r = q / D;
                    const int c = q - r * D;
                    const bool ok = q < qend;
                    const unsigned off = ok ? (unsigned)c * s1 + (unsigned)(r * Hb + k) : (unsigned)k;
                    v[u] = inb[off];
                    if (!ok) v[u] = {T(0), T(0)};
                }
#pragma unroll
                for (int u = 0; u < kQ; u++) {
                    const int q = q0 + u * qstep;
                    if (q < 2 * npairs) Sx[(q >> 1) * (L + 1) + (q & 1) * Hb + k] = v[u];
                }
            }
    }
    if (late) tc.store(tw);
    lds_barrier();
    last_transform<T, D, L1, L2>(a, tw, Sx);
    const double acc = last_epilogue_tile<T, D, L, epi>(a, tab, row0, Zr);
    const double tot = block_sum(acc, red);
    if (threadIdx.x == 0) a.partials[b] = tot;
    if (a.defer_sc && b == 0 && threadIdx.x == 0) {
        a.defer_sc->pend = 1;
        a.defer_sc->pend_op = a.redop;
    }
}

template <typename T, int D, int L1, int L2, int epi>
__global__ __launch_bounds__(kThreads) void k2_last(LastArgs<T> a)
{
    last_body<T, D, L1, L2, epi>(a, blockIdx.x, gridDim.x);
}

template <typename T, int D, int L1, int L2, int epi>
__global__ __launch_bounds__(kThreads) void k2_last_b(const LastArgs<T>* __restrict__ tab)
{
    last_body<T, D, L1, L2, epi>(tab[blockIdx.y], blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------------------------------
// Last pass of one loop body fused with the first pass of the next (Richardson, Chebyshev,
// Eyre-Milton).  Their updates are pointwise with scalars known before the pass, so once a
// point's iterate is updated the next operator application's operand is known there too:
//   Richardson   x' = x - w y,                   next z = A (x' + E)
//   Chebyshev    r' = r - a y, x' = x + a p,      next z = A p',  p' = r' - b p
//   Eyre-Milton  x' = (A + wI)^{-1} (y + src),    next z = (A - wI) x'
// The tile of rows is inverse-transformed as in the last pass; each point's update and its next
// z are computed by one thread, which writes z into the very LDS slot its y came from; the rows
// are then forward-transformed in place (row stride L + 1) and stored as the next body's first
// spectrum.  This saves the next first pass's read of the iterate and one launch per body.
// ------------------------------------------------------------------------------------------
template <typename T, int D, int LT, int epi, int KU>
__device__ __forceinline__ double lastfirst_chunk(const LastArgs<T>& a, const T* tab, const T* tabinv, int base,
                                                  int total, int lim, long long pt0, T* Zr, RowLen<LT> rl, int RS)
{
    const unsigned npts = (unsigned)a.g.npts;  // 32-bit offsets: d |grid| < 2^31 here
    unsigned pt[KU];
    bool ok[KU];
    int at[KU];  // the point's position within its row
    T y[KU][D];
#pragma unroll
    for (int u = 0; u < KU; u++) {
        const int idx = base + u * (int)blockDim.x + (int)threadIdx.x;
        ok[u] = idx < lim;
        pt[u] = ok[u] ? (unsigned)(pt0 + idx) : 0u;
        const int r = rl.row(idx);
        const int i = idx - r * rl.len();
        at[u] = i;
#pragma unroll
        for (int c = 0; c < D; c++) {
            const int q = r * D + c;
            y[u][c] = ok[u] ? Zr[((q >> 1) * RS + i) * 2 + (q & 1)] : T(0);
        }
    }
    T un[KU][D];
    double acc = 0.0;
    if constexpr (epi == EPI_RICH) {
        T xv[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) xv[u][c] = comp(a.x, c, npts)[pt[u]];
        const T w = T(-a.omega);
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const T st = w * y[u][c];
                const T xn = xv[u][c] + st;
                un[u][c] = xn + T(a.E[c]);
                if (ok[u]) {
                    comp(a.x, c, npts)[pt[u]] = xn;
                    acc += double(st) * double(st);
                }
            }
    } else if constexpr (epi == EPI_CHEB) {
        T xv[KU][D], rv[KU][D], pv[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const unsigned o = pt[u];
                xv[u][c] = comp(a.x, c, npts)[o];
                rv[u][c] = comp(a.r, c, npts)[o];
                pv[u][c] = comp(a.p, c, npts)[o];
            }
        const T al = T(a.sc ? a.sc->alpha : a.alpha), be = T(a.sc ? a.sc->beta : a.beta);
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const T rn = rv[u][c] - al * y[u][c];
                const T pn = rn - be * pv[u][c];
                un[u][c] = pn + T(a.E[c]);
                if (ok[u]) {
                    const unsigned o = pt[u];
                    comp(a.r, c, npts)[o] = rn;
                    comp(a.x, c, npts)[o] = xv[u][c] + al * pv[u][c];
                    comp(a.p, c, npts)[o] = pn;
                    acc += double(rn) * double(rn);
                }
            }
    } else {  // EPI_EM
        T xv[KU][D], sv[KU][D];
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                const unsigned o = pt[u];
                xv[u][c] = comp(a.x, c, npts)[o];
                sv[u][c] = a.src ? comp(a.src, c, npts)[o] : T(2.0 * a.omega * a.E[c]);
            }
        const T w = T(a.omega);
#pragma unroll
        for (int u = 0; u < KU; u++) {
            T v[D];
#pragma unroll
            for (int c = 0; c < D; c++) v[c] = a.src ? y[u][c] : y[u][c] + sv[u][c];
            coef_shift_solve_rt<T, D>(a.A, tabinv, w, pt[u], npts, v, un[u]);
        }
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) {
                if (a.src) un[u][c] += sv[u][c];
                const T st = un[u][c] - xv[u][c];
                if (ok[u]) {
                    comp(a.x, c, npts)[pt[u]] = un[u][c];
                    acc += double(st) * double(st);
                }
            }
    }
    // the next body's first pass: z = A u (Richardson, Chebyshev) or (A - w I) u (Eyre-Milton)
    T z[KU][D];
#pragma unroll
    for (int u = 0; u < KU; u++) coef_mul_rt<T, D>(a.A, tab, pt[u], npts, un[u], z[u]);
    if constexpr (epi == EPI_EM) {
#pragma unroll
        for (int u = 0; u < KU; u++)
#pragma unroll
            for (int c = 0; c < D; c++) z[u][c] -= T(a.omega) * un[u][c];
    }
#pragma unroll
    for (int u = 0; u < KU; u++) {
        const int idx = base + u * (int)blockDim.x + (int)threadIdx.x;
        if (idx < total) {
            const int r = rl.row(idx);
#pragma unroll
            for (int c = 0; c < D; c++) {
                const int q = r * D + c;
                Zr[((q >> 1) * RS + at[u]) * 2 + (q & 1)] = ok[u] ? z[u][c] : T(0);
            }
        }
    }
    return acc;
}

template <typename T, int D, int L1, int L2, int epi>
__device__ __forceinline__ void lastfirst_body(const LastArgs<T>& a, int b, int nb)
{
    static_assert(epi == EPI_RICH || epi == EPI_CHEB || epi == EPI_EM, "pointwise updates only");
    if (a.done && *a.done) return;
    constexpr int L = L1 * L2;
    extern __shared__ __align__(16) unsigned char smem[];
    const int npairs = (a.rpb * D + 1) / 2;
    cpx<T>* tw = reinterpret_cast<cpx<T>*>(smem);
    cpx<T>* Sx = tw + L;  // npairs packed rows of L + 1 slots
    T* Zr = reinterpret_cast<T*>(Sx);
    T* tab = reinterpret_cast<T*>(Sx + npairs * (L + 1));
    T* tabinv = tab + kMaxPhases * 6;
    __shared__ double red[kThreads / 64];
    for (int m = threadIdx.x; m < L; m += blockDim.x) tw[m] = a.twg[m];
    if (a.A.kind == AK_PHASE)
        for (int m = threadIdx.x; m < kMaxPhases * 6; m += blockDim.x) {
            tab[m] = T(a.A.tab[m / 6][m % 6]);
            tabinv[m] = T(a.A.tab_inv[m / 6][m % 6]);
        }
    const long long row0 = xcd_tile(b, nb) * a.rpb;
    const int Hb = a.g.Hb;
    const int nrows = (int)(a.g.rows - row0 < a.rpb ? a.g.rows - row0 : a.rpb);
    {
        // stage L as in the last pass
        constexpr int kQ = 6;
        const int qstep = (int)blockDim.x / Hb;
        const int tq = (int)threadIdx.x / Hb;
        const int k = (int)threadIdx.x - tq * Hb;
        const int qend = nrows * D;
        const unsigned s1 = (unsigned)a.g.s1;
        const cpx<T>* inb = a.in + row0 * Hb;
        if (tq < qstep)
            for (int q0 = tq; q0 < 2 * npairs; q0 += kQ * qstep) {
                cpx<T> v[kQ];
#pragma unroll
                for (int u = 0; u < kQ; u++) {
                    const int q = q0 + u * qstep;
                    const int r = q / D;
                    const int c = q - r * D;
                    const bool ok = q < qend;
                    const unsigned off = ok ? (unsigned)c * s1 + (unsigned)(r * Hb + k) : (unsigned)k;
                    v[u] = inb[off];
                    if (!ok) v[u] = {T(0), T(0)};
                }
#pragma unroll
                for (int u = 0; u < kQ; u++) {
                    const int q = q0 + u * qstep;
                    if (q < 2 * npairs) Sx[(q >> 1) * (L + 1) + (q & 1) * Hb + k] = v[u];
                }
            }
    }
    lds_barrier();
    last_transform<T, D, L1, L2>(a, tw, Sx);
    double acc = 0.0;
    {
        const int total = a.rpb * L;
        const long long pt0 = row0 * L;
        const long long left = a.g.rows * (long long)L - pt0;
        const int lim = left < total ? (int)left : total;
        constexpr int KU = epi == EPI_RICH ? (ku_for(L) > 3 ? 3 : ku_for(L)) : (ku_for(L) > 2 ? 2 : ku_for(L));
        for (int base = 0; base < total; base += KU * blockDim.x)
            acc += lastfirst_chunk<T, D, L, epi, KU>(a, tab, tabinv, base, total, lim, pt0, Zr, RowLen<L>{}, L + 1);
        if ((a.rpb * D) & 1)  // the imaginary half of the last packed row is a zero row
            for (int i = threadIdx.x; i < L; i += blockDim.x) Sx[(npairs - 1) * (L + 1) + i].y = T(0);
    }
    lds_barrier();
    first_transform_store_ip<T, D, L1, L2, L + 1>(a, row0, tw, Sx);
    const double tot = block_sum(acc, red);
    if (threadIdx.x == 0) a.partials[b] = tot;
    if (a.defer_sc && b == 0 && threadIdx.x == 0) {
        a.defer_sc->pend = 1;
        a.defer_sc->pend_op = a.redop;
    }
}

template <typename T, int D, int L1, int L2, int epi>
__global__ __launch_bounds__(kThreads) void k2_lastfirst(LastArgs<T> a)
{
    lastfirst_body<T, D, L1, L2, epi>(a, blockIdx.x, gridDim.x);
}

template <typename T, int D, int L1, int L2, int epi>
__global__ __launch_bounds__(kThreads) void k2_lastfirst_b(const LastArgs<T>* __restrict__ tab)
{
    lastfirst_body<T, D, L1, L2, epi>(tab[blockIdx.y], blockIdx.x, gridDim.x);
}

// Lengths with specialised kernels; their splits L = L1 * L2 (L1 = 5, 7 or 9: the middle pass holds
// d x L1 values per job in registers) are listed with the launches.
constexpr int kV2Lengths[] = {45, 63, 81, 125, 135, 243};

inline bool v2_supported(int L)
{
    for (int v : kV2Lengths)
        if (v == L) return true;
    return false;
}

}  // namespace fgh
