// Dark/flat normalisation with -log (section 2.3) and the ramp filter of FBP.
//
// The filter is a linear convolution with the Ram-Lak kernel on [0, L), done
// as a zero-padded FFT of length P >= 2L - 1 in LDS (the circular result then
// equals the linear one on [0, L)).  The kernel is real and even, so its
// spectrum is real and two real rows share one complex FFT (row a in the real
// part, row b in the imaginary part).  Forward: decimation in frequency,
// natural in, bit-reversed out; the spectrum is stored bit-reversed with 1/P
// folded in; inverse: decimation in time, bit-reversed in, natural out.  Two
// radix-2 stages are fused per LDS pass (radix-4 data movement).
//
// For raw input the normalisation is fused into the load: uint16 radiograph
// rows are read in acquisition order [K][R][nb] and the filtered rows are
// written in sinogram order [R][K][L], so the -log sinogram never goes to HBM.
#include "internal.hpp"

namespace pyhst {

struct FlatInfo {
    double pos[32];
    int n;
};

namespace {

__device__ inline float2 operator+(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ inline float2 operator-(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ inline float2 cmul(float2 a, float2 w) { return make_float2(a.x * w.x - a.y * w.y, a.x * w.y + a.y * w.x); }
__device__ inline float2 cmulc(float2 a, float2 w) { return make_float2(a.x * w.x + a.y * w.y, a.y * w.x - a.x * w.y); }

__device__ inline void flat_interp(const FlatInfo &fi, int k, int &i0, int &i1, float &a)
{
    i0 = i1 = 0;
    double al = 0.0;
    if (fi.n > 1) {
        if (k <= fi.pos[0]) {
            i0 = i1 = 0;
        } else if (k >= fi.pos[fi.n - 1]) {
            i0 = i1 = fi.n - 1;
        } else {
            int i = 0;
            while (i + 1 < fi.n && !(k < fi.pos[i + 1])) ++i;
            i0 = i;
            i1 = i + 1;
            al = ((double)k - fi.pos[i0]) / (fi.pos[i1] - fi.pos[i0]);
        }
    }
    a = (float)al;
}

__device__ inline float norm_value(float I, float d, float f0, float f1, float a, float eps)
{
    const float f = (1.0f - a) * f0 + a * f1;
    const float den = f - d;
    if (!(den > 0.0f)) return 0.0f;
    float ratio = (I - d) / den;
    if (!(ratio >= eps)) ratio = eps;
    return -logf(ratio);
}

__global__ __launch_bounds__(256) void normalize_kernel(const uint16_t *__restrict__ raw,
                                                        const float *__restrict__ flats, FlatInfo fi,
                                                        const float *__restrict__ dark, float eps, int K, int R,
                                                        int nb, float *__restrict__ out)
{
    const int row = blockIdx.x;          // raw row order: k * R + r
    const int k = row / R, r = row - k * R;
    int i0, i1;
    float a;
    flat_interp(fi, k, i0, i1, a);
    const uint16_t *src = raw + (int64_t)row * nb;
    const float *f0 = flats + ((int64_t)i0 * R + r) * nb;
    const float *f1 = flats + ((int64_t)i1 * R + r) * nb;
    const float *dk = dark + (int64_t)r * nb;
    float *dst = out + ((int64_t)r * K + k) * nb;
    for (int j = threadIdx.x; j < nb; j += blockDim.x)
        dst[j] = norm_value((float)src[j], dk[j], f0[j], f1[j], a, eps);
}

// Hot-spot removal on the flat-field-corrected transmission (section 2.3): a pixel whose 3x3
// neighbours' median (up to 8 neighbours of the same radiograph, mean of the middle two for an
// even count) is below it by more than thr takes that median; then -log as above.  The input
// rows are R_in = h0 + R + (halo after): output row r reads input row h0 + r, and the halo rows
// serve only as neighbours, so a volume reconstructed in chunks of rows gives the same result as
// in one piece.  A workgroup takes 256 bins of HS_ROWS rows of a radiograph and computes each transmission once, into
// LDS (with a border of one; absent pixels are +inf): a thread that made its nine itself spent its time on their
// divisions and loads (7 rows x 721 x 1003: 67 us, now 35, most of it the sorting network and the logarithm).
// Of radiographs with one or two rows a workgroup takes these, four or two times as many bins (1 row x 1973 x 1295:
// 20.6 us, with four rows and 256 bins 27, without LDS 20).
constexpr int HS_ROWS = 4;

__device__ inline float transmission(const uint16_t *raw, const float *f0, const float *f1, const float *dk, float a,
                                     int64_t o, bool &dead)
{
    const float d = dk[o];
    const float den = ((1.0f - a) * f0[o] + a * f1[o]) - d;
    dead = !(den > 0.0f);
    return dead ? 1.0f : ((float)raw[o] - d) / den;
}

__device__ inline void cswap(float &a, float &b)
{
    const float lo = fminf(a, b), hi = fmaxf(a, b);
    a = lo;
    b = hi;
}

template <int HS>
__global__ __launch_bounds__(256) void normalize_hotspot_kernel(const uint16_t *__restrict__ raw,
                                                                const float *__restrict__ flats, FlatInfo fi,
                                                                const float *__restrict__ dark, float eps, float thr,
                                                                int K, int R, int R_in, int h0, int nb, int n_rb,
                                                                float *__restrict__ out)
{
    __shared__ float t_[HS + 2][258];
    __shared__ bool dead_[HS + 2][258];
    const int k = blockIdx.x / n_rb, r0 = (blockIdx.x - k * n_rb) * HS;   // projection, first output row
    int i0, i1;
    float a;
    flat_interp(fi, k, i0, i1, a);
    const uint16_t *img = raw + (int64_t)k * R_in * nb;      // radiograph k, [R_in][nb]
    const float *f0 = flats + (int64_t)i0 * R_in * nb, *f1 = flats + (int64_t)i1 * R_in * nb;
    for (int b = 0; b < HS_ROWS / HS; ++b) {
        const int j0 = (blockIdx.y * (HS_ROWS / HS) + b) * 256;
        if (j0 >= nb) return;                            // uniform over the workgroup
        if (b > 0) __syncthreads();
        for (int i = threadIdx.x; i < (HS + 2) * 258; i += 256) {
            const int q = i / 258, c = i - q * 258;
            const int rr = r0 + h0 + q - 1, jj = j0 + c - 1;
            bool dead = false;
            const bool in = rr >= 0 && rr < R_in && jj >= 0 && jj < nb;
            t_[q][c] = in ? transmission(img, f0, f1, dark, a, (int64_t)rr * nb + jj, dead) : INFINITY;
            dead_[q][c] = dead;
        }
        __syncthreads();
        const int j = j0 + threadIdx.x, c = threadIdx.x + 1;
#pragma unroll
        for (int q = 1; q <= HS; ++q) {
            const int r = r0 + q - 1, ri = r + h0;
            if (r >= R || j >= nb) break;
            float *dst = out + ((int64_t)r * K + k) * nb;
            float t = t_[q][c];
            if (dead_[q][c]) {
                dst[j] = 0.0f;
                continue;
            }
            float v[8] = {t_[q - 1][c - 1], t_[q - 1][c], t_[q - 1][c + 1], t_[q][c - 1],
                          t_[q][c + 1], t_[q + 1][c - 1], t_[q + 1][c], t_[q + 1][c + 1]};
            const int nr = (ri > 0) + 1 + (ri + 1 < R_in), nc = (j > 0) + 1 + (j + 1 < nb);
            const int n = nr * nc - 1;   // neighbours that exist
            // sorting network for 8 values (absent neighbours are +inf and sort last)
            cswap(v[0], v[1]); cswap(v[2], v[3]); cswap(v[4], v[5]); cswap(v[6], v[7]);
            cswap(v[0], v[2]); cswap(v[1], v[3]); cswap(v[4], v[6]); cswap(v[5], v[7]);
            cswap(v[1], v[2]); cswap(v[5], v[6]); cswap(v[0], v[4]); cswap(v[3], v[7]);
            cswap(v[1], v[5]); cswap(v[2], v[6]);
            cswap(v[1], v[4]); cswap(v[3], v[6]);
            cswap(v[2], v[4]); cswap(v[3], v[5]);
            cswap(v[3], v[4]);
            float lo = v[0], hi = v[0];
#pragma unroll
            for (int i = 1; i < 8; ++i) {
                if (i == (n - 1) / 2) lo = v[i];
                if (i == n / 2) hi = v[i];
            }
            if (n > 0) {
                const float med = (n & 1) ? hi : 0.5f * (lo + hi);
                if (t - med > thr) t = med;
            }
            if (!(t >= eps)) t = eps;
            dst[j] = -logf(t);
        }
    }
}

// Ring filter (section 2.3).  m[s][j] = mean_k (p - obj)[s][k][j] (FP64).  64 bins per workgroup, the projections split
// over 16 groups of threads whose sums are added in a fixed order: one thread per bin left the chip to 28 workgroups
// (7 slices x 721 x 1003: 187 us, now 8).
__global__ __launch_bounds__(1024) void ring_mean_kernel(const float *__restrict__ p, const float *__restrict__ obj,
                                                         int K, int L, double *__restrict__ m)
{
    __shared__ double part[16][64];
    const int c = threadIdx.x & 63, q = threadIdx.x >> 6, j = blockIdx.x * 64 + c, s = blockIdx.y;
    double acc = 0.0;
    if (j < L) {
        const int64_t base = (int64_t)s * K * L + j;
#pragma unroll 8
        for (int k = q; k < K; k += 16) acc += (double)p[base + (int64_t)k * L] - (obj ? (double)obj[base + (int64_t)k * L] : 0.0);
    }
    part[q][c] = acc;
    __syncthreads();
    if (q == 0 && j < L) {
        for (int i = 1; i < 16; ++i) acc += part[i][c];
        m[(int64_t)s * L + j] = acc / K;
    }
}

// m[j] - mean of m over the bins j-w..j+w that exist
__device__ inline double ring_highpass(const double *ms, int j, int L, int w)
{
    const int lo = max(0, j - w), hi = min(L - 1, j + w);
    double acc = 0.0;
#pragma unroll 8
    for (int i = lo; i <= hi; ++i) acc += ms[i];
    return ms[j] - acc / (hi - lo + 1);
}

__global__ __launch_bounds__(256) void ring_highpass_kernel(const double *__restrict__ m, int L, int w,
                                                            double *__restrict__ hp)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x, s = blockIdx.y;
    if (j < L) hp[(int64_t)s * L + j] = ring_highpass(m + (int64_t)s * L, j, L, w);
}

// p[s][k][j] -= the high-pass value of m (HP: which m is already); a workgroup takes 256 bins of RING_ROWS rows
constexpr int RING_ROWS = 16;

template <bool HP>
__global__ __launch_bounds__(256) void ring_subtract_kernel(float *__restrict__ p, const double *__restrict__ m,
                                                            int K, int L, int w)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x, s = blockIdx.z;
    if (j >= L) return;
    const double *ms = m + (int64_t)s * L;
    const float hp = (float)(HP ? ms[j] : ring_highpass(ms, j, L, w));
    const int k1 = min(K, (int)(blockIdx.y + 1) * RING_ROWS);
    for (int k = blockIdx.y * RING_ROWS; k < k1; ++k) p[((int64_t)s * K + k) * L + j] -= hp;
}

__device__ inline float2 times_mi(float2 a) { return make_float2(a.y, -a.x); }   // a * (-i)

// One table load per radix-4 butterfly: of its three twiddles w^i, w^(i + h/2), w^(2i) (w a root of
// unity of order 2h), the second is the first times -i exactly and the third is its square.
__device__ void fft_forward(float2 *z, int P, int lg, const float2 *__restrict__ tw, int lgmax)
{
    int h = P >> 1, lh = lg - 1;
    while (h >= 2) {
        const int h2 = h >> 1;
        for (int t = threadIdx.x; t < (P >> 2); t += blockDim.x) {
            const int gq = t >> (lh - 1), i = t & (h2 - 1);
            const int b0 = (gq << (lh + 1)) + i;
            const float2 e0 = z[b0], e1 = z[b0 + h2], e2 = z[b0 + h], e3 = z[b0 + h + h2];
            const float2 w0 = tw[i << (lgmax - lh - 1)];
            const float2 w1 = times_mi(w0);
            const float2 w2 = cmul(w0, w0);
            const float2 s0 = e0 + e2, d0 = cmul(e0 - e2, w0);
            const float2 s1 = e1 + e3, d1 = cmul(e1 - e3, w1);
            z[b0] = s0 + s1;
            z[b0 + h2] = cmul(s0 - s1, w2);
            z[b0 + h] = d0 + d1;
            z[b0 + h + h2] = cmul(d0 - d1, w2);
        }
        __syncthreads();
        h >>= 2;
        lh -= 2;
    }
    if (h == 1) {
        for (int t = threadIdx.x; t < (P >> 1); t += blockDim.x) {
            const float2 a = z[2 * t], b = z[2 * t + 1];
            z[2 * t] = a + b;
            z[2 * t + 1] = a - b;
        }
        __syncthreads();
    }
}

__device__ void fft_inverse(float2 *z, int P, int lg, const float2 *__restrict__ tw, int lgmax)
{
    int h = 1, lh = 0;
    if (lg & 1) {
        for (int t = threadIdx.x; t < (P >> 1); t += blockDim.x) {
            const float2 a = z[2 * t], b = z[2 * t + 1];
            z[2 * t] = a + b;
            z[2 * t + 1] = a - b;
        }
        __syncthreads();
        h = 2;
        lh = 1;
    }
    while (h < P) {
        for (int t = threadIdx.x; t < (P >> 2); t += blockDim.x) {
            const int gq = t >> lh, i = t & (h - 1);
            const int b0 = (gq << (lh + 2)) + i;
            const float2 e0 = z[b0], e1 = z[b0 + h], e2 = z[b0 + 2 * h], e3 = z[b0 + 3 * h];
            const float2 u = tw[i << (lgmax - lh - 2)];   // u^i of order 4h: w = u^2, u^(i + h) = -i u^i
            const float2 w = cmul(u, u);
            const float2 b1 = cmulc(e1, w), b3 = cmulc(e3, w);
            const float2 s0 = e0 + b1, d0 = e0 - b1, s1 = e2 + b3, d1 = e2 - b3;
            const float2 t1 = cmulc(s1, u);
            const float2 t2 = cmulc(d1, times_mi(u));
            z[b0] = s0 + t1;
            z[b0 + 2 * h] = s0 - t1;
            z[b0 + h] = d0 + t2;
            z[b0 + 3 * h] = d0 - t2;
        }
        __syncthreads();
        h <<= 2;
        lh += 2;
    }
}

struct FilterArgs {
    Tables T;
    GeoDev g;      // uniform plans: the geometry, and the work items of a slice (the plan's tables are not read for them)
    int per;
    const float *sino;
    const uint16_t *raw;
    const float *flats;
    FlatInfo fi;
    const float *dark;
    float eps;
    int R;
    float *out;
};

// UNI: a uniform plan, whose geometry comes with the launch
template <bool RAW, bool UNI>
__global__ __launch_bounds__(256) void filter_kernel(FilterArgs A)
{
    extern __shared__ float2 z[];
    const Tables &T = A.T;
    const int2 pr = UNI ? make_int2((int)blockIdx.x / A.per, 2 * ((int)blockIdx.x % A.per)) : T.pairs[blockIdx.x];
    const SliceDev sd = UNI ? SliceDev{0, 0, (int64_t)pr.x * A.g.K * A.g.nb, (int64_t)pr.x * A.g.K * A.g.Lf, 0} : T.slc[pr.x];
    const GeoDev &g = UNI ? A.g : T.geo[sd.g];
    const int K = g.K, nb = g.nb, Lf = g.Lf, pad = g.fpad, P = g.P, lg = g.log2P;
    const int ka = pr.y, kb = pr.y + 1;
    const bool hasb = kb < K;
    const float *hw = T.haw + g.hw_off, *sino = A.sino, *flats = A.flats, *dark = A.dark;
    const uint16_t *raw = A.raw;
    const FlatInfo &fi = A.fi;
    const float eps = A.eps;
    const int R = A.R;

    int a0 = 0, a1 = 0, b0 = 0, b1 = 0;
    float aa = 0.0f, ab = 0.0f;
    if (RAW) {
        flat_interp(fi, ka, a0, a1, aa);
        flat_interp(fi, hasb ? kb : ka, b0, b1, ab);
    }
    const int r = pr.x;   // raw input: uniform plan, slice index = detector row
    const bool half = g.half != 0;
    const bool same_flats = a0 == b0 && a1 == b1;   // both rows between the same two flats (uniform)
    for (int n = threadIdx.x; n < P; n += blockDim.x) {
        float va = 0.0f, vb = 0.0f;
        const int jj = n - pad;
        if (n < Lf && jj >= 0 && jj < nb) {
            const float w = half ? hw[n] : 1.0f;
            if (RAW) {
                const float d = dark[(int64_t)r * nb + jj];
                const float Ia = (float)raw[((int64_t)ka * R + r) * nb + jj];
                const float fa0 = flats[((int64_t)a0 * R + r) * nb + jj], fa1 = flats[((int64_t)a1 * R + r) * nb + jj];
                va = norm_value(Ia, d, fa0, fa1, aa, eps);
                if (hasb) {
                    const float Ib = (float)raw[((int64_t)kb * R + r) * nb + jj];
                    const float fb0 = same_flats ? fa0 : flats[((int64_t)b0 * R + r) * nb + jj];
                    const float fb1 = same_flats ? fa1 : flats[((int64_t)b1 * R + r) * nb + jj];
                    vb = norm_value(Ib, d, fb0, fb1, ab, eps);
                }
            } else {
                va = sino[sd.sino_off + (int64_t)ka * nb + jj];
                vb = hasb ? sino[sd.sino_off + (int64_t)kb * nb + jj] : 0.0f;
            }
            va *= w;
            vb *= w;
        }
        z[n] = make_float2(va, vb);
    }
    __syncthreads();
    fft_forward(z, P, lg, T.twid, T.log2Pmax);
    const float *H = T.spec + g.spec_off;
    for (int n = threadIdx.x; n < P; n += blockDim.x) {
        const float h = H[n];
        const float2 v = z[n];
        z[n] = make_float2(v.x * h, v.y * h);
    }
    __syncthreads();
    fft_inverse(z, P, lg, T.twid, T.log2Pmax);
    const float wa = T.wang[g.ang_off + ka];
    const float wb = hasb ? T.wang[g.ang_off + kb] : 0.0f;
    float *oa = A.out + sd.filt_off + (int64_t)ka * Lf;
    for (int n = threadIdx.x; n < Lf; n += blockDim.x) {
        const float2 v = z[n];
        oa[n] = wa * v.x;
        if (hasb) oa[Lf + n] = wb * v.y;
    }
}

// The same filter with the FFT in registers, for P = 256 R (R = 1, 2, 4, 8, 16: rows of up to 2048 bins).  Each of
// the 16 R threads of a row pair holds 16 points; a pass is DFTs in registers followed by one twiddle multiply, and
// the passes exchange data through LDS twice per direction (R = 1: once) instead of log4(P) passes through LDS.  The
// twiddles are products of eight values of the plan's table (half circle) per thread, loaded once.
//   forward, thread a:        x[a + 16 R m] over m -> Y1[a][k1] = w^(a k1) DFT16_m(..)[k1]
//   forward, thread (k1, c):  Y1[c + R d][k1] over d -> Y2[k1][c][b1] = w^(16 c b1) DFT16_d(..)[b1]
//   forward, thread (k1, e):  Y2[k1][c][b1] over c -> X[k1 + 16 b1 + 256 b2] = DFT_R_c(..)[b2], for the 16 / R values
//                             of b1 whose bit reversal is 16 / R e + i: the thread's 16 values of the spectrum
//                             (bit-reversed order) lie side by side
// with w = exp(-2 pi i / P); the inverse runs the same passes backwards with conjugate twiddles.
// LDS: Y1 at k1 S1 + a, Y2 at k1 S2 + b1 T2 + c (the strides spread the reads over the banks).  Inside a 16-point
// DFT, input m sits at register m and output k at register rev4(k) = (k >> 2) | ((k & 3) << 2).
// Rows are at most P / 2 long, so half of the points are zero on the way in and not needed on the way out.
// A workgroup takes 16 / R row pairs of a slice; for R <= 4 a pair stays within one wavefront and needs no barrier.
// Bound by memory (2.6 to 3.3 TB/s of the 5.0 a copy reaches): 184320 rows of 256 bins 0.116 ms (LDS passes: 0.324),
// 46144 rows of 1003 bins 0.125 ms (0.279), 57600 rows of 2048 bins 0.33 ms (the register kernel for this length alone,
// without its loads made together: 0.42).
namespace f16 {

__device__ __forceinline__ float2 mul_mi(float2 a) { return make_float2(a.y, -a.x); }   // a * (-i)

// 4-point DFT in place, exp(-+2 pi i / 4) per step (INV: inverse, +)
template <bool INV>
__device__ __forceinline__ void dft4(float2 &x0, float2 &x1, float2 &x2, float2 &x3)
{
    const float2 s02 = x0 + x2, d02 = x0 - x2, s13 = x1 + x3, d13 = x1 - x3;
    const float2 r = mul_mi(d13);   // -i (x1 - x3)
    x0 = s02 + s13;
    x2 = s02 - s13;
    x1 = INV ? d02 - r : d02 + r;
    x3 = INV ? d02 + r : d02 - r;
}

constexpr int rev4(int k) { return (k >> 2) | ((k & 3) << 2); }

// 16-point DFT of v[0..15] (input m at register m); output k at register rev4(k)
template <bool INV>
__device__ __forceinline__ void dft16(float2 (&v)[16])
{
    // cos / sin of 2 pi e / 16, e = 0..9
    constexpr float C[10] = {1.0f, 0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f, 0.0f,
                             -0.38268343236508977f, -0.70710678118654752f, -0.92387953251128674f, -1.0f,
                             -0.92387953251128674f};
    constexpr float S[10] = {0.0f, 0.38268343236508977f, 0.70710678118654752f, 0.92387953251128674f, 1.0f,
                             0.92387953251128674f, 0.70710678118654752f, 0.38268343236508977f, 0.0f,
                             -0.38268343236508977f};
#pragma unroll
    for (int q = 0; q < 4; ++q) dft4<INV>(v[q], v[q + 4], v[q + 8], v[q + 12]);   // over p, m = q + 4 p
    // v[q + 4 r] *= exp(-+2 pi i q r / 16)
#pragma unroll
    for (int q = 1; q < 4; ++q)
#pragma unroll
        for (int r = 1; r < 4; ++r) {
            const float c = C[q * r], sn = INV ? S[q * r] : -S[q * r];
            const float2 a = v[q + 4 * r];
            v[q + 4 * r] = make_float2(a.x * c - a.y * sn, a.x * sn + a.y * c);
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) dft4<INV>(v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]);   // over q
    // now X[r + 4 s] sits at register 4 r + s = rev4(r + 4 s)
}

__device__ __forceinline__ int rev_bits4(int x) { return (int)(__brev((unsigned)x) >> 28); }

__device__ __forceinline__ float2 twiddle(float2 a, float2 w, bool conj)
{
    return conj ? cmulc(a, w) : cmul(a, w);
}

// w^k, 0 <= k < 16, from the bases w, w^2, w^4, w^8 (table values): a product of at most four of
// them, so each twiddle stays within a few FP32 roundings of the table (k is a constant once unrolled)
__device__ __forceinline__ float2 wpow(const float2 (&b)[4], int k)
{
    float2 r = make_float2(1.0f, 0.0f);
    bool first = true;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if ((k >> i) & 1) {
            r = first ? b[i] : cmul(r, b[i]);
            first = false;
        }
    return r;
}

// R-point DFT of v[0..R-1] in place, natural order in; output k at register out_at<R>(k)
template <int R>
constexpr int out_at(int k) { return R == 16 ? rev4(k) : k; }

template <int R, bool INV>
__device__ __forceinline__ void dft(float2 *v)
{
    if constexpr (R == 16) {
        dft16<INV>(*(float2(*)[16])v);
    } else if constexpr (R == 8) {
        constexpr float H = 0.70710678118654752f;
        // even and odd inputs
        dft4<INV>(v[0], v[2], v[4], v[6]);
        dft4<INV>(v[1], v[3], v[5], v[7]);
        const float2 o1 = v[3], o2 = v[5], o3 = v[7];
        const float2 t1 = INV ? make_float2(H * (o1.x - o1.y), H * (o1.x + o1.y)) : make_float2(H * (o1.x + o1.y), H * (o1.y - o1.x));
        const float2 t2 = INV ? make_float2(-o2.y, o2.x) : make_float2(o2.y, -o2.x);
        const float2 t3 = INV ? make_float2(-H * (o3.x + o3.y), H * (o3.x - o3.y)) : make_float2(H * (o3.y - o3.x), -H * (o3.x + o3.y));
        const float2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6], o0 = v[1];
        v[0] = e0 + o0; v[4] = e0 - o0;
        v[1] = e1 + t1; v[5] = e1 - t1;
        v[2] = e2 + t2; v[6] = e2 - t2;
        v[3] = e3 + t3; v[7] = e3 - t3;
    } else if constexpr (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else if constexpr (R == 2) {
        const float2 a = v[0], b = v[1];
        v[0] = a + b;
        v[1] = a - b;
    }
}

constexpr int rev_bits(int x, int n)
{
    int r = 0;
    for (int i = 0; i < n; ++i) r |= ((x >> i) & 1) << (n - 1 - i);
    return r;
}

}  // namespace f16

// strides of the exchanges, and float2 of a workgroup's 16 / R row pairs
constexpr int fft_s1(int R) { return R == 16 ? 256 : 17 * R; }
constexpr int fft_t2(int R) { return R <= 2 ? R : R + 1; }
constexpr int fft_s2(int R) { return R == 2 ? 34 : R == 4 ? 84 : R == 8 ? 152 : R == 16 ? 272 : 0; }
constexpr int fft_pair(int R) { return 16 * (fft_s1(R) > fft_s2(R) ? fft_s1(R) : fft_s2(R)); }
constexpr int fft_lds(int R) { return R ? 16 / R * fft_pair(R) : fft_lds(4); }
static_assert(fft_lds(0) >= fft_lds(1) && fft_lds(0) >= fft_lds(2) && fft_lds(0) >= fft_lds(8) && fft_lds(0) >= fft_lds(16));

template <int R, bool RAW>
__device__ __forceinline__ void filter_rows(const FilterArgs &A, float2 *zwg, const GeoDev &g, int64_t sino_off,
                                            int64_t filt_off, int slice, int k0)
{
    using namespace f16;
    constexpr int M = 16 * R, LG = R == 16 ? 4 : R == 8 ? 3 : R == 4 ? 2 : R == 2 ? 1 : 0;
    constexpr int S1 = fft_s1(R), T2 = fft_t2(R), S2 = fft_s2(R);
    const Tables &T = A.T;
    const int K = g.K, nb = g.nb, Lf = g.Lf, pad = g.fpad;
    const int f = threadIdx.x / M, u = threadIdx.x % M;          // row pair of the workgroup, thread of the pair
    const int ka = min(k0 + 2 * f, K - 1), kb = ka + 1;
    const bool live = k0 + 2 * f < K, hasb = kb < K;
    float2 *z = zwg + f * fft_pair(R);
    auto sync = [] {
        if constexpr (M <= 64) {
            asm volatile("" ::: "memory");
            __builtin_amdgcn_wave_barrier();
        } else {
            __syncthreads();
        }
    };

    float2 v[16];
    {
        int a0 = 0, a1 = 0, b0 = 0, b1 = 0;
        float aa = 0.0f, ab = 0.0f;
        if (RAW) {
            flat_interp(A.fi, ka, a0, a1, aa);
            flat_interp(A.fi, hasb ? kb : ka, b0, b1, ab);
        }
        const bool half = g.half != 0;
        const int64_t rb = (int64_t)slice * nb;   // raw input: uniform plan, slice index = detector row
        // every load is made (at a bin that exists) so that all are in flight together; bins that do not are cleared
        const float *sa = RAW ? nullptr : A.sino + sino_off + (int64_t)ka * nb;
        const float *sb = RAW ? nullptr : A.sino + sino_off + (int64_t)(hasb ? kb : ka) * nb;
        const uint16_t *ra = RAW ? A.raw + ((int64_t)ka * A.R + slice) * nb : nullptr;
        const uint16_t *rw = RAW ? A.raw + ((int64_t)(hasb ? kb : ka) * A.R + slice) * nb : nullptr;
        const float *fa0 = RAW ? A.flats + (int64_t)a0 * A.R * nb + rb : nullptr, *fa1 = RAW ? A.flats + (int64_t)a1 * A.R * nb + rb : nullptr;
        const float *fb0 = RAW ? A.flats + (int64_t)b0 * A.R * nb + rb : nullptr, *fb1 = RAW ? A.flats + (int64_t)b1 * A.R * nb + rb : nullptr;
        const bool same_flats = a0 == b0 && a1 == b1;   // both rows between the same two flats
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int n = u + M * m, jj = n - pad;
            const bool in = n < Lf && jj >= 0 && jj < nb;
            const int j = min(max(jj, 0), nb - 1);
            float va, vb;
            if (RAW) {
                const float d = A.dark[rb + j], p0 = fa0[j], p1 = fa1[j];
                va = norm_value((float)ra[j], d, p0, p1, aa, A.eps);
                const float q0 = same_flats ? p0 : fb0[j], q1 = same_flats ? p1 : fb1[j];
                vb = norm_value((float)rw[j], d, q0, q1, ab, A.eps);
            } else {
                va = sa[j];
                vb = sb[j];
            }
            if (half) {
                const float w = T.haw[g.hw_off + min(n, Lf - 1)];
                va *= w;
                vb *= w;
            }
            v[m] = make_float2(in ? va : 0.0f, in && hasb ? vb : 0.0f);
        }
#pragma unroll
        for (int m = 8; m < 16; ++m) v[m] = make_float2(0.0f, 0.0f);
    }

    // twiddle bases: w^(a k1) and w^(16 c b1) are products of these
    const int k1 = u / R, c0 = u % R;
    float2 b1w[4], b2w[4];
    {
        const float2 *tw = T.twid;
        const int sh = T.log2Pmax - 8 - LG;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            b1w[i] = tw[(u << i) << sh];
            b2w[i] = tw[((16 * c0) << i) << sh];
        }
    }
    const float4 *H = (const float4 *)(T.spec + g.spec_off + (rev_bits4(k1) << (4 + LG)) + 16 * c0);
    float h[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float4 q = H[i];
        h[4 * i] = q.x;
        h[4 * i + 1] = q.y;
        h[4 * i + 2] = q.z;
        h[4 * i + 3] = q.w;
    }
    const float wa = T.wang[g.ang_off + ka], wb = hasb ? T.wang[g.ang_off + kb] : 0.0f;
    // forward pass 1 (thread a = u)
    dft16<false>(v);
#pragma unroll
    for (int k = 0; k < 16; ++k) z[k * S1 + u] = twiddle(v[rev4(k)], wpow(b1w, k), false);
    sync();
    // forward pass 2 (thread (k1, c))
#pragma unroll
    for (int d = 0; d < 16; ++d) v[d] = z[k1 * S1 + c0 + R * d];
    dft16<false>(v);
    if constexpr (R == 1) {
        // the thread holds b1 = 0 .. 15 (at rev4(b1)): the spectrum's value of b1 is the one at its bit reversal
#pragma unroll
        for (int b = 0; b < 16; ++b) {
            const float2 x = v[rev4(b)];
            const float q = h[rev_bits(b, 4)];
            v[rev4(b)] = make_float2(x.x * q, x.y * q);
        }
        float2 w[16];
#pragma unroll
        for (int b = 0; b < 16; ++b) w[b] = v[rev4(b)];
        dft16<true>(w);
        sync();
#pragma unroll
        for (int d = 0; d < 16; ++d) z[k1 * S1 + d] = w[rev4(d)];
    } else {
        sync();   // every pass-2 read is done before the exchange is overwritten
#pragma unroll
        for (int b = 0; b < 16; ++b) z[k1 * S2 + b * T2 + c0] = twiddle(v[rev4(b)], wpow(b2w, b), false);
        sync();
        // forward pass 3 (thread (k1, e = c0)), spectrum (1/P folded), inverse pass 3
#pragma unroll
        for (int i = 0; i < 16 / R; ++i) {
            const int b = rev_bits4(16 / R * c0 + i);
#pragma unroll
            for (int c = 0; c < R; ++c) v[i * R + c] = z[k1 * S2 + b * T2 + c];
        }
#pragma unroll
        for (int i = 0; i < 16 / R; ++i) {
            dft<R, false>(v + i * R);
            float2 w[R];
#pragma unroll
            for (int b2 = 0; b2 < R; ++b2) {
                const float2 x = v[i * R + out_at<R>(b2)];
                const float q = h[i * R + rev_bits(b2, LG)];
                w[b2] = make_float2(x.x * q, x.y * q);
            }
            dft<R, true>(w);
#pragma unroll
            for (int c = 0; c < R; ++c) v[i * R + c] = w[out_at<R>(c)];
        }
        sync();   // every pass-3 read is done
#pragma unroll
        for (int i = 0; i < 16 / R; ++i) {
            const int b = rev_bits4(16 / R * c0 + i);
#pragma unroll
            for (int c = 0; c < R; ++c) z[k1 * S2 + b * T2 + c] = v[i * R + c];
        }
        sync();
        // inverse pass 2 (thread (k1, c))
#pragma unroll
        for (int b = 0; b < 16; ++b) v[b] = twiddle(z[k1 * S2 + b * T2 + c0], wpow(b2w, b), true);
        dft16<true>(v);
        sync();
#pragma unroll
        for (int d = 0; d < 16; ++d) z[k1 * S1 + c0 + R * d] = v[rev4(d)];
    }
    sync();
    // inverse pass 1 (thread a = u)
#pragma unroll
    for (int k = 0; k < 16; ++k) v[k] = twiddle(z[k * S1 + u], wpow(b1w, k), true);
    dft16<true>(v);
    if (!live) return;
    float *oa = A.out + filt_off + (int64_t)ka * Lf;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        const int n = u + M * m;
        if (n < Lf) {
            const float2 x = v[rev4(m)];
            oa[n] = wa * x.x;
            if (hasb) oa[Lf + n] = wb * x.y;
        }
    }
}

// RT: R of a uniform plan (which passes its geometry with the launch: four dependent loads before the rows' own less,
// a third of a single slice's filter), or 0: each workgroup takes its slice's
template <int RT, bool RAW>
__global__ __launch_bounds__(256, 4) void filter_reg_kernel(FilterArgs A)
{
    __shared__ float2 z[fft_lds(RT)];
    if constexpr (RT != 0) {
        const int slice = (int)blockIdx.x / A.per, k0 = ((int)blockIdx.x - slice * A.per) * (32 / RT);
        filter_rows<RT, RAW>(A, z, A.g, (int64_t)slice * A.g.K * A.g.nb, (int64_t)slice * A.g.K * A.g.Lf, slice, k0);
    } else {
        const int2 pr = A.T.pairs[blockIdx.x];
        const SliceDev sd = A.T.slc[pr.x];
        const GeoDev &g = A.T.geo[sd.g];
        switch (g.P >> 8) {
        case 1: filter_rows<1, RAW>(A, z, g, sd.sino_off, sd.filt_off, pr.x, pr.y); break;
        case 2: filter_rows<2, RAW>(A, z, g, sd.sino_off, sd.filt_off, pr.x, pr.y); break;
        case 4: filter_rows<4, RAW>(A, z, g, sd.sino_off, sd.filt_off, pr.x, pr.y); break;
        case 8: filter_rows<8, RAW>(A, z, g, sd.sino_off, sd.filt_off, pr.x, pr.y); break;
        default: filter_rows<16, RAW>(A, z, g, sd.sino_off, sd.filt_off, pr.x, pr.y); break;
        }
    }
}

template <bool RAW>
hipError_t launch_reg(const FilterArgs &A, int R, int n, hipStream_t st)
{
    switch (R) {
    case 1: filter_reg_kernel<1, RAW><<<(unsigned)n, 256, 0, st>>>(A); break;
    case 2: filter_reg_kernel<2, RAW><<<(unsigned)n, 256, 0, st>>>(A); break;
    case 4: filter_reg_kernel<4, RAW><<<(unsigned)n, 256, 0, st>>>(A); break;
    case 8: filter_reg_kernel<8, RAW><<<(unsigned)n, 256, 0, st>>>(A); break;
    case 16: filter_reg_kernel<16, RAW><<<(unsigned)n, 256, 0, st>>>(A); break;
    default:
        if constexpr (RAW) return hipErrorInvalidValue;   // raw input needs a uniform plan
        else filter_reg_kernel<0, false><<<(unsigned)n, 256, 0, st>>>(A);
    }
    return hipGetLastError();
}

FlatInfo make_flats(const double *pos, int n)
{
    FlatInfo fi{};
    fi.n = n;
    for (int i = 0; i < n && i < 32; ++i) fi.pos[i] = pos[i];
    return fi;
}

}  // namespace

hipError_t launch_normalize_hotspot(const pyhst_plan &p, const uint16_t *raw, const float *flats,
                                    const double *flat_pos, int n_flats, const float *dark, float eps, float thr,
                                    int halo_lo, int halo_hi, float *sino, hipStream_t st)
{
    const GeoDev &g = p.gd[0];
    const int R = p.n_slices;
    auto run = [&](auto kernel, int rows) {
        const int n_rb = (R + rows - 1) / rows;
        const int bins = 256 * (HS_ROWS / rows);
        kernel<<<dim3((unsigned)((int64_t)g.K * n_rb), (g.nb + bins - 1) / bins), 256, 0, st>>>(
            raw, flats, make_flats(flat_pos, n_flats), dark, eps, thr, g.K, R, halo_lo + R + halo_hi, halo_lo, g.nb, n_rb, sino);
        return hipGetLastError();
    };
    return R == 1 ? run(normalize_hotspot_kernel<1>, 1) : R == 2 ? run(normalize_hotspot_kernel<2>, 2)
                                                                 : run(normalize_hotspot_kernel<HS_ROWS>, HS_ROWS);
}

hipError_t launch_ring_filter(const pyhst_plan &p, float *sino, const float *obj, int width, double *work,
                              hipStream_t st)
{
    const GeoDev &g = p.gd[0];
    const int S = p.n_slices, K = g.K, L = g.nb;
    ring_mean_kernel<<<dim3((L + 63) / 64, S), 1024, 0, st>>>(sino, obj, K, L, work);
    const dim3 grid((L + 255) / 256, (K + RING_ROWS - 1) / RING_ROWS, S);
    // The window is summed once for all rows, in a launch of its own, unless every workgroup has a compute unit of its own
    // (3 x 24 x 54 9.5 us, apart 13): summed by each workgroup again, 64 slices x 1800 x 2048 take 0.76 ms with half-width 8, 1.6 with 64 and 8.4 with 600, here 0.58,
    // 0.59 and 0.63 (a row per workgroup: 1.31, 1.32 and 1.40); 7 x 721 x 1003 with 8 22 us and 22 (204).
    if ((int64_t)grid.x * grid.y * grid.z > p.cu_count) {
        double *hp = work + (int64_t)S * L;
        ring_highpass_kernel<<<dim3((L + 255) / 256, S), 256, 0, st>>>(work, L, width, hp);
        ring_subtract_kernel<true><<<grid, 256, 0, st>>>(sino, hp, K, L, 0);
    } else {
        ring_subtract_kernel<false><<<grid, 256, 0, st>>>(sino, work, K, L, width);
    }
    return hipGetLastError();
}

hipError_t launch_normalize(const pyhst_plan &p, const uint16_t *raw, const float *flats, const double *flat_pos,
                            int n_flats, const float *dark, float eps, float *sino, hipStream_t st)
{
    const GeoDev &g = p.gd[0];
    const int R = p.n_slices;
    normalize_kernel<<<(unsigned)((int64_t)g.K * R), 256, 0, st>>>(raw, flats, make_flats(flat_pos, n_flats), dark,
                                                                   eps, g.K, R, g.nb, sino);
    return hipGetLastError();
}

hipError_t launch_filter(const pyhst_plan &p, const float *sino, const uint16_t *raw, const float *flats,
                         const double *flat_pos, int n_flats, const float *dark, float eps, float *filt,
                         hipStream_t st)
{
    const GeoDev &g0 = p.gd[p.sd[0].g];
    FilterArgs A{p.t, g0, 0, sino, raw, flats, raw ? make_flats(flat_pos, n_flats) : FlatInfo{}, dark, eps, p.n_slices, filt};
    const int64_t pairs = (int64_t)p.n_slices * ((g0.K + 1) / 2);
    // Few pairs of short rows (a single small slice) keep the LDS passes: with one or two points a thread a pair's own
    // latency is shorter, and the chip has room for every pair at once (256 bins: 90 pairs 4.8 us against 6.3, 720 pairs
    // 5.8 against 6.4, 1024 x 90 pairs 320 against 116; 512 bins: 45 pairs 6.2 against 6.35, 720 pairs 8.2 against 6.8).
    const bool few = p.uniform && g0.P <= 512 && pairs <= 768;
    if (p.n_reg && !few) {
        if (p.uniform) A.per = p.n_reg / p.n_slices;
        const int R = p.uniform ? g0.P >> 8 : 0;
        hipError_t e = raw ? launch_reg<true>(A, R, p.n_reg, st) : launch_reg<false>(A, R, p.n_reg, st);
        if (e != hipSuccess) return e;
    }
    const int rest = few ? (int)pairs : p.n_pairs - p.n_reg;   // row pairs that the register filter does not take
    if (rest == 0) return hipSuccess;
    if (p.uniform) A.per = (g0.K + 1) / 2;
    A.T.pairs += p.n_reg;
    int Pmax = 0;
    for (const auto &g : p.gd)
        if (few || !reg_filter_length(g.P)) Pmax = std::max(Pmax, g.P);
    const size_t lds = (size_t)Pmax * sizeof(float2);
    auto run = [&](auto kernel) {
        if (lds > 65536) {
            hipError_t e = hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        kernel<<<(unsigned)rest, 256, lds, st>>>(A);
        return hipGetLastError();
    };
    if (raw) return run(filter_kernel<true, true>);   // raw input needs a uniform plan
    return p.uniform ? run(filter_kernel<false, true>) : run(filter_kernel<false, false>);
}

}  // namespace pyhst
