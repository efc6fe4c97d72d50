// Least-squares fit of the coefficients (Optimal Image Subtraction, Sec. 2):
// loss and its gradient in D, the float64 normal matrix, an in-place
// Cholesky factorisation, the two triangular solves and the Gauss-Newton
// update.  Everything here is float64 except the basis responses, which come
// from the float32 matrix-core contraction.
//
// Normal matrix.  With Phi[p][(n,m)] = P_m(p) T_n(p),
//   JtJ[(n,m)][(n',m')] = sum_p mask(p) T_n(p) T_n'(p) P_m(p) P_m'(p),
// and P_m P_m' is itself one monomial xh^(i+i') yh^(j+j') of degree at most
// 2 d_s.  So JtJ is assembled from
//   S[mu][n][n'] = sum_p mask(p) Q_mu(p) T_n(p) T_n'(p)
// over the (d_s + 1)(2 d_s + 1) monomials Q_mu of degree <= 2 d_s, which needs
// N^2 per monomial instead of (N M)^2 products per pixel.  Within one image
// row yh is constant, so with Q_mu = xh^a yh^b the Gram sums of a row segment
// are taken for the 2 d_s + 1 powers of xh only,
//   G_a[n][n'] = sum_{x in segment} mask xh^a T_n T_n',
// and S[(a, b)] = sum_segments yh^b G_a is formed by the reduction: 2 d_s + 1
// instead of (d_s + 1)(2 d_s + 1) weighted products per pixel.  The T_n of a
// band of rows are produced by the forward contraction (written out instead
// of being contracted with c_n), then G is accumulated on the float64 matrix
// cores (v_mfma_f64_16x16x4_f64).
#include <cmath>

#include "internal.hpp"

namespace svc {

typedef double d4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------ loss ----

__device__ __forceinline__ bool in_mask(const unsigned char* mask, int H, int W, int h, int x, int y) {
    if (mask) return mask[(size_t)y * W + x] != 0;
    return x >= h && x <= W - 1 - h && y >= h && y <= H - 1 - h;
}

constexpr int LOSS_BLOCKS = 1024;

__global__ void loss_grad_kernel(const float* __restrict__ D, const unsigned char* __restrict__ mask,
                                 int H, int W, int h, float* __restrict__ gD,
                                 double* __restrict__ part) {
    double s = 0.0;
    const size_t n = (size_t)H * W;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const int y = (int)(i / W), x = (int)(i % W);
        const float d = D[i];
        const bool m = in_mask(mask, H, W, h, x, y);
        gD[i] = m ? 2.f * d : 0.f;
        if (m) s += (double)d * d;
    }
    __shared__ double red[256];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) part[blockIdx.x] = red[0];
}

__global__ void sum_kernel(const double* __restrict__ part, int n, double* __restrict__ out) {
    __shared__ double red[256];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) s += part[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

int launch_loss_grad(svconv_plan* p, const float* D, const unsigned char* mask, float* gD,
                     double* loss) {
    hipLaunchKernelGGL(loss_grad_kernel, dim3(LOSS_BLOCKS), dim3(256), 0, p->stream, D, mask, p->H,
                       p->W, p->h, gD, p->dRed);
    int st = hip_status(hipGetLastError(), "loss_grad_kernel");
    if (st || !loss) return st;
    hipLaunchKernelGGL(sum_kernel, dim3(1), dim3(256), 0, p->stream, p->dRed, LOSS_BLOCKS, loss);
    return hip_status(hipGetLastError(), "sum_kernel");
}

// --------------------------------------------------- normal matrix ----

constexpr int NM_PIX_CHUNK = 4096;    // most pixels of one segment
constexpr size_t NM_BAND_BYTES = (size_t)512 << 20;   // basis responses of a band
constexpr size_t NM_PART_BYTES = (size_t)256 << 20;   // its partial sums
constexpr int NM_CHUNKS = 32;         // partial sums of the reduction over segments

// The planes X_0 .. X_(P-1) whose products are summed: the basis responses,
// then (with a background) the constant 1, then (with a right-hand side) I.
struct GramPlanes {
    const float* T;             // responses [N][rows][W] of the band; or R itself for a delta basis
    size_t stride;              // rows * W
    int dfb_k;                  // > 0: plane n is R shifted by the kernel pixel n of this width
    int N, P;
    const float* ones;          // [W + 16] of 1
    const float* I;             // [H][W], nullable
};

struct GramArgs {
    GramPlanes q;
    int W, y_begin, segs, cpr, seg_len, x_lo, x_hi, n_a;
    const unsigned char* mask;  // nullable
    const double* xw;           // [n_a][W] xh^a, 0 outside the interior when mask is null
    double* part;               // [segs][n_a][E]
};

// X_p at row y, band row `row`: pointer to its column 0
__device__ __forceinline__ const float* plane_row(const GramPlanes& q, int p, int row, int y, int W) {
    if (p >= q.N) return (q.I && p == q.P - 1) ? q.I + (size_t)y * W : q.ones;
    if (q.dfb_k) {
        const int h = q.dfb_k / 2, v = p / q.dfb_k - h, u = p % q.dfb_k - h;
        return q.T + (long)(y - v) * W - u;
    }
    return q.T + p * q.stride + (size_t)row * W;
}

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef double d2u __attribute__((ext_vector_type(2), aligned(8)));

// G_a[p][p'] = sum over a segment (up to NM_PIX_CHUNK pixels of one row) of
// mask xh^a X_p X_p', by one wave per segment and power a on the float64
// matrix cores.  The planes are taken as NBF blocks of 16 and R planes over.
// One register serves as both operands (lane (kq, j) of the 16x16x4
// instruction holds row j, k = kq of A and column j, k = kq of B: plane j at
// pixel kq), so a wave that forms all NBF (NBF + 1) / 2 blocks of the upper
// triangle loads and widens each plane once.  The R planes over (2 of 50 in
// the 49-basis fits) would cost a block column padded to 16; their products
// are float64 FMAs on the same registers instead, each lane for its plane and
// pixel, summed over kq at the end.
//
// Bound: float64 matrix cores and vector FMAs, which share an issue rate (66
// and 4.2 cycles measured per instruction, not overlapped): per 4 pixels and
// power 10 blocks -> 6 blocks + 19 vector instructions at 50 planes.  2048 x
// 2048, 50 planes, second order: 2700 -> 1345 us, the reduction below 490 -> 60
// us; 1024 x 1024, delta basis: 780 -> 324 us.
//
// The segments of the powers of one row run on one XCD, whose L2 then serves
// the n_a passes over its planes.
template <int NBF, int R>
__global__ __launch_bounds__(64) void gram_kernel(GramArgs g) {
    constexpr int NBLK = NBF * (NBF + 1) / 2, NR = R ? NBF + 1 : NBF;   // row blocks read
    constexpr int E = NBLK * 256 + R * NR * 16;
    const int xcd = blockIdx.x & 7, i8 = blockIdx.x >> 3;
    const int ea = i8 % g.n_a, seg = (i8 / g.n_a) * 8 + xcd;
    if (seg >= g.segs) return;
    const int lane = threadIdx.x, kq = lane >> 4, j = lane & 15;
    const int row = seg / g.cpr, x_begin = g.x_lo + (seg - row * g.cpr) * g.seg_len;
    const int x_end = min(g.x_hi, x_begin + g.seg_len), y = g.y_begin + row;

    const float* rp[NR];                 // this lane's plane of each row block
    const float* cp[R ? R : 1];          // the planes over (uniform)
#pragma unroll
    for (int b = 0; b < NR; ++b) rp[b] = plane_row(g.q, min(16 * b + j, g.q.P - 1), row, y, g.W);
#pragma unroll
    for (int c = 0; c < R; ++c) cp[c] = plane_row(g.q, min(16 * NBF + c, g.q.P - 1), row, y, g.W);
    const double* wrow = g.xw + (size_t)ea * g.W;
    const unsigned char* mrow = g.mask ? g.mask + (size_t)y * g.W : nullptr;

    d4 acc[NBLK];
    double rem[R ? R : 1][NR];
#pragma unroll
    for (int b = 0; b < NBLK; ++b) acc[b] = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int c = 0; c < R; ++c)
#pragma unroll
        for (int b = 0; b < NR; ++b) rem[c][b] = 0.0;

    // 16 pixels per step: lane group kq takes pixels x0 + 4 kq .. x0 + 4 kq + 3
    // (the k slot of instruction s is pixel x0 + 4 kq + s in both operands)
    struct Step {
        f4u r[NR], c[R ? R : 1];
        d2u w[2];
        unsigned m;
    };
    auto load = [&](int x0) {
        Step o;
        const int x = x0 + 4 * kq;
#pragma unroll
        for (int b = 0; b < NR; ++b) o.r[b] = *reinterpret_cast<const f4u*>(rp[b] + x);
#pragma unroll
        for (int c = 0; c < R; ++c) o.c[c] = *reinterpret_cast<const f4u*>(cp[c] + x);
        o.w[0] = *reinterpret_cast<const d2u*>(wrow + x);
        o.w[1] = *reinterpret_cast<const d2u*>(wrow + x + 2);
        if (mrow) {
            o.m = 0;
#pragma unroll
            for (int s = 0; s < 4; ++s) o.m |= mrow[x + s] ? 1u << s : 0u;
        }
        return o;
    };
    // the last pixels: loads from clamped columns, weight 0 past the end
    auto load_tail = [&](int x0) {
        Step o;
        o.m = 0;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int x = x0 + 4 * kq + s, xc = min(x, x_end - 1);
#pragma unroll
            for (int b = 0; b < NR; ++b) o.r[b][s] = rp[b][xc];
#pragma unroll
            for (int c = 0; c < R; ++c) o.c[c][s] = cp[c][xc];
            o.w[s >> 1][s & 1] = x < x_end ? wrow[xc] : 0.0;
            if (mrow) o.m |= mrow[xc] ? 1u << s : 0u;
        }
        return o;
    };
    auto products = [&](const Step& o) {
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            double w = o.w[s >> 1][s & 1];
            if (mrow && !((o.m >> s) & 1)) w = 0.0;
            double a[NR];
#pragma unroll
            for (int b = 0; b < NR; ++b) a[b] = (double)o.r[b][s];
            int blk = 0;
#pragma unroll
            for (int cb = 0; cb < NBF; ++cb) {
                const double bw = a[cb] * w;
#pragma unroll
                for (int rb = 0; rb <= cb; ++rb, ++blk)
                    acc[blk] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[rb], bw, acc[blk], 0, 0, 0);
            }
#pragma unroll
            for (int c = 0; c < R; ++c) {
                const double d = (double)o.c[c][s] * w;
#pragma unroll
                for (int b = 0; b < NR; ++b) rem[c][b] = fma(a[b], d, rem[c][b]);
            }
        }
    };
    // the operands of one step are requested (into a register set of their
    // own) before the products of the step before it
    const int n_full = max(0, (x_end - x_begin) / 16);
    int x0 = x_begin;
    if (n_full > 0) {
        Step oa = load(x0);
        int t = 0;
        for (; t + 2 <= n_full; t += 2, x0 += 32) {
            const Step ob = load(x0 + 16);
            products(oa);
            oa = load(t + 2 < n_full ? x0 + 32 : x0 + 16);   // past the end: unused
            products(ob);
        }
        if (t < n_full) {
            products(oa);
            x0 += 16;
        }
    }
    if (x0 < x_end) products(load_tail(x0));

    // the float64 16x16x4 instruction stores row 4 e + kq of the 16 x 16
    // block in register e of lane (kq, j): lane (kq, j) holds
    // G[16 rb + 4 e + kq][16 cb + j], block cb (cb + 1) / 2 + rb
    double* dst = g.part + ((size_t)seg * g.n_a + ea) * E;
#pragma unroll
    for (int b = 0; b < NBLK; ++b)
#pragma unroll
        for (int e = 0; e < 4; ++e) dst[b * 256 + (4 * e + kq) * 16 + j] = acc[b][e];
#pragma unroll
    for (int c = 0; c < R; ++c)
#pragma unroll
        for (int b = 0; b < NR; ++b) {
            double v = rem[c][b];
            v += __shfl_xor(v, 16);
            v += __shfl_xor(v, 32);
            if (kq == 0) dst[NBLK * 256 + (c * NR + b) * 16 + j] = v;
        }
}

// Blocks of 16 planes and planes over: a block column padded to 16 costs
// (nbf + 1) matrix products of 66 cycles per 4 pixels, a plane over 2 + nbf + 1
// vector instructions of 4.2 (times the next instance's R), so up to 8 planes
// over two or more blocks and up to 4 over one are cheaper than the block.
struct GramShape {
    int nbf, r;
    int blocks() const { return nbf * (nbf + 1) / 2; }
    int entries() const { return blocks() * 256 + r * (nbf + 1) * 16; }
};

static GramShape gram_shape(int planes) {
    const int full = planes / 16, over = planes % 16;
    const int most = full >= 2 ? 8 : full == 1 ? 4 : 0;
    if (over == 0) return {full, 0};
    if (over > most) return {full + 1, 0};
    return {full, over <= 2 ? 2 : over <= 4 ? 4 : 8};
}

// Entry of the pair (p, p') of planes
__device__ __forceinline__ int gram_entry(int nbf, int r, int p, int p2) {
    const int lo = min(p, p2), hi = max(p, p2), cb = hi >> 4, rb = lo >> 4;
    if (cb < nbf || r == 0) return (cb * (cb + 1) / 2 + rb) * 256 + (lo & 15) * 16 + (hi & 15);
    return nbf * (nbf + 1) / 2 * 256 + ((hi - 16 * nbf) * (nbf + 1) + rb) * 16 + (lo & 15);
}

static int launch_gram(const GramArgs& g, GramShape sh, hipStream_t s) {
    const dim3 grid((unsigned)((g.segs + 7) / 8 * 8 * g.n_a)), block(64);
#define GRAM(NBF, R)                                                                     \
    if (sh.nbf == NBF && sh.r == R) {                                                    \
        hipLaunchKernelGGL((gram_kernel<NBF, R>), grid, block, 0, s, g);                 \
        return hip_status(hipGetLastError(), "gram_kernel");                             \
    }
    GRAM(1, 0) GRAM(1, 2) GRAM(1, 4) GRAM(2, 0) GRAM(2, 2) GRAM(2, 4) GRAM(2, 8)
    GRAM(3, 0) GRAM(3, 2) GRAM(3, 4) GRAM(3, 8) GRAM(4, 0)
#undef GRAM
    return fail(SVCONV_EUNSUPPORTED, "normal matrix: more than 64 planes");
}

// part2[chunk][(a, b)][.] = sum over the chunk's segments (in order) of
// yh(segment row)^b G_a.  Thread (a, e) reads entry e once for every y power
// b <= 2 d - a.  Bound: one read of the partial sums; NM_CHUNKS ranges of
// segments keep the chip busy (in one range, 490 us of the 2048 x 2048 case).
__global__ __launch_bounds__(256) void gram_reduce(const double* __restrict__ part, int E, int n_seg, int cpr,
                                                   int n_a, int y_begin, double sy, double oy,
                                                   double* __restrict__ part2) {
    constexpr int NB_MAX = 2 * kMaxSpatialDegree + 1;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    const int ea = blockIdx.y, n_mu = n_a * (n_a + 1) / 2;
    if (e >= E) return;
    const int per = (n_seg + NM_CHUNKS - 1) / NM_CHUNKS;
    const int c_begin = blockIdx.z * per, c_end = min(n_seg, c_begin + per);
    const int n_eb = n_a - ea;                        // uniform
    double acc[NB_MAX];
#pragma unroll
    for (int eb = 0; eb < NB_MAX; ++eb) acc[eb] = 0.0;
#pragma unroll 8
    for (int c = c_begin; c < c_end; ++c) {
        const double v = part[((size_t)c * n_a + ea) * E + e];
        const double yh = sy * (y_begin + c / cpr) + oy;
        double pw = 1.0;
#pragma unroll
        for (int eb = 0; eb < NB_MAX; ++eb) {
            if (eb < n_eb) acc[eb] += pw * v;
            pw *= yh;
        }
    }
    double* dst = part2 + (size_t)blockIdx.z * n_mu * E + e;
#pragma unroll
    for (int eb = 0; eb < NB_MAX; ++eb) {
        if (eb < n_eb) {
            const int tt = ea + eb;
            dst[(size_t)(tt * (tt + 1) / 2 + eb) * E] = acc[eb];
        }
    }
}

// S (+)= the chunks' sums, in order
__global__ __launch_bounds__(256) void gram_total(const double* __restrict__ part2, int n, int first,
                                                  double* __restrict__ S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = first ? 0.0 : S[i];
#pragma unroll 8
    for (int c = 0; c < NM_CHUNKS; ++c) s += part2[(size_t)c * n + i];
    S[i] = s;
}

// xw[a][x] = xh^a (0 outside [x_lo, x_hi)), the row of ones, and S = 0
__global__ void gram_tables_kernel(int W, int x_lo, int x_hi, double sx, double ox, int n_a, double* __restrict__ xw,
                                   float* __restrict__ ones, double* __restrict__ S, int n_s) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_s) S[i] = 0.0;
    if (i < W + 16) ones[i] = 1.f;
    if (i >= n_a * W) return;
    const int a = i / W, x = i - a * W;
    const double xh = sx * x + ox;
    double p = 1.0;
    for (int t = 0; t < a; ++t) p *= xh;
    xw[i] = (x >= x_lo && x < x_hi) ? p : 0.0;
}

// JtJ[(n,m)][(n',m')] = S[mu(i_m + i_m', j_m + j_m')][n][n'] and, with q >= 0,
// rhs[(n,m)] = S[mu(i_m, j_m)][n][q] = sum_{p in mask} P_m T_n I (plane q holds I)
__global__ void assemble_jtj(const double* __restrict__ S, int E, int nbf, int r, int N, int M, int q,
                             double* __restrict__ JtJ, double* __restrict__ rhs) {
    const int NM = N * M;
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= NM * NM) return;
    const int row = idx / NM, c = idx - row * NM;
    const int n = row / M, m = row - n * M, n2 = c / M, m2 = c - n2 * M;
    auto expo = [](int k, int& i, int& jj) {
        int t = 0;
        while ((t + 1) * (t + 2) / 2 <= k) ++t;
        jj = k - t * (t + 1) / 2;
        i = t - jj;
    };
    int i1, j1, i2, j2;
    expo(m, i1, j1);
    expo(m2, i2, j2);
    const int t = i1 + i2 + j1 + j2, mu = t * (t + 1) / 2 + j1 + j2;
    JtJ[idx] = S[(size_t)mu * E + gram_entry(nbf, r, n, n2)];
    if (q >= 0 && c == 0) rhs[row] = S[(size_t)m * E + gram_entry(nbf, r, n, q)];   // mu(i_m, j_m) = m
}

// The basis responses T_n + s beta_n of rows [y0, y0 + rows) into the plan's band
static int band_responses(svconv_plan* p, const float* R, int y0, int rows) {
    double sx = 0, ox = 0, sy = 0, oy = 0;
    if (p->Wf > 1) { sx = 2.0 / (p->Wf - 1); ox = sx * p->x0 - 1.0; }
    if (p->Hf > 1) { sy = 2.0 / (p->Hf - 1); oy = sy * p->y0 - 1.0; }
    if (sep_form(p)) {
        // through the separable factors
        SepArgs sa{};
        sa.X = R;
        sa.H = p->H;
        sa.W = p->W;
        sa.h = p->h;
        sa.ped = p->pedestal;
        sa.G = (int)p->sigmas.size();
        sa.fam = p->dSepFam;
        sa.f1d = p->dSep1d;
        sa.beta = p->dBeta;
        sa.coef = p->dF32;   // not read in this mode
        sa.M = p->M;
        sa.d_s = p->d_s;
        sa.sx = sx; sa.ox = ox; sa.sy = sy; sa.oy = oy;
        sa.y_begin = y0;
        sa.n_rows = rows;
        sa.tout = p->dTband;
        return launch_contract_sep(sa, p->stream);
    }
    ContractArgs c{};
    c.X = R;
    c.H = p->H;
    c.W = p->W;
    c.h = p->h;
    c.NF = p->N;
    c.M = p->M;
    c.d_s = p->d_s;
    c.beta = p->dBeta;
    c.ped = p->pedestal;
    c.sx = sx; c.ox = ox; c.sy = sy; c.oy = oy;
    c.tout = p->dTband;
    // basis-form kernel with out == nullptr: coefficients are neither read nor used
    c.coef = p->dF32;
    c.y_begin = y0;
    c.n_rows = rows;
    return launch_contract_f32(c, p->dFragF32, (p->N + 15) / 16, p->stream);
}

// With a background polynomial the fit has one more "basis" whose response
// is the constant 1 (bg = sum_m b_m P_m * 1), so the same Gram sums give the
// background rows and columns of the normal matrix.  With I and rhs given, one
// more plane is I, and the Gram sums of the basis planes with it are the
// right-hand side rhs[(n,m)] = sum_p P_m T_n I of the normal equations.
int launch_normal_matrix(svconv_plan* p, const float* R, const float* I, const unsigned char* mask,
                         double* JtJ, double* rhs) {
    const int NF = p->N + p->bg;
    const bool want_rhs = (I != nullptr && rhs != nullptr);
    const int planes = NF + (want_rhs ? 1 : 0);
    if (planes > 64)
        return fail(SVCONV_EUNSUPPORTED,
                    "normal equations need N (+1 with a background, +1 with the right-hand side) <= 64");
    const GramShape sh = gram_shape(planes);
    const int E = sh.entries();
    const int n_mu = (2 * p->d_s + 1) * (2 * p->d_s + 2) / 2;
    const int n_a = 2 * p->d_s + 1;                       // powers of xh
    // The responses of a delta basis at interior pixels are pixels of R: no
    // response planes are written for it (with a mask, stamps may reach the
    // border, where R is 0 outside the image, so the planes are formed)
    const bool shifts = p->dfb && !mask;
    // rows and columns that can have weight; columns start on 4 where the
    // weights cover the columns below (a shifted R has none left of x = h)
    const int y_lo = mask ? 0 : p->h, y_hi = mask ? p->H : p->H - p->h;
    const int x_in = mask ? 0 : p->h, x_hi = mask ? p->W : p->W - p->h;
    const int x_lo = shifts ? x_in : x_in & ~3;
    const int rows_all = y_hi > y_lo && x_hi > x_in ? y_hi - y_lo : 0;
    // segments: whole rows up to NM_PIX_CHUNK pixels, shorter where there would
    // be less than four waves per SIMD
    int seg_len = NM_PIX_CHUNK, cpr = 1;
    for (;; seg_len /= 2) {
        cpr = x_hi > x_lo ? (x_hi - x_lo + seg_len - 1) / seg_len : 1;
        if ((long)cpr * rows_all * n_a >= 4096 || seg_len <= 128) break;
    }
    const size_t row_bytes = (size_t)p->N * p->W * sizeof(float), part_row = (size_t)cpr * n_a * E;
    size_t band = shifts ? (size_t)rows_all : NM_BAND_BYTES / row_bytes;
    if (band > NM_PART_BYTES / (part_row * sizeof(double))) band = NM_PART_BYTES / (part_row * sizeof(double));
    if (band < 8) band = 8;
    if (band > (size_t)rows_all) band = rows_all;
    const size_t part_elems = band * part_row, part2_elems = (size_t)NM_CHUNKS * n_mu * E;
    const size_t s_elems = (size_t)n_mu * E, xw_elems = (size_t)n_a * p->W, ones_elems = ((size_t)p->W + 16 + 1) / 2;
    const size_t tband_bytes = shifts ? 0 : band * row_bytes;
    const size_t nmpart_bytes = (part_elems + part2_elems + s_elems + xw_elems + ones_elems) * sizeof(double);
    // scratch of the normal matrix: allocated on its first call (grown when
    // a later call needs more), kept by the plan
    if (p->tband_bytes < tband_bytes || p->nmpart_bytes < nmpart_bytes) {
        if (p->dTband) (void)hipFree(p->dTband);
        if (p->dNMpart) (void)hipFree(p->dNMpart);
        p->dTband = nullptr;
        p->dNMpart = nullptr;
        p->tband_bytes = p->nmpart_bytes = 0;
        if ((tband_bytes && hipMalloc((void**)&p->dTband, tband_bytes) != hipSuccess) ||
            hipMalloc((void**)&p->dNMpart, nmpart_bytes) != hipSuccess) {
            (void)hipGetLastError();
            if (p->dTband) (void)hipFree(p->dTband);
            p->dTband = nullptr;
            p->dNMpart = nullptr;
            return fail(SVCONV_ENOMEM, "normal-matrix scratch");
        }
        p->tband_bytes = tband_bytes;
        p->nmpart_bytes = nmpart_bytes;
    }
    double* part2 = p->dNMpart + part_elems;
    double* S = part2 + part2_elems;
    double* xw = S + s_elems;
    float* ones = reinterpret_cast<float*>(xw + xw_elems);
    double sx = 0, ox = 0, sy = 0, oy = 0;
    if (p->Wf > 1) { sx = 2.0 / (p->Wf - 1); ox = sx * p->x0 - 1.0; }
    if (p->Hf > 1) { sy = 2.0 / (p->Hf - 1); oy = sy * p->y0 - 1.0; }
    {
        size_t n = s_elems > xw_elems ? s_elems : xw_elems;
        if (n < (size_t)p->W + 16) n = (size_t)p->W + 16;
        hipLaunchKernelGGL(gram_tables_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, p->stream, p->W, x_in,
                           x_hi, sx, ox, n_a, xw, ones, S, (int)s_elems);
    }
    int st = hip_status(hipGetLastError(), "gram_tables_kernel");
    if (st) return st;

    GramArgs g{};
    g.q.dfb_k = shifts ? p->k : 0;
    g.q.T = shifts ? R : p->dTband;
    g.q.N = p->N;
    g.q.P = planes;
    g.q.ones = ones;
    g.q.I = want_rhs ? I : nullptr;
    g.W = p->W;
    g.cpr = cpr;
    g.seg_len = seg_len;
    g.x_lo = x_lo;
    g.x_hi = x_hi;
    g.n_a = n_a;
    g.mask = mask;
    g.xw = xw;
    g.part = p->dNMpart;
    for (int y0 = y_lo; y0 < y_lo + rows_all; y0 += (int)band) {
        const int rows = min((int)band, y_lo + rows_all - y0);
        if (!shifts) {
            st = band_responses(p, R, y0, rows);
            if (st) return st;
        }
        g.q.stride = (size_t)rows * p->W;
        g.y_begin = y0;
        g.segs = rows * cpr;
        st = launch_gram(g, sh, p->stream);
        if (st) return st;
        hipLaunchKernelGGL(gram_reduce, dim3((E + 255) / 256, n_a, NM_CHUNKS), dim3(256), 0, p->stream, p->dNMpart, E,
                           g.segs, cpr, n_a, y0, sy, oy, part2);
        st = hip_status(hipGetLastError(), "gram_reduce");
        if (st) return st;
        hipLaunchKernelGGL(gram_total, dim3((unsigned)((s_elems + 255) / 256)), dim3(256), 0, p->stream, part2,
                           (int)s_elems, y0 == y_lo ? 1 : 0, S);
        st = hip_status(hipGetLastError(), "gram_total");
        if (st) return st;
    }
    const int NM = NF * p->M;
    hipLaunchKernelGGL(assemble_jtj, dim3((NM * NM + 255) / 256), dim3(256), 0, p->stream, S, E, sh.nbf, sh.r, NF,
                       p->M, want_rhs ? NF : -1, JtJ, rhs);
    return hip_status(hipGetLastError(), "assemble_jtj");
}

// -------------------------------------------------------- Cholesky ----

// Right-looking in-place factorisation by one workgroup; A stays in global
// memory (at most 1024 x 1024 doubles, resident in L2).  status[0] becomes
// the first non-positive pivot index + 1 (0 = SPD).
__global__ __launch_bounds__(1024) void cholesky_kernel(double* __restrict__ A, int n,
                                                        int* __restrict__ status) {
    __shared__ int bad;
    __shared__ double piv;
    const int tid = threadIdx.x;
    if (tid == 0) bad = 0;
    __syncthreads();
    for (int jc = 0; jc < n; ++jc) {
        if (tid == 0) {
            const double d = A[(size_t)jc * n + jc];
            if (!(d > 0.0) || !isfinite(d)) {
                bad = jc + 1;
                piv = 1.0;
            } else {
                piv = sqrt(d);
                A[(size_t)jc * n + jc] = piv;
            }
        }
        __syncthreads();
        if (bad) break;
        const double inv = 1.0 / piv;
        for (int i = jc + 1 + tid; i < n; i += 1024) A[(size_t)i * n + jc] *= inv;
        __syncthreads();
        // trailing update of the lower triangle: A[i][c] -= L[i][jc] L[c][jc], jc < c <= i
        const int m = n - jc - 1;
        const long cnt = (long)m * (m + 1) / 2;
        for (long q = tid; q < cnt; q += 1024) {
            // row-major enumeration of the lower triangle of an m x m block
            long i = (long)((sqrt(8.0 * q + 1.0) - 1.0) * 0.5);
            while (i * (i + 1) / 2 > q) --i;
            while ((i + 1) * (i + 2) / 2 <= q) ++i;
            const long c = q - i * (i + 1) / 2;
            const int ii = jc + 1 + (int)i, cc = jc + 1 + (int)c;
            A[(size_t)ii * n + cc] -= A[(size_t)ii * n + jc] * A[(size_t)cc * n + jc];
        }
        __syncthreads();
    }
    __syncthreads();
    if (!bad) {
        for (long q = tid; q < (long)n * n; q += 1024) {
            const int i = (int)(q / n), c = (int)(q % n);
            if (c > i) A[q] = 0.0;
        }
    }
    if (tid == 0) status[0] = bad;
}

// Blocked right-looking factorisation for larger matrices: for each block
// column k0 of width CH_NB, one workgroup factors the diagonal block in LDS
// and solves the panel below it (L21 = A21 L11^-T), then one workgroup per
// 32 x 32 tile of the trailing lower triangle applies A22 -= L21 L21^T.
constexpr int CH_NB = 32;

__global__ __launch_bounds__(256) void chol_panel_kernel(double* __restrict__ A, int n, int k0,
                                                         int* __restrict__ status) {
    __shared__ double L[CH_NB][CH_NB + 1];
    __shared__ int bad;
    const int tid = threadIdx.x;
    const int nb = min(CH_NB, n - k0);
    for (int q = tid; q < nb * nb; q += 256) {
        const int r = q / nb, c = q - r * nb;
        L[r][c] = A[(size_t)(k0 + r) * n + k0 + c];
    }
    if (tid == 0) bad = status[0];
    __syncthreads();
    for (int j = 0; j < nb; ++j) {
        if (tid == 0) {
            double d = L[j][j];
            if (!(d > 0.0) || !isfinite(d)) {
                if (!bad) bad = k0 + j + 1;
                d = 1.0;
            }
            L[j][j] = sqrt(d);
        }
        __syncthreads();
        const double inv = 1.0 / L[j][j];
        for (int i = j + 1 + tid; i < nb; i += 256) L[i][j] *= inv;
        __syncthreads();
        const int m = nb - j - 1;
        for (int q = tid; q < m * m; q += 256) {
            const int i = j + 1 + q / m, c = j + 1 + q % m;
            if (c <= i) L[i][c] -= L[i][j] * L[c][j];
        }
        __syncthreads();
    }
    for (int q = tid; q < nb * nb; q += 256) {
        const int r = q / nb, c = q - r * nb;
        A[(size_t)(k0 + r) * n + k0 + c] = (c <= r) ? L[r][c] : 0.0;
    }
    // panel rows below: x L11^T = a, forward substitution over the block's
    // columns on the row held in registers; the empty asm with a memory clobber
    // keeps the compiler from hoisting all of L11 into registers across rows
    for (int i = k0 + nb + tid; i < n; i += 256) {
        asm volatile("" ::: "memory");
        double x[CH_NB];
        double* row = A + (size_t)i * n + k0;
#pragma unroll
        for (int c = 0; c < CH_NB; ++c) {
            if (c < nb) {
                double s = row[c];
#pragma unroll
                for (int t = 0; t < c; ++t) s -= x[t] * L[c][t];
                x[c] = s / L[c][c];
                row[c] = x[c];
            }
        }
    }
    if (tid == 0) status[0] = bad;
}

// A22 -= L21 L21^T on the lower triangle; block b is tile (ti, tj), tj <= ti
__global__ __launch_bounds__(256) void chol_update_kernel(double* __restrict__ A, int n, int k0,
                                                          int nb) {
    __shared__ double Li[CH_NB][CH_NB + 1], Lj[CH_NB][CH_NB + 1];
    const int b = blockIdx.x;
    int ti = (int)((sqrt(8.0 * b + 1.0) - 1.0) * 0.5);
    while (ti * (ti + 1) / 2 > b) --ti;
    while ((ti + 1) * (ti + 2) / 2 <= b) ++ti;
    const int tj = b - ti * (ti + 1) / 2;
    const int k1 = k0 + nb;
    const int r0 = k1 + 32 * ti, c0 = k1 + 32 * tj;
    const int tid = threadIdx.x;
    for (int q = tid; q < 32 * nb; q += 256) {
        const int r = q / nb, c = q - r * nb;
        Li[r][c] = (r0 + r < n) ? A[(size_t)(r0 + r) * n + k0 + c] : 0.0;
        Lj[r][c] = (c0 + r < n) ? A[(size_t)(c0 + r) * n + k0 + c] : 0.0;
    }
    __syncthreads();
    const int cc = tid & 31, rb = tid >> 5;     // column, first of 4 rows (stride 8)
    for (int rr = rb; rr < 32; rr += 8) {
        const int gi = r0 + rr, gj = c0 + cc;
        if (gi < n && gj < n && gj <= gi) {
            double s = 0.0;
            for (int t = 0; t < nb; ++t) s = fma(Li[rr][t], Lj[cc][t], s);
            A[(size_t)gi * n + gj] -= s;
        }
    }
}

__global__ void chol_zero_upper(double* __restrict__ A, int n) {
    const size_t total = (size_t)n * n;
    for (size_t q = (size_t)blockIdx.x * blockDim.x + threadIdx.x; q < total;
         q += (size_t)gridDim.x * blockDim.x) {
        const int i = (int)(q / n), c = (int)(q % n);
        if (c > i) A[q] = 0.0;
    }
}

__global__ void chol_status_clear(int* status) {
    if (threadIdx.x == 0) status[0] = 0;
}

int launch_cholesky(svconv_plan* p, double* A, int n) {
    int st = SVCONV_OK;
    if (n <= 64) {
        hipLaunchKernelGGL(cholesky_kernel, dim3(1), dim3(1024), 0, p->stream, A, n, p->dStatus);
        st = hip_status(hipGetLastError(), "cholesky_kernel");
    } else {
        hipLaunchKernelGGL(chol_status_clear, dim3(1), dim3(64), 0, p->stream, p->dStatus);
        st = hip_status(hipGetLastError(), "chol_status_clear");
        for (int k0 = 0; k0 < n && !st; k0 += CH_NB) {
            const int nb = (n - k0) < CH_NB ? (n - k0) : CH_NB;
            hipLaunchKernelGGL(chol_panel_kernel, dim3(1), dim3(256), 0, p->stream, A, n, k0, p->dStatus);
            st = hip_status(hipGetLastError(), "chol_panel_kernel");
            const int rest = n - k0 - nb;
            if (!st && rest > 0) {
                const int nt = (rest + 31) / 32;
                hipLaunchKernelGGL(chol_update_kernel, dim3(nt * (nt + 1) / 2), dim3(256), 0, p->stream,
                                   A, n, k0, nb);
                st = hip_status(hipGetLastError(), "chol_update_kernel");
            }
        }
        if (!st) {
            hipLaunchKernelGGL(chol_zero_upper, dim3(256), dim3(256), 0, p->stream, A, n);
            st = hip_status(hipGetLastError(), "chol_zero_upper");
        }
    }
    if (st) return st;
    int bad = 0;
    st = hip_status(hipMemcpyAsync(&bad, p->dStatus, sizeof(int), hipMemcpyDeviceToHost, p->stream),
                    "copy status");
    if (!st) st = hip_status(hipStreamSynchronize(p->stream), "hipStreamSynchronize");
    if (st) return st;
    if (bad) return fail(SVCONV_ENOTSPD, "pivot " + std::to_string(bad - 1) + " is not positive");
    return SVCONV_OK;
}

// x = L^-T L^-1 rhs by blocked substitutions in one workgroup of 1024
// threads.  Per block of 32 unknowns, one wave solves the 32 x 32 triangle
// (each unknown broadcast across the lanes, the diagonal's reciprocals formed
// first); then every thread folds the block's unknowns into the right-hand
// side entries still to be solved (right-looking): one row of the panel per
// thread in the forward pass (32 independent loads of contiguous doubles),
// one column per thread in the backward pass (loads coalesced across the
// wave).  So each block waits on memory once.  v holds the right-hand side,
// then the solution.
constexpr int CS_B = 32;

__global__ __launch_bounds__(1024) void chol_solve_kernel(const double* __restrict__ L,
                                                          const double* __restrict__ rhs,
                                                          double* __restrict__ x, int n) {
    extern __shared__ double v[];   // n doubles
    const int tid = threadIdx.x;
    for (int i = tid; i < n; i += 1024) v[i] = rhs[i];
    __syncthreads();
    const int nblk = (n + CS_B - 1) / CS_B;
    // forward: L y = b
    for (int kb = 0; kb < nblk; ++kb) {
        const int j0 = kb * CS_B, nb = min(CS_B, n - j0);
        if (tid < 64) {
            // lane t < nb: row j0 + t of the triangle, loaded into registers first
            const int t = tid;
            const bool live = t < nb;
            const double* Lt = L + (size_t)(j0 + (live ? t : 0)) * n + j0;
            double l[CS_B];
#pragma unroll
            for (int j = 0; j < CS_B; ++j) l[j] = (live && j < nb) ? Lt[j] : 0.0;
            const double inv = live ? 1.0 / Lt[t] : 0.0;
            double acc = live ? v[j0 + t] : 0.0;
#pragma unroll
            for (int j = 0; j < CS_B; ++j) {
                if (j < nb) {
                    const double yj = __shfl(acc, j) * __shfl(inv, j);
                    if (t > j) acc = fma(-l[j], yj, acc);
                    if (t == j) acc = yj;
                }
            }
            if (live) v[j0 + t] = acc;
        }
        __syncthreads();
        // rows below the block: v[i] -= L[i][j0 .. j0 + nb) y
        for (int i = j0 + nb + tid; i < n; i += 1024) {
            const double* Li = L + (size_t)i * n + j0;
            double s = 0.0;
            if (nb == CS_B) {
                // a full block: the row's loads issued together
                double l[CS_B];
#pragma unroll
                for (int c = 0; c < CS_B; ++c) l[c] = Li[c];
#pragma unroll
                for (int c = 0; c < CS_B; ++c) s = fma(l[c], v[j0 + c], s);
            } else {
                for (int c = 0; c < nb; ++c) s = fma(Li[c], v[j0 + c], s);
            }
            v[i] -= s;
        }
        __syncthreads();
    }
    // backward: L^T x = y
    for (int kb = nblk - 1; kb >= 0; --kb) {
        const int j0 = kb * CS_B, nb = min(CS_B, n - j0);
        if (tid < 64) {
            // lane t < nb: column j0 + t of the triangle, loaded into registers first
            const int t = tid;
            const bool live = t < nb;
            const double* Lc = L + (size_t)j0 * n + j0 + (live ? t : 0);
            double l[CS_B];
#pragma unroll
            for (int j = 0; j < CS_B; ++j) l[j] = (live && j < nb) ? Lc[(size_t)j * n] : 0.0;
            const double inv = live ? 1.0 / Lc[(size_t)t * n] : 0.0;
            double acc = live ? v[j0 + t] : 0.0;
#pragma unroll
            for (int j = CS_B - 1; j >= 0; --j) {
                if (j < nb) {
                    const double xj = __shfl(acc, j) * __shfl(inv, j);
                    if (t < j) acc = fma(-l[j], xj, acc);
                    if (t == j) acc = xj;
                }
            }
            if (live) v[j0 + t] = acc;
        }
        __syncthreads();
        // columns left of the block: v[c] -= sum_r L[j0 + r][c] x[j0 + r]
        for (int c = tid; c < j0; c += 1024) {
            double s = 0.0;
            if (nb == CS_B) {
                double l[CS_B];
#pragma unroll
                for (int r = 0; r < CS_B; ++r) l[r] = L[(size_t)(j0 + r) * n + c];
#pragma unroll
                for (int r = 0; r < CS_B; ++r) s = fma(l[r], v[j0 + r], s);
            } else {
                for (int r = 0; r < nb; ++r) s = fma(L[(size_t)(j0 + r) * n + c], v[j0 + r], s);
            }
            v[c] -= s;
        }
        __syncthreads();
    }
    for (int i = tid; i < n; i += 1024) x[i] = v[i];
}

int launch_cholesky_solve(svconv_plan* p, const double* L, const double* rhs, double* x, int n) {
    hipLaunchKernelGGL(chol_solve_kernel, dim3(1), dim3(1024), (size_t)n * sizeof(double), p->stream,
                       L, rhs, x, n);
    return hip_status(hipGetLastError(), "chol_solve_kernel");
}

// --------------------------------------------------------- updates ----

__global__ void scale_kernel(double* v, double s, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) v[i] *= s;
}

__global__ void copy_a_kernel(const double* a64, float* a32, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) a32[i] = (float)a64[i];
}

// a64 -= delta, a32 = float(a64), norm = ||delta||_2 (one workgroup)
__global__ __launch_bounds__(1024) void gn_update_kernel(const double* __restrict__ delta,
                                                         double* __restrict__ a64,
                                                         float* __restrict__ a32, int n,
                                                         double* __restrict__ norm) {
    __shared__ double red[1024];
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) {
        const double d = delta[i];
        const double v = a64[i] - d;
        a64[i] = v;
        a32[i] = (float)v;
        s += d * d;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *norm = sqrt(red[0]);
}

int launch_scale(svconv_plan* p, double* v, double s, int n) {
    hipLaunchKernelGGL(scale_kernel, dim3((n + 255) / 256), dim3(256), 0, p->stream, v, s, n);
    return hip_status(hipGetLastError(), "scale_kernel");
}

int launch_copy_a(svconv_plan* p, const double* a64, float* a32, int n) {
    hipLaunchKernelGGL(copy_a_kernel, dim3((n + 255) / 256), dim3(256), 0, p->stream, a64, a32, n);
    return hip_status(hipGetLastError(), "copy_a_kernel");
}

// g = A a - rhs (the half-gradient of the loss, J^T D, from the normal
// equations): one wave per row of the symmetric A, lanes over its columns.
// The dot product is compensated (error-free products and sums, Ogita, Rump
// and Oishi's Dot2): g is then as accurate as if formed in twice the float64
// precision and rounded once, which iterative refinement needs to converge
// past cond(A) eps (A a and rhs nearly cancel at the solution).
__device__ __forceinline__ void two_sum(double a, double b, double& s, double& e) {
#pragma clang fp contract(off)
    s = a + b;
    const double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

__device__ __forceinline__ void two_prod(double a, double b, double& p, double& e) {
#pragma clang fp contract(off)
    p = a * b;
    e = fma(a, b, -p);
}

__global__ __launch_bounds__(256) void ls_grad_kernel(const double* __restrict__ A,
                                                      const double* __restrict__ a,
                                                      const double* __restrict__ rhs, int n,
                                                      double* __restrict__ g) {
#pragma clang fp contract(off)
    const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (row >= n) return;
    const double* Ar = A + (size_t)row * n;
    double s = 0.0, c = 0.0;   // sum and its accumulated error terms
    for (int k = lane; k < n; k += 64) {
        double p, pe, t, te;
        two_prod(Ar[k], a[k], p, pe);
        two_sum(s, p, t, te);
        s = t;
        c += te + pe;
    }
    for (int o = 32; o > 0; o >>= 1) {
        const double so = __shfl_xor(s, o), co = __shfl_xor(c, o);
        double t, te;
        two_sum(s, so, t, te);
        s = t;
        c += co + te;
    }
    if (lane == 0) {
        double t, te;
        two_sum(s, -rhs[row], t, te);
        g[row] = t + (c + te);
    }
}

int launch_ls_grad(svconv_plan* p, const double* A, const double* a64, const double* rhs, double* g, int n) {
    hipLaunchKernelGGL(ls_grad_kernel, dim3((n + 3) / 4), dim3(256), 0, p->stream, A, a64, rhs, n, g);
    return hip_status(hipGetLastError(), "ls_grad_kernel");
}

int launch_gn_update(svconv_plan* p, const double* delta, double* a64, float* a32, int n) {
    // the step norm lands right after the loss scalar in the plan's vector scratch
    double* norm = p->dVec + 2 * (size_t)n + 1;
    hipLaunchKernelGGL(gn_update_kernel, dim3(1), dim3(1024), 0, p->stream, delta, a64, a32, n, norm);
    return hip_status(hipGetLastError(), "gn_update_kernel");
}

}  // namespace svc
