// Least-squares fit of the coefficients (Optimal Image Subtraction, Sec. 2):
// loss and its gradient in D, the float64 normal matrix, an in-place
// Cholesky factorisation, the two triangular solves and the Gauss-Newton
// update.  Everything here is float64 except the planes of basis responses,
// which are held in float32: those of the dense forms come from the float32
// matrix-core contraction, those of the separable forms are formed in float64
// and rounded once, and those of a delta basis without a mask are pixels of R.
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
constexpr int NM_CHUNKS = 32;         // most partial sums of the reduction over segments

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
// b <= 2 d - a.  Bound: one read of the partial sums; up to NM_CHUNKS ranges of
// segments keep the chip busy (in one range, 490 us of the 2048 x 2048 case), at
// least 8 segments each, so that the sums of small frames, which gram_total
// reads again, stay few (20 x 30, 49 bases, fourth order: 64.3 -> 55.1 us a call).
__global__ __launch_bounds__(256) void gram_reduce(const double* __restrict__ part, int E, int n_seg, int cpr,
                                                   int n_a, int y_begin, double sy, double oy,
                                                   double* __restrict__ part2) {
    constexpr int NB_MAX = 2 * kMaxSpatialDegree + 1;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    const int ea = blockIdx.y, n_mu = n_a * (n_a + 1) / 2;
    if (e >= E) return;
    const int per = (n_seg + gridDim.z - 1) / gridDim.z;
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
__global__ __launch_bounds__(256) void gram_total(const double* __restrict__ part2, int chunks, int n, int first,
                                                  double* __restrict__ S) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double s = first ? 0.0 : S[i];
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) s += part2[(size_t)c * n + i];
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

// Scratch of the normal matrix, kept by the plan: allocated on its first call,
// and grown by a later call that needs more.  Each buffer on its own, and never
// smaller: calls with and without a mask, a background or a right-hand side
// need different shares of the two, and would otherwise free and allocate both
// on every change from one to the other.
template <class T>
static int grow(T*& ptr, size_t& have, size_t need) {
    if (have >= need) return SVCONV_OK;
    if (ptr) (void)hipFree(ptr);
    ptr = nullptr;
    have = 0;
    if (hipMalloc((void**)&ptr, need) != hipSuccess) {
        (void)hipGetLastError();
        ptr = nullptr;
        return fail(SVCONV_ENOMEM, "normal-matrix scratch");
    }
    have = need;
    return SVCONV_OK;
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
    int st = grow(p->dTband, p->tband_bytes, tband_bytes);
    if (!st) st = grow(p->dNMpart, p->nmpart_bytes, nmpart_bytes);
    if (st) return st;
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
    st = hip_status(hipGetLastError(), "gram_tables_kernel");
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
        const int chunks = min(NM_CHUNKS, (g.segs + 7) / 8);
        hipLaunchKernelGGL(gram_reduce, dim3((E + 255) / 256, n_a, chunks), dim3(256), 0, p->stream, p->dNMpart, E,
                           g.segs, cpr, n_a, y0, sy, oy, part2);
        st = hip_status(hipGetLastError(), "gram_reduce");
        if (st) return st;
        hipLaunchKernelGGL(gram_total, dim3((unsigned)((s_elems + 255) / 256)), dim3(256), 0, p->stream, part2,
                           chunks, (int)s_elems, y0 == y_lo ? 1 : 0, S);
        st = hip_status(hipGetLastError(), "gram_total");
        if (st) return st;
    }
    const int NM = NF * p->M;
    hipLaunchKernelGGL(assemble_jtj, dim3((NM * NM + 255) / 256), dim3(256), 0, p->stream, S, E, sh.nbf, sh.r, NF,
                       p->M, want_rhs ? NF : -1, JtJ, rhs);
    return hip_status(hipGetLastError(), "assemble_jtj");
}

// -------------------------------------------------------- Cholesky ----

// Blocked right-looking factorisation, one launch per block column k0 of
// CH_NB = 32: every workgroup factors the 32 x 32 diagonal block for itself,
// solves the two 32-row panels its tile of the trailing lower triangle needs
// (L21 = A21 L11^-T) and applies A22 -= L21 L21^T to that tile.  Factoring the
// block in every workgroup costs nothing (they run side by side) and saves the
// launch between panel and update; it is done by one wave with a row per lane
// in registers, entries of other rows broadcast by v_readlane.
// Bound: the serial chain of the 32 pivots (a square root, a quotient and a
// rank-1 update each).  n = 294: 443 us (panel kernel with 4 barriers per
// column 34 us a block, then an update kernel) -> 196 us with the host's launches
// and status copy; n = 735: 1420 -> 422 us.
//
// Workgroups still read the lower triangle of the block column while others
// finish it, so the results go where nobody reads: L21^T and the strict lower
// part of L11, transposed, into the upper triangle, the diagonal into `diag`.
// chol_finish_kernel moves them to their places and clears the upper triangle
// (a matrix of one block is written in place: n = 6 39.1 -> 32.5 us a call).
constexpr int CH_NB = 32;

// v of lane `l` (uniform), through scalar registers
__device__ __forceinline__ double lane_value(double v, int l) {
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), l);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), l);
    return __hiloint2double(hi, lo);
}

// root = sqrt(d) and inv = 1 / sqrt(d) for finite d > 0, by Goldschmidt's
// iteration from the hardware's estimate, which is within 2^-23: two steps take
// that past 2^-52 (1.5 e^2 each), and the root is corrected by its remainder.
// inv is within an ulp or two, which quotient() makes up for.  The library's
// square root and division after one another are 40 dependent instructions,
// the larger part of a pivot's latency.
__device__ __forceinline__ void sqrt_both(double d, double& root, double& inv) {
    const double y = __builtin_amdgcn_rsq(d);
    double g = d * y, h = 0.5 * y;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const double r = fma(-h, g, 0.5);
        g = fma(g, r, g);
        h = fma(h, r, h);
    }
    root = fma(fma(-g, g, d), h, g);
    inv = h + h;
}

// v / piv from inv = 1 / piv within an ulp or two: the remainder of v inv,
// formed exactly, corrects it to the rounded quotient but for rare last bits.
__device__ __forceinline__ double quotient(double v, double piv, double inv) {
    const double x = v * inv;
    return fma(fma(-x, piv, v), inv, x);
}

__global__ __launch_bounds__(256) void chol_step_kernel(double* __restrict__ A, int n, int k0,
                                                        double* __restrict__ diag, int* __restrict__ status) {
    __shared__ double L11[CH_NB][CH_NB + 1];                    // A11, then L11
    __shared__ __attribute__((aligned(16))) double Lt[CH_NB][CH_NB + 2];   // its transpose
    __shared__ double inv[CH_NB], P[2][CH_NB][CH_NB + 1];       // 1 / pivots; the two panels
    const int tid = threadIdx.x;
    const int nb = min(CH_NB, n - k0), k1 = k0 + nb;
    int ti = (int)((sqrt(8.0 * blockIdx.x + 1.0) - 1.0) * 0.5);
    while (ti * (ti + 1) / 2 > (int)blockIdx.x) --ti;
    while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.x) ++ti;
    const int tj = (int)blockIdx.x - ti * (ti + 1) / 2;
    const int r0 = k1 + 32 * ti, c0 = k1 + 32 * tj;

    // all of the workgroup's operands are requested together
    const int cc = tid & 31, rq = tid >> 5;
    double d11[4], pi[4], pj[4], a22[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = rq + 8 * i;
        d11[i] = A[(size_t)min(k0 + r, n - 1) * n + min(k0 + cc, n - 1)];
        pi[i] = A[(size_t)min(r0 + r, n - 1) * n + min(k0 + cc, n - 1)];
        pj[i] = A[(size_t)min(c0 + r, n - 1) * n + min(k0 + cc, n - 1)];
        a22[i] = A[(size_t)min(r0 + r, n - 1) * n + min(c0 + cc, n - 1)];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = rq + 8 * i;
        // a short block is completed with the identity
        L11[r][cc] = (r < nb && cc <= r) ? d11[i] : (r == cc ? 1.0 : 0.0);
        P[0][r][cc] = (r0 + r < n && cc < nb) ? pi[i] : 0.0;
        P[1][r][cc] = (c0 + r < n && cc < nb) ? pj[i] : 0.0;
    }
    __syncthreads();
    if (tid < 64) {
        const int r = tid & 31;
        double row[CH_NB];
#pragma unroll
        for (int c = 0; c < CH_NB; ++c) row[c] = L11[r][c];
        int bad = 0;
        double my_inv = 1.0, my_piv = 1.0;
#pragma unroll
        for (int j = 0; j < CH_NB; ++j) {
            if (j % 8 == 0 && j >= nb) break;   // uniform: a short block's identity rows need no pivots
            double d = lane_value(row[j], j);
            if (!(d > 0.0) || !isfinite(d)) {   // uniform
                if (!bad) bad = k0 + j + 1;
                d = 1.0;
            }
            double piv, q;
            sqrt_both(d, piv, q);
            if (r == j) {
                my_inv = q;
                my_piv = piv;
            }
            row[j] = r == j ? piv : quotient(row[j], piv, q);
            // entries above the diagonal become meaningless and are never read
#pragma unroll
            for (int c = j + 1; c < CH_NB; ++c) row[c] = fma(-row[j], lane_value(row[j], c), row[c]);
        }
        if (tid < 32) {
            inv[r] = quotient(1.0, my_piv, my_inv);
#pragma unroll
            for (int c = 0; c < CH_NB; ++c) {
                const double v = c <= r ? row[c] : 0.0;
                L11[r][c] = v;
                Lt[c][r] = v;
            }
            if (tid == 0 && blockIdx.x == 0) {
                // the first block column starts the status word
                if (k0 == 0) status[0] = bad;
                else if (bad && status[0] == 0) status[0] = bad;
            }
        }
    }
    __syncthreads();
    if (n <= CH_NB) {   // uniform: the whole matrix, and no other workgroup reads it
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = rq + 8 * i;
            if (r < n && cc < n) A[(size_t)r * n + cc] = L11[r][cc];
        }
        return;
    }
    if (blockIdx.x == 0) {
        if (tid < nb) diag[k0 + tid] = L11[tid][tid];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int c = rq + 8 * i;   // L11[cc][c], c < cc, to row c of the upper triangle
            if (cc < nb && c < cc) A[(size_t)(k0 + c) * n + k0 + cc] = L11[cc][c];
        }
    }
    if (k1 >= n) return;   // uniform
    // the panels: x L11^T = a, a row per lane, one wave per panel
    if (tid < 128 && (tid & 63) < 32) {
        const int w = tid >> 6, r = tid & 31;
        if (w == 0 || ti != tj) {
            double x[CH_NB];
#pragma unroll
            for (int c = 0; c < CH_NB; ++c) x[c] = P[w][r][c];
#pragma unroll
            for (int c = 0; c < CH_NB; ++c) {
                x[c] *= inv[c];
#pragma unroll
                for (int t = c + 1; t < CH_NB; ++t) x[t] = fma(-x[c], Lt[c][t], x[t]);
            }
#pragma unroll
            for (int c = 0; c < CH_NB; ++c) P[w][r][c] = x[c];
            // the tiles of the first column write the panel, transposed
            if (w == 0 && tj == 0 && r0 + r < n) {
#pragma unroll
                for (int c = 0; c < CH_NB; ++c)
                    if (c < nb) A[(size_t)(k0 + c) * n + r0 + r] = x[c];
            }
        }
    }
    __syncthreads();
    const double (*Pj)[CH_NB + 1] = ti == tj ? P[0] : P[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = rq + 8 * i, gi = r0 + r, gj = c0 + cc;
        double s = a22[i];
#pragma unroll
        for (int t = 0; t < CH_NB; ++t) s = fma(-P[0][r][t], Pj[cc][t], s);
        if (gi < n && gj <= gi) A[(size_t)gi * n + gj] = s;
    }
}

// Tile (ti, tj) of the lower triangle from its transpose in the upper one
// (which becomes zero), the diagonal from `diag`.
__global__ __launch_bounds__(256) void chol_finish_kernel(double* __restrict__ A, int n,
                                                          const double* __restrict__ diag) {
    __shared__ double t[32][33];
    int ti = (int)((sqrt(8.0 * blockIdx.x + 1.0) - 1.0) * 0.5);
    while (ti * (ti + 1) / 2 > (int)blockIdx.x) --ti;
    while ((ti + 1) * (ti + 2) / 2 <= (int)blockIdx.x) ++ti;
    const int tj = (int)blockIdx.x - ti * (ti + 1) / 2;
    const int cc = threadIdx.x & 31, rq = threadIdx.x >> 5;
    const int r0 = 32 * ti, c0 = 32 * tj;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = rq + 8 * i;   // upper tile: rows c0 + r, columns r0 + cc
        if (c0 + r < n && r0 + cc < n) t[r][cc] = A[(size_t)(c0 + r) * n + r0 + cc];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = rq + 8 * i, gi = r0 + r, gj = c0 + cc;
        if (ti != tj && c0 + r < n && r0 + cc < n) A[(size_t)(c0 + r) * n + r0 + cc] = 0.0;
        if (gi < n && gj < n) A[(size_t)gi * n + gj] = gj < gi ? t[cc][r] : gj == gi ? diag[gi] : 0.0;
    }
}

int launch_cholesky(svconv_plan* p, double* A, int n) {
    int st = SVCONV_OK;
    double* diag = p->dVec + kVecPivots;   // [n]
    for (int k0 = 0; k0 < n && !st; k0 += CH_NB) {
        const int nt = n - k0 > CH_NB ? (n - k0 - 1) / CH_NB : 0;   // tiles of the rows below the block
        hipLaunchKernelGGL(chol_step_kernel, dim3(nt ? nt * (nt + 1) / 2 : 1), dim3(256), 0, p->stream, A, n, k0, diag,
                           p->dStatus);
        st = hip_status(hipGetLastError(), "chol_step_kernel");
    }
    if (st) return st;
    if (n > CH_NB) {
        const int nt = (n + 31) / 32;
        hipLaunchKernelGGL(chol_finish_kernel, dim3(nt * (nt + 1) / 2), dim3(256), 0, p->stream, A, n, diag);
        st = hip_status(hipGetLastError(), "chol_finish_kernel");
        if (st) return st;
    }
    int bad = 0;
    st = hip_status(hipMemcpyAsync(&bad, p->dStatus, sizeof(int), hipMemcpyDeviceToHost, p->stream),
                    "copy status");
    if (!st) st = hip_status(hipStreamSynchronize(p->stream), "hipStreamSynchronize");
    if (st) return st;
    if (bad) return fail(SVCONV_ENOTSPD, "pivot " + std::to_string(bad - 1) + " is not positive");
    return SVCONV_OK;
}

// x = L^-T L^-1 rhs by blocked substitutions in one workgroup, n <= 1024.
// Wave 0 solves one 32 x 32 triangle after the other, each unknown broadcast
// by v_readlane, while eight helper waves form what the next block takes from
// the unknowns found so far (coalesced loads, thread (hr, hc) for the rows hr and
// hr + 16) and stage its triangle and the 32 x 32 piece that meets the block
// being solved, which wave 0 applies itself: one barrier per block.
// Bound: the serial chain of the triangles, about 100 cycles per unknown.  n =
// 294: 78 us (panels after triangles, every thread a row of its own with 64
// cache lines per load) -> 33 us; n = 735: 227 -> 124 us, in a loop over a factor
// that stays in L2 (306 -> 204 us where each iteration's images displace it).
// With a64, the Newton update is applied at the end: a64 -= x, a32 =
// float(a64), norm = ||x||_2.
constexpr int CS_B = 32, CS_HELPERS = 512, CS_NT = 64 + CS_HELPERS;

__global__ __launch_bounds__(CS_NT) void chol_solve_kernel(const double* __restrict__ L,
                                                           const double* __restrict__ rhs,
                                                           double* __restrict__ x, int n,
                                                           double* __restrict__ a64, float* __restrict__ a32,
                                                           double* __restrict__ norm) {
    // per buffer: the triangle below its diagonal, the reciprocals, the piece
    // and the sums of the block to solve next
    __shared__ double v[kMaxCoefficients], T[2][CS_B][CS_B + 1], piece[2][CS_B][CS_B + 1], part[2][CS_B][CS_B + 1];
    __shared__ double dinv[2][CS_B];
    const int tid = threadIdx.x, nblk = (n + CS_B - 1) / CS_B;
    const int ht = tid - 64, hr = ht >> 5, hc = ht & 31;   // helpers
    // entry (r, c) of L, zero outside
    auto at = [&](int r, int c) {
        const double t = L[(size_t)min(max(r, 0), n - 1) * n + min(max(c, 0), n - 1)];
        return r >= 0 && r < n && c >= 0 && c < n ? t : 0.0;
    };
    // helpers: block kb into `buf`, `known` blocks of unknowns before (after) it
    // summed, the one next to it staged as the piece
    auto prepare = [&](int buf, int kb, bool forward) {
        const int j0 = kb * CS_B;
        double t[2], p[2], s[2] = {0.0, 0.0};
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int r = hr + 16 * q;
            // T[t][j] is what unknown j takes from row t: L[t][j], j < t, or L[j][t], j > t
            t[q] = at(j0 + r, j0 + hc);
            p[q] = forward ? at(j0 + r, j0 - CS_B + hc) : at(j0 + CS_B + r, j0 + hc);
        }
        if (forward) {
#pragma unroll 8
            for (int i = 0; i < kb - 1; ++i) {
                const double y = v[CS_B * i + hc];
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    s[q] = fma(L[(size_t)min(j0 + hr + 16 * q, n - 1) * n + CS_B * i + hc], y, s[q]);
            }
        } else {
#pragma unroll 8
            for (int i = kb + 2; i < nblk; ++i)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int r = CS_B * i + hr + 16 * q;   // v is 0 past n
                    s[q] = fma(L[(size_t)min(r, n - 1) * n + j0 + hc], v[r], s[q]);
                }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int r = hr + 16 * q;
            if (forward) {
                T[buf][r][hc] = hc < r ? t[q] : 0.0;
                piece[buf][r][hc] = p[q];
                part[buf][r][hc] = s[q];
            } else {
                T[buf][hc][r] = hc < r ? t[q] : 0.0;
                piece[buf][hc][r] = p[q];
                part[buf][hc][r] = s[q];
            }
            if (r == hc) dinv[buf][r] = j0 + r < n ? 1.0 / t[q] : 1.0;
        }
    };
    // wave 0: the unknowns of block kb, given those of block `from` next to it
    auto solve = [&](int buf, int kb, int from, bool forward) {
        const int t = tid & 31, half = (tid >> 5) * 16;
        const double inv = dinv[buf][t];
        double s0 = 0.0, s1 = 0.0;
#pragma unroll
        for (int i = 0; i < 16; ++i) s0 += part[buf][t][half + i];
        if (from >= 0 && from < nblk) {
#pragma unroll
            for (int i = 0; i < 16; ++i) s1 = fma(piece[buf][t][half + i], v[CS_B * from + half + i], s1);
        }
        s0 += s1;
        double acc = v[CS_B * kb + t] - (s0 + __shfl_xor(s0, 32));
#pragma unroll
        for (int i = 0; i < CS_B; ++i) {
            const int j = forward ? i : CS_B - 1 - i;
            acc = fma(-T[buf][t][j], lane_value(acc * inv, j), acc);   // 0 for the unknowns already found
        }
        if (tid < 32) v[CS_B * kb + t] = CS_B * kb + t < n ? acc * inv : 0.0;
    };
    for (int i = tid; i < nblk * CS_B; i += CS_NT) v[i] = i < n ? rhs[i] : 0.0;
    __syncthreads();
    if (tid >= 64) prepare(0, 0, true);
    __syncthreads();
    for (int kb = 0; kb < nblk; ++kb) {
        if (tid < 64) solve(kb & 1, kb, kb - 1, true);
        else if (kb + 1 < nblk) prepare((kb + 1) & 1, kb + 1, true);
        else prepare((kb + 1) & 1, kb, false);   // the backward pass starts where this one ends
        __syncthreads();
    }
    for (int q = 0; q < nblk; ++q) {
        const int kb = nblk - 1 - q, buf = (nblk + q) & 1;
        if (tid < 64) solve(buf, kb, kb + 1, false);
        else if (kb > 0) prepare(buf ^ 1, kb - 1, false);
        __syncthreads();
    }
    double ss = 0.0;
    for (int i = tid; i < n; i += CS_NT) {
        const double d = v[i];
        x[i] = d;
        if (a64) {
            const double a = a64[i] - d;
            a64[i] = a;
            a32[i] = (float)a;
            ss += d * d;
        }
    }
    if (!a64) return;   // uniform
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    __syncthreads();
    if ((tid & 63) == 0) v[tid >> 6] = ss;
    __syncthreads();
    if (tid == 0) {
        double t = 0.0;
        for (int w = 0; w < CS_NT / 64; ++w) t += v[w];
        *norm = sqrt(t);
    }
}

int launch_cholesky_solve(svconv_plan* p, const double* L, const double* rhs, double* x, int n, double* a64,
                          float* a32, double* norm) {
    hipLaunchKernelGGL(chol_solve_kernel, dim3(1), dim3(CS_NT), 0, p->stream, L, rhs, x, n, a64, a32, norm);
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

}  // namespace svc
