// Regrouped contraction in float64 on the vector units.
//
// D = sum_m P_m (Kt_m (x) R) - I (Eq. 1 with Eq. 2 regrouped: P_m depends
// only on the output pixel, so the M kernels Kt_m = sum_n a[n][m] B_n carry
// all of the coefficients).  For the Dirac delta basis (Sec. 2) Kt_m is the
// coefficient array itself, Kt_m[u,v] = a[n(u,v)][m], so the taps are read
// straight from a and no per-call table is built.
//
// A thread keeps its column x, and P_m = xh^i yh^j, so the M taps of a kernel
// pixel fold into d_s + 1 taps b_j(x) = sum_i xh^i Kt_(i,j), one per power of
// yh, once for all the rows the thread owns: d_s + 1 products per tap and
// pixel instead of M (3 instead of 6 at second order), plus M - 1 per tap and
// column.  Everything is float64: on this chip a float64 FMA issues at the rate
// of an unpacked float32 one (4 cycles a wave), so what float32 products with
// float64 row sums spent on conversions and additions is saved as well, and D
// is rounded once.  The taps arrive by scalar loads (uniform over the wave),
// requested once the ones before are folded: two sets at once overflow the
// scalar registers at high order (31 x 31, sixth order, 256 x 256: 148 -> 58 us;
// 31 x 31, third order, 2048 x 2048: 705 -> 616 us).
//
// Bound: the float64 FMA rate (248 vector instructions per pixel at 7 x 7,
// second order, 165 of them FMAs, on 86 % of the cycles; 21 x 21: 88 %). 7 x 7
// delta basis, second order, 4846 x 4868: 315 us (float32 FMAs over six terms,
// float64 row sums) -> 182 us, error against float64 4.0e-8 -> 2.5e-8 of D; 21
// x 21, 49 bases, second order, 2048 x 4096: 741 us (float32 matrix cores) ->
// 450 us (482 with two sets of taps); 31 x 31, third order, 2048 x 2048: 1323
// -> 632 us.
//
// Per kernel column du and DR_CH kernel rows (an item), the samples the
// thread's rows need are read from LDS once and widened.  ROWS = 16 rows per
// thread amortise the folding and the windows; where the frame is too small to
// fill the chip with such waves, S waves share the same pixels and take every
// S-th item, and their sums are added through LDS.
#include "internal.hpp"
#include "sep_fold.hpp"

namespace svc {

constexpr int DR_TW = 64;
constexpr int DR_CH = 7;        // kernel rows per window: 7 and 21 rows are whole windows
constexpr int DR_STAGE = 8;     // staging loads in flight per thread

// Workgroups go round-robin over the 8 XCDs; each XCD takes a contiguous run of
// tiles, so that the halo rows and the partly used lines of neighbours meet in
// one L2 (7 x 7: 195.5 -> 189.2 us at 4846 x 4868, 16.4 -> 15.0 us at 1024 x
// 1024; 21 x 21, which reads little per product, is the same).
__device__ __forceinline__ int xcd_tile(int b, int n) {
    const int x = b & 7, q = n >> 3, r = n & 7;
    return x * q + (x < r ? x : r) + (b >> 3);
}

// Where the taps are: TAPS_DELTA: in a itself (float32), tap (m, dv, du) =
// a[(k^2 - 1 - (dv k + du)) M + m] (the delta basis in correlation orientation);
// TAPS_TABLE: taps64[du][dv][m]; TAPS_FORMED: the same table in LDS, formed by
// every workgroup.
enum { TAPS_TABLE = 0, TAPS_DELTA = 1, TAPS_FORMED = 2 };

// Filter entry idx of M k^2 (m, then dv, du): sum_n a[n][m] F_n[dv][du], and its
// place in a table [du][dv][m].
__device__ __forceinline__ double regrouped_tap(const double* __restrict__ F64, const float* __restrict__ a, int N,
                                                int M, int k, int idx, int& at) {
    const int kk = k * k, m = idx / kk, q = idx - m * kk;
    double s = 0.0;
#pragma unroll 8
    for (int n = 0; n < N; ++n) s += (double)a[n * M + m] * F64[(size_t)n * kk + q];
    const int dv = q / k, du = q - dv * k;
    at = (du * k + dv) * M + m;
    return s;
}

// HC: the half-width where it is known at compile time, else 0.
template <int J, int ROWS, int WAVES, int S, int SRC, int HC>
__global__ __launch_bounds__(64 * WAVES) void contract_direct_kernel(DirectArgs a) {
    constexpr int DS = J - 1, M = J * (J + 1) / 2;
    constexpr int NT = 64 * WAVES, TH = ROWS * WAVES / S;
    extern __shared__ float tile[];
    constexpr int CH = HC && 2 * HC + 1 < DR_CH ? 2 * HC + 1 : DR_CH;   // kernel rows of an item
    const int h = HC ? HC : a.h, K = 2 * h + 1;
    const int SC = DR_TW + 2 * h, SR = TH + 2 * h;

    const int tid = threadIdx.x, c = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile_id = xcd_tile(blockIdx.x, gridDim.x);
    const int ty = tile_id / a.tiles_x, tx = tile_id - ty * a.tiles_x;
    const int X0 = tx * DR_TW, Y0 = ty * TH;

    double* formed = reinterpret_cast<double*>(tile + a.taps_at);
    if constexpr (SRC == TAPS_FORMED) {
        for (int i = tid; i < M * K * K; i += NT) {
            int at;
            const double t = regrouped_tap(a.F64, a.coef, a.N, M, K, i, at);
            formed[at] = t;
        }
    }
    // stage R, 0 outside the image: loads from clamped addresses, several rows
    // in flight, masks at the store.  First 64 columns of whole rows (scalar
    // row addresses), then the 2 h columns right of them.
    {
        const int gx = X0 - h + c;
        const unsigned gxc = min(max(gx, 0), a.W - 1);
        const bool inx = gx >= 0 && gx < a.W;
        for (int r0 = wave; r0 < SR; r0 += WAVES * DR_STAGE) {
            float v[DR_STAGE];
#pragma unroll
            for (int b = 0; b < DR_STAGE; ++b) {
                const int gy = min(max(Y0 - h + r0 + WAVES * b, 0), a.H - 1);
                v[b] = (a.X + (size_t)gy * a.W)[gxc];
            }
#pragma unroll
            for (int b = 0; b < DR_STAGE; ++b) {
                const int r = r0 + WAVES * b, gy = Y0 - h + r;
                if (r < SR) tile[r * SC + c] = (inx && gy >= 0 && gy < a.H) ? v[b] : 0.f;
            }
        }
        const int n = SR * 2 * h;
        const float inv = 1.f / (float)(2 * h);
        for (int q0 = tid; q0 < n; q0 += NT * DR_STAGE) {
            float v[DR_STAGE];
            int at[DR_STAGE];
#pragma unroll
            for (int b = 0; b < DR_STAGE; ++b) {
                // q / 2 h: exact, as q < 2^14 and (q + 1/2) / 2 h is 1/124 from an integer at least
                const int q = min(q0 + NT * b, n - 1), r = (int)(((float)q + 0.5f) * inv);
                const int cc = DR_TW + q - r * 2 * h;
                const int gy = Y0 - h + r, gx2 = X0 - h + cc;
                at[b] = r * SC + cc;
                const float s = a.X[(size_t)min(max(gy, 0), a.H - 1) * a.W + min(max(gx2, 0), a.W - 1)];
                v[b] = (gy >= 0 && gy < a.H && gx2 >= 0 && gx2 < a.W) ? s : 0.f;
            }
#pragma unroll
            for (int b = 0; b < DR_STAGE; ++b) tile[at[b]] = v[b];   // past the end: the last sample again
        }
    }
    __syncthreads();

    const int x = X0 + c;
    const double xh = a.sx * x + a.ox;
    double acc[J][ROWS];
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int r = 0; r < ROWS; ++r) acc[j][r] = 0.0;

    // taps of a kernel pixel at a byte offset: uniform, so they arrive by scalar
    // loads (or one LDS read for the whole wave)
    constexpr bool DFB = SRC == TAPS_DELTA;
    typedef typename std::conditional<DFB, float, double>::type tap_t;
    struct Taps { tap_t v[M]; };
    const cptr<char> taps = (cptr<char>)(DFB ? (const void*)a.taps : (const void*)a.taps64);
    auto load_taps = [&](unsigned off) {
        Taps t;
        if constexpr (SRC == TAPS_FORMED) {
            const double* p = formed + off / sizeof(double);
#pragma unroll
            for (int m = 0; m < M; ++m) t.v[m] = p[m];
        } else {
            const cptr<tap_t> p = (cptr<tap_t>)(taps + off);
#pragma unroll
            for (int m = 0; m < M; ++m) t.v[m] = p[m];
        }
        return t;
    };
    // byte offset of (dv, du), and from there to (dv + 1, du)
    constexpr unsigned TB = M * sizeof(tap_t);
    auto offset = [&](int dv, int du) {
        return (unsigned)(DFB ? K * K - 1 - (dv * K + du) : du * K + dv) * TB;
    };
    const unsigned down = DFB ? 0u - (unsigned)K * TB : TB;
    const int group = S == 1 ? wave : wave / S, member = S == 1 ? 0 : wave % S;
    // items in order of du, then dv0; this wave takes items member, member + S, ...
    const unsigned n_ch = (K + CH - 1) / CH, inv_ch = 65536u / n_ch + 1u;
    unsigned item = member;
    int du, dv0;
    auto place = [&]() {
        du = (int)((item * inv_ch) >> 16);   // item / n_ch: exact, as item <= 63 x 9 + 8
        dv0 = (int)(item - du * n_ch) * CH;
    };
    place();
    unsigned off = offset(dv0, min(du, K - 1));
    Taps next = load_taps(off);
#pragma unroll 1
    while (du < K) {
        double s[ROWS + CH - 1];
        const float* col = tile + (group * ROWS + dv0) * SC + c + du;
#pragma unroll
        for (int i = 0; i < ROWS + CH - 1; ++i) s[i] = (double)col[i * SC];
        const int n = K - dv0;   // taps of this item, if fewer than CH
        item += S;
        place();
        const unsigned off_item = offset(dv0, min(du, K - 1));
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            if (i < n) {   // uniform
                // spatial term m = q (q + 1) / 2 + j is xh^(q - j) yh^j
                double b[J];
#pragma unroll
                for (int j = 0; j < J; ++j) {
                    b[j] = (double)next.v[DS * (DS + 1) / 2 + j];
#pragma unroll
                    for (int q = DS - 1; q >= j; --q) b[j] = fma(b[j], xh, (double)next.v[q * (q + 1) / 2 + j]);
                }
                // the taps of the next kernel pixel, once these are folded (two
                // sets do not fit the scalar registers from fourth order on) and
                // before the products of this one
                __builtin_amdgcn_sched_barrier(0);
                off = (i + 1 < CH && i + 1 < n) ? off + down : off_item;
                next = load_taps(off);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int r = 0; r < ROWS; ++r)
#pragma unroll
                    for (int j = 0; j < J; ++j) acc[j][r] = fma(b[j], s[r + i], acc[j][r]);
            }
        }
    }

    // this wave's part of D at its rows
    const int y0 = Y0 + group * ROWS;
    double v[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const double yh = a.sy * (y0 + r) + a.oy;
        v[r] = acc[DS][r];
#pragma unroll
        for (int j = DS - 1; j >= 0; --j) v[r] = fma(v[r], yh, acc[j][r]);
    }
    // with S waves on the same pixels each finishes 1 / S of the rows
    constexpr int RW = ROWS / S;
    if constexpr (S > 1) {
        double* red = reinterpret_cast<double*>(tile);   // [WAVES][ROWS][64], over the samples
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ROWS; ++r) red[(wave * ROWS + r) * 64 + c] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            double t = 0.0;
#pragma unroll
            for (int q = 0; q < S; ++q) t += red[((group * S + q) * ROWS + member * RW + r) * 64 + c];
            v[r] = t;
        }
    }
    if (x >= a.W) return;
    // I at this thread's pixels, all requested at once from clamped addresses
    // (without I, R stands in for the loads)
    const int yo = y0 + member * RW;
    float iv[RW];
    {
        const float* ip = a.I ? a.I : a.X;
#pragma unroll
        for (int r = 0; r < RW; ++r) iv[r] = ip[(size_t)min(yo + r, a.H - 1) * a.W + x];
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const int y = yo + r;
        if (y >= a.H) break;
        a.out[(size_t)y * a.W + x] = (float)(a.I ? v[r] - (double)iv[r] : v[r]);
    }
}

// taps64[du][dv][m] = sum_n a[n][m] F_n[dv][du] (the regrouped filters)
__global__ void regroup64_kernel(const double* __restrict__ F64, const float* __restrict__ a, int N, int M, int k,
                                 double* __restrict__ taps) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= M * k * k) return;
    int at;
    const double t = regrouped_tap(F64, a, N, M, k, idx, at);
    taps[at] = t;
}

int regroup_filters64(const double* F64, const float* a, int N, int M, int k, double* taps, hipStream_t s) {
    hipLaunchKernelGGL(regroup64_kernel, dim3((M * k * k + 127) / 128), dim3(128), 0, s, F64, a, N, M, k, taps);
    return hip_status(hipGetLastError(), "regroup64_kernel");
}

static int direct_tiles(const DirectArgs& a, int th) { return a.tiles_x * ((a.H + th - 1) / th); }

// Few bases on a small kernel and frame: the workgroups form the filters, in at
// most a few rounds of loads each, which saves the launch before (whole calls in
// the default form, 256 x 256: 3 x 3, six bases, second order 12.9 us with it,
// 10.3 without; the dense product takes 10.1).  More rounds only where few
// workgroups repeat them (700 x 760, 7 x 7, 22 bases, second order: 13.8 us with
// the launch, 16.3 without).
constexpr int FORMED_J = 4;   // up to third order

bool direct_forms_taps(int H, int W, int h, int d_s, int N, int cus) {
    const int M = (d_s + 1) * (d_s + 2) / 2, taps = M * (2 * h + 1) * (2 * h + 1);
    const long tiles = (long)((W + DR_TW - 1) / DR_TW) * ((H + 31) / 32);
    const int rounds = (taps + 255) / 256 * ((N + 7) / 8);
    return d_s <= 2 && tiles <= 2L * cus && rounds <= (tiles <= cus && (N <= 8 || taps <= 75) ? 8 : 3);
}

// Whether the table fits LDS beside the largest tile.  Forming it there keeps
// float64 without a table in memory whatever the number of bases (replays, 49
// bases, 21 x 21, 2048 x 4096: second order 625 us, 510 with a table, the dense
// product 6.4 ms; third order 955, 640 and 6.5 ms).
bool direct_can_form_taps(int h, int d_s) {
    const int M = (d_s + 1) * (d_s + 2) / 2, k = 2 * h + 1, rows = 64 + (k + DR_CH - 1) / DR_CH * DR_CH;
    return d_s < FORMED_J && (size_t)rows * (DR_TW + 2 * h) * sizeof(float) + (size_t)k * k * M * sizeof(double) <= 160 * 1024;
}

template <int J, int ROWS, int WAVES, int S, int HC = 0>
static void launch_direct(DirectArgs a, hipStream_t s) {
    constexpr int TH = ROWS * WAVES / S;
    // the rows of the last window are read past the tile's 2 h halo rows, unused
    const int k = 2 * a.h + 1, rows = TH + (k + DR_CH - 1) / DR_CH * DR_CH - 1;
    a.taps_at = (rows * (DR_TW + 2 * a.h) + 1) / 2 * 2;
    size_t lds = (size_t)a.taps_at * sizeof(float) + (a.coef ? (size_t)k * k * J * (J + 1) / 2 * sizeof(double) : 0);
    if (S > 1 && lds < (size_t)WAVES * ROWS * 64 * sizeof(double)) lds = (size_t)WAVES * ROWS * 64 * sizeof(double);
    const dim3 grid(direct_tiles(a, TH)), block(64 * WAVES);
    if constexpr (J <= FORMED_J) {
        if (a.coef) {
            hipLaunchKernelGGL((contract_direct_kernel<J, ROWS, WAVES, S, TAPS_FORMED, HC>), grid, block, lds, s, a);
            return;
        }
    }
    if (a.taps64)
        hipLaunchKernelGGL((contract_direct_kernel<J, ROWS, WAVES, S, TAPS_TABLE, HC>), grid, block, lds, s, a);
    else if (a.taps)
        hipLaunchKernelGGL((contract_direct_kernel<J, ROWS, WAVES, S, TAPS_DELTA, HC>), grid, block, lds, s, a);
}

template <int J>
static void launch_direct_rows(const DirectArgs& a, hipStream_t s) {
    // above third order the totals of 16 rows no longer fit the registers.
    // (8 rows at second order: more waves, but 13 % more instructions per pixel;
    // 21 x 21, 2048 x 4096, with two sets of taps 435 -> 471 us)
    constexpr int ROWS = J <= 4 ? 16 : 8;
    const int cus = a.cus;
    // Small kernels up to second order (3 x 3 and 5 x 5 at third): little work per sample, so the window
    // of exactly their rows and the loops over them unrolled count (1500 x 1400,
    // constant filters: 3 x 3 13.4 -> 7.5 us, 7 x 7 17.1 -> 11.9; 4846 x 4868, 5 x
    // 5, first order 103 -> 77).  Frames of few tiles are better shared by the
    // waves, the more so the more products there are to share (256 x 256, 7 x 7,
    // second order: 6.0 us, 9.6 with these).
    if constexpr (J <= 4) {
        const int products = (2 * a.h + 1) * (2 * a.h + 1) * J;
        if (a.h * J <= 2 || direct_tiles(a, 32) >= (products <= 50 ? cus : products <= 75 ? 2 * cus : 4 * cus)) switch (a.h) {
            case 1: return launch_direct<J, 8, 4, 1, 1>(a, s);
            case 2: return launch_direct<J, 8, 4, 1, 2>(a, s);
            case 3: if constexpr (J <= 3) return launch_direct<J, 8, 4, 1, 3>(a, s); else break;
            case 4: if constexpr (J <= 3) return launch_direct<J, 8, 4, 1, 4>(a, s); else break;
        }
    }
    // whole tiles per wave while they give every CU three workgroups (what the
    // registers hold); then four waves on the same pixels, and eight where there
    // is at most one such tile per CU (21 x 21 at 512 x 512, 256 tiles: 34 us with
    // four on 16 rows, 24 us with eight; at 700 x 760, 528 tiles, 49 us with four,
    // 58 us with eight).  A 3 x 3 or 5 x 5 kernel has no eight items to share.
    // Tiles of half the rows where even those give a CU at most one (256 x 256:
    // 23 -> 20 us).
    if (direct_tiles(a, 4 * ROWS) >= 3 * cus) return launch_direct<J, ROWS, 4, 1>(a, s);
    if (direct_tiles(a, ROWS) > cus || a.h < 3) return launch_direct<J, ROWS, 4, 4>(a, s);
    if constexpr (ROWS == 16) {
        if (direct_tiles(a, 8) <= cus) return launch_direct<J, 8, 8, 8>(a, s);
    }
    launch_direct<J, ROWS, 8, 8>(a, s);
}

int launch_contract_direct(DirectArgs a, hipStream_t s) {
    a.tiles_x = (a.W + DR_TW - 1) / DR_TW;
    if (a.h < 0 || a.h > kMaxHalfWidth || a.H <= 0 || a.W <= 0 || a.cus <= 0 || !!a.taps + !!a.taps64 + !!a.coef != 1 ||
        (a.coef && (!a.F64 || !direct_can_form_taps(a.h, a.d_s))))
        return fail(SVCONV_EUNSUPPORTED, "direct regrouped kernel: bad arguments");
    switch (a.d_s) {
        case 0: launch_direct_rows<1>(a, s); break;
        case 1: launch_direct_rows<2>(a, s); break;
        case 2: launch_direct_rows<3>(a, s); break;
        case 3: launch_direct_rows<4>(a, s); break;
        case 4: launch_direct_rows<5>(a, s); break;
        case 5: launch_direct_rows<6>(a, s); break;
        case 6: launch_direct_rows<7>(a, s); break;
        default: return fail(SVCONV_EUNSUPPORTED, "direct regrouped kernel needs spatial degree <= 6");
    }
    return hip_status(hipGetLastError(), "contract_direct_kernel");
}

}  // namespace svc
