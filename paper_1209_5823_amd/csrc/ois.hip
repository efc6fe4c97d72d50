// Optimal Image Subtraction on isolated stars (Sec. 2: the kernel is
// determined by least squares from isolated stars of the reference):
//   * stamp selection: isolated local maxima of R above a threshold, and the
//     mask of the boxes around them;
//   * the differential background polynomial bg = sum_m b_m P_m of the fit
//     model D = (R (x) K) + bg - I, and its gradient;
//   * the whole-image fit by conjugate gradients on the normal equations,
//     preconditioned by a Cholesky factor (typically that of the stamp normal
//     matrix, which is far cheaper to build than the whole-image one).
#include <cmath>

#include "internal.hpp"

namespace svc {

// ---------------------------------------------------------- stamps ----

// Stamp centres as one bit per pixel: bits[y][x / 32] bit x % 32 is set for a
// strict local maximum with R - sky > threshold, at least `margin` from every
// edge, and no other strict local maximum q in the (2 r_iso + 1)^2 window with
// R(q) - sky >= frac (R(p) - sky).  Every comparison is taken in float64 on
// the float32 values.
//
// Bound: vector and scalar instructions of the staging and of the tests (a wave
// instruction takes 4 cycles), then the one read of R.  A workgroup stages 64
// x 32 pixels and the window's halo in LDS, pixels outside the image as -inf,
// so that a window has the same lane offsets for every candidate.  Pixels above
// the threshold are few: the neighbour tests run only where a ballot finds one,
// and the wave scans a candidate's window together, 64 window pixels a step,
// leaving at the first step that rejects it.  2048 x 4096, 20000 stars, r_iso =
// 10: 650 us as one lane per pixel with its own window loop and 64-bit index
// divisions -> 32 us (40 us with the windows read from L2 instead of LDS, 42 us
// with clamped row addresses in every tile and the neighbours tested one by one).
//
// Windows above CENTRE_WHOLE are scanned in two steps: the part within
// CENTRE_NEAR from LDS, and only for the candidates that it leaves, which are
// then far from each other, all of the window that lies inside the image from
// L2.  In one step the halo of r_iso = 64 takes 123 KiB of LDS (four waves per
// CU) and 15 times the tile, and every scan starts at the far corner: crowded
// fields (sky noise above 0.6 sigma, frac 0.1) at r_iso = 64 took 911 us at 64
// x 64 and 3714 at 2048 x 4096, now 45 and 151 (whole calls).  A frac above 1
// takes the second step alone (1200 x 1600, frac 3, r_iso = 25: 420 us, 600 with both).
// A wave takes the candidates of its rows one after the other, so on frames of
// at most two tiles per CU, which two workgroups of 16 waves fill, 16 waves
// share a tile: the field above at 700 x 900, r_iso = 10 and 24, took 71 and
// 169 us with four waves, 56 and 56 with 16.  Windows above CENTRE_NEAR scanned
// whole do so up to four tiles per CU (1200 x 1600, r_iso = 24: 163 and 74); on
// larger frames the staging is what counts (chip, 20,000 stars: 73 and 80).
constexpr int CENTRE_TX = 64, CENTRE_TY = 32, CENTRE_WHOLE = 24, CENTRE_NEAR = 16, CENTRE_FAR = 4;
constexpr int COUNT_SLOTS = 64, COUNT_STRIDE = 32;   // counters on 128-byte lines of their own

// t[0] strictly larger than each of its neighbours
__device__ __forceinline__ bool strict_local_max(const float* t, int pitch) {
    const float v = t[0];
    const float a0 = t[-pitch - 1], a1 = t[-pitch], a2 = t[-pitch + 1], b0 = t[-1], b2 = t[1];
    const float c0 = t[pitch - 1], c1 = t[pitch], c2 = t[pitch + 1];
    // no short circuit: the loads go out together
    return (v > a0) & (v > a1) & (v > a2) & (v > b0) & (v > b2) & (v > c0) & (v > c1) & (v > c2);
}

// the same at (x, y) of the image, from memory; neighbours outside it do not count
__device__ __forceinline__ bool strict_local_max(const float* __restrict__ R, int H, int W, int x, int y) {
    const float v = R[(size_t)y * W + x];
    const int xl = max(x - 1, 0), xr = min(x + 1, W - 1);
    bool ok = true;
#pragma unroll
    for (int d = -1; d <= 1; ++d) {
        const float* row = R + (size_t)min(max(y + d, 0), H - 1) * W;
        const float l = row[xl], c = row[x], r = row[xr];
        const bool in = y + d >= 0 && y + d < H;
        ok &= !in | (x == 0) | (v > l);
        ok &= !in | (x == W - 1) | (v > r);
        if (d) ok &= !in | (v > c);
    }
    return ok;
}

// FAR: the window reaches past the staged halo
template <int NW, bool FAR>
__global__ __launch_bounds__(64 * NW) void centre_kernel(const float* __restrict__ R, int H, int W, double sky,
                                                     double thr, double frac, int r_iso, int margin,
                                                     unsigned* __restrict__ bits, int wpr, int tiles_x,
                                                     int* __restrict__ count) {
    constexpr int CENTRE_STAGE = NW == 4 ? 14 : 5;   // rows requested together
    extern __shared__ float tile[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // consecutive tiles on one XCD (workgroups go round the 8 XCDs), whose L2 then serves the halos
    const int xcd = blockIdx.x & 7, q8 = gridDim.x >> 3, r8 = gridDim.x & 7;
    const int t = xcd * q8 + min(xcd, r8) + (blockIdx.x >> 3);
    const int ty = t / tiles_x, tx = t - ty * tiles_x;
    const int x0 = tx * CENTRE_TX, y0 = ty * CENTRE_TY;
    // the counters are added to by the next kernel on the stream
    if (blockIdx.x == 0 && threadIdx.x < COUNT_SLOTS) count[threadIdx.x * COUNT_STRIDE] = 0;
    const int r_near = FAR ? CENTRE_NEAR : r_iso, halo = r_near + 1, pitch = CENTRE_TX + 2 * halo, rows = CENTRE_TY + 2 * halo;
    // columns 0..63 of each row by a whole wave, the others by half a wave per row
    const bool inner = x0 >= halo && x0 + CENTRE_TX + halo <= W && y0 >= halo && y0 + CENTRE_TY + halo <= H;
    auto stage = [&](int r0, int r_step, int col) {
        float v[CENTRE_STAGE];
        float* dst = tile + r0 * pitch + col;
        if (inner) {
            // no clamps or masks: the row steps are one scalar add each
            const int last = rows - 1 - r0;   // rows past the tile read its last row
            const float* src = R + (size_t)(y0 - halo + r0) * W + (x0 - halo + min(col, pitch - 1));
#pragma unroll
            for (int b = 0; b < CENTRE_STAGE; ++b) v[b] = src[(long)min(r_step * b, last) * W];
        } else {
            const int x = x0 - halo + col;
            const bool inx = x >= 0 && x < W;
            const float* src = R + min(max(x, 0), W - 1);
#pragma unroll
            for (int b = 0; b < CENTRE_STAGE; ++b) {
                const int y = y0 - halo + r0 + r_step * b;
                const float r = src[(size_t)min(max(y, 0), H - 1) * W];
                v[b] = (inx && y >= 0 && y < H) ? r : -INFINITY;
            }
        }
        if (col < pitch) {
#pragma unroll
            for (int b = 0; b < CENTRE_STAGE; ++b)
                if (r0 + r_step * b < rows) dst[r_step * b * pitch] = v[b];
        }
    };
    for (int r0 = wave; r0 < rows; r0 += NW * CENTRE_STAGE) stage(r0, NW, lane);
    for (int c0 = 64; c0 < pitch; c0 += 32)
        for (int r0 = 2 * wave + (lane >> 5); r0 < rows; r0 += 2 * NW * CENTRE_STAGE)
            stage(r0, 2 * NW, c0 + (lane & 31));
    __syncthreads();
    // this lane's first pixel of a window, and the step to its next (64 on)
    const int ww = 2 * r_near + 1;
    const int col_first = lane % ww, row_first = lane / ww, row_step = 64 / ww, col_step = 64 - row_step * ww;
    const int x = x0 + lane;
    const bool inx = x < W && x >= margin && x <= W - 1 - margin;
    constexpr int ROWS = CENTRE_TY / NW;
    constexpr bool CLIP = NW != 4 || FAR;
    const float* mine = tile + (wave * ROWS + halo) * pitch + lane + halo;
    float v[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) v[r] = mine[r * pitch];
    unsigned out = 0;   // lane 2 r + half: that half of row r's bits
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        const int y = y0 + wave * ROWS + r;
        const bool above = inx && y >= margin && y <= H - 1 - margin && (double)v[r] - sky > thr;
        unsigned long long found = 0;
        if (__any(above)) {
            const float* here = mine + r * pitch;
            found = __ballot(above && strict_local_max(here, pitch));
            // isolation: the wave scans the window, on small frames its rows inside the
            // image, one candidate at a time (a neighbour of a strict maximum is none)
            // a frac above 1 leaves most of them to the whole window
            const int up = CLIP ? min(r_near, y) : r_near, total = CLIP ? (up + min(r_near, H - 1 - y) + 1) * ww : ww * ww;
            for (unsigned long long todo = r_iso > 1 && !(FAR && frac > 1.) ? found : 0; todo; todo &= todo - 1) {
                const int c = __ffsll(todo) - 1;
                const float* centre = here - lane + c;
                const double lim = frac * ((double)centre[0] - sky);
                const float* corner = centre - up * pitch - r_near;
                int row = row_first, col = col_first;
                for (int t = lane; t - lane < total; t += 64) {
                    const float* q = corner + row * pitch + col;
                    const bool bright = t < total && (double)*q - sky >= lim && q != centre;
                    if (__any(bright) && __any(bright && strict_local_max(q, pitch))) {
                        found &= ~(1ull << c);
                        break;
                    }
                    row += row_step;
                    col += col_step;
                    if (col >= ww) {
                        col -= ww;
                        ++row;
                    }
                }
            }
            // the whole window of those left, as far as it lies inside the image
            if (FAR) {
                for (unsigned long long todo = found; todo; todo &= todo - 1) {
                    const int c = __ffsll(todo) - 1, cx = x0 + c;
                    const double lim = frac * ((double)here[c - lane] - sky);
                    const int wx = max(cx - r_iso, 0), wy = max(y - r_iso, 0);
                    const int nx = min(cx + r_iso, W - 1) - wx + 1, n = nx * (min(y + r_iso, H - 1) - wy + 1);
                    const float inv = 1.f / (float)nx;
                    for (int t0 = 0; t0 < n; t0 += 64 * CENTRE_FAR) {
                        int qx[CENTRE_FAR], qy[CENTRE_FAR];
                        float q[CENTRE_FAR];
#pragma unroll
                        for (int b = 0; b < CENTRE_FAR; ++b) {
                            // t / nx: exact, as t < 129^2 + 256 and (t + 1/2) / nx is 1/258 from an integer at least
                            const int t = min(t0 + 64 * b + lane, n - 1), row = (int)(((float)t + 0.5f) * inv);
                            qy[b] = wy + row;
                            qx[b] = wx + t - row * nx;
                            q[b] = R[(size_t)qy[b] * W + qx[b]];
                        }
                        bool bright = false;
#pragma unroll
                        for (int b = 0; b < CENTRE_FAR; ++b)
                            if ((double)q[b] - sky >= lim && !(qx[b] == cx && qy[b] == y))
                                bright |= strict_local_max(R, H, W, qx[b], qy[b]);
                        if (__any(bright)) {
                            found &= ~(1ull << c);
                            break;
                        }
                    }
                }
            }
        }
        if ((lane >> 1) == r) out = (unsigned)(found >> (32 * (lane & 1)));
    }
    const int y = y0 + wave * ROWS + (lane >> 1), word = tx * 2 + (lane & 1);
    if (lane < 2 * ROWS && y < H && word < wpr) bits[(size_t)y * wpr + word] = out;
}

// mask = union of the (2 s + 1)^2 boxes around the centres, s <= 64, and the
// number of centres.  On the bits the box is an OR of 2 s + 1 words down a
// column and shifts along the row, so a workgroup of 32 words x 8 rows reads
// its words (cached: 1 bit per pixel) and writes 8 KB of mask bytes, the
// bound.  2048 x 4096, s = 10: 117 us as two passes over bytes, plus 24 us for
// the count -> 8 us.
constexpr int STAMP_WORDS = 32, STAMP_ROWS = 8, STAMP_HALO = 2, STAMP_STAGE = 4;   // 2 words >= 64 columns each side
constexpr int STAMP_COLS = STAMP_WORDS + 2 * STAMP_HALO;

// OR of the bits of `cur` with those up to r <= 32 columns to either side
__device__ __forceinline__ unsigned dilate_word(unsigned prev, unsigned cur, unsigned next, int r) {
    unsigned long long up = ((unsigned long long)cur << 32) | prev;    // towards higher columns
    unsigned long long dn = ((unsigned long long)next << 32) | cur;    // towards lower columns
    for (int done = 0; done < r;) {
        const int step = min(done + 1, r - done);
        up |= up << step;
        dn |= dn >> step;
        done += step;
    }
    return (unsigned)(up >> 32) | (unsigned)dn;
}

__global__ __launch_bounds__(256) void stamp_kernel(const unsigned* __restrict__ bits, int H, int W, int wpr, int s,
                                                    int tiles_x, unsigned char* __restrict__ mask, int* __restrict__ count) {
    __shared__ unsigned in[STAMP_ROWS + 128][STAMP_COLS];   // s <= 64 rows above and below
    __shared__ unsigned col[STAMP_ROWS][STAMP_COLS], row1[STAMP_ROWS][STAMP_COLS], row2[STAMP_ROWS][STAMP_WORDS];
    __shared__ int red[4];
    const int ty = blockIdx.x / tiles_x;
    const int w0 = (blockIdx.x - ty * tiles_x) * STAMP_WORDS, y0 = ty * STAMP_ROWS;
    int n = 0;
    const int in_words = (STAMP_ROWS + 2 * s) * STAMP_COLS;
    for (int i0 = threadIdx.x; i0 < in_words; i0 += 256 * STAMP_STAGE) {
        unsigned v[STAMP_STAGE];
#pragma unroll
        for (int b = 0; b < STAMP_STAGE; ++b) {
            const int i = i0 + 256 * b, r = i / STAMP_COLS;
            const int y = y0 - s + r, w = w0 - STAMP_HALO + i - r * STAMP_COLS;
            const unsigned word = bits[(size_t)min(max(y, 0), H - 1) * wpr + min(max(w, 0), wpr - 1)];
            v[b] = (y >= 0 && y < H && w >= 0 && w < wpr) ? word : 0;
        }
#pragma unroll
        for (int b = 0; b < STAMP_STAGE; ++b) {
            const int i = i0 + 256 * b, r = i / STAMP_COLS, c = i - r * STAMP_COLS;
            if (i >= in_words) break;
            in[r][c] = v[b];
            if (r >= s && r < s + STAMP_ROWS && c >= STAMP_HALO && c < STAMP_HALO + STAMP_WORDS) n += __popc(v[b]);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < STAMP_ROWS * STAMP_COLS; i += 256) {
        const int r = i / STAMP_COLS, c = i - r * STAMP_COLS;
        unsigned any = 0;
#pragma unroll 8
        for (int d = 0; d <= 2 * s; ++d) any |= in[r + d][c];
        col[r][c] = any;
    }
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        const int t = red[0] + red[1] + red[2] + red[3];
        // one counter for all workgroups took 10 us of same-address atomics
        if (t) atomicAdd(count + (blockIdx.x % COUNT_SLOTS) * COUNT_STRIDE, t);
    }
    // the row dilation in two steps of at most 32 columns
    const int s1 = min(s, 32), s2 = s - s1;
    for (int i = threadIdx.x; i < STAMP_ROWS * STAMP_COLS; i += 256) {
        const int r = i / STAMP_COLS, c = i - r * STAMP_COLS;
        row1[r][c] = dilate_word(c > 0 ? col[r][c - 1] : 0, col[r][c], c + 1 < STAMP_COLS ? col[r][c + 1] : 0, s1);
    }
    __syncthreads();
    {
        const int r = threadIdx.x / STAMP_WORDS, c = threadIdx.x % STAMP_WORDS;   // 8 x 32 = 256 threads
        const unsigned* q = &row1[r][c + STAMP_HALO];
        row2[r][c] = dilate_word(q[-1], q[0], q[1], s2);
    }
    __syncthreads();
    // bits to bytes: 16 at a time where rows start on 16 bytes, else one per lane
    const int x0 = w0 * 32, cols = min(STAMP_WORDS * 32, W - x0), rows = min(STAMP_ROWS, H - y0);
    if ((W & 15) == 0 && ((size_t)mask & 15) == 0) {
        for (int i = threadIdx.x; i < STAMP_ROWS * STAMP_WORDS * 2; i += 256) {
            const int r = i / (STAMP_WORDS * 2), q = i % (STAMP_WORDS * 2);
            if (r < rows && 16 * q < cols) {
                const unsigned b = (row2[r][q >> 1] >> (16 * (q & 1))) & 0xffffu;
                auto bytes4 = [](unsigned v) { return (v * 0x00204081u) & 0x01010101u; };   // bit i -> byte i
                const uint4 o = {bytes4(b & 15), bytes4((b >> 4) & 15), bytes4((b >> 8) & 15), bytes4(b >> 12)};
                *reinterpret_cast<uint4*>(mask + (size_t)(y0 + r) * W + x0 + 16 * q) = o;
            }
        }
    } else {
        for (int r = 0; r < rows; ++r)
            for (int c = threadIdx.x; c < cols; c += 256)
                mask[(size_t)(y0 + r) * W + x0 + c] = (row2[r][c >> 5] >> (c & 31)) & 1u;
    }
}

// ------------------------------------------------------ background ----

__device__ __forceinline__ double ipow_d(double x, int e) {
    double r = 1.0;
    for (int t = 0; t < e; ++t) r *= x;
    return r;
}

// D += sum_m b_m P_m, P_m = xh^i yh^j in the order t = 0..d_s, i = t..0 (Eq. 3)
__global__ void add_background_kernel(float* __restrict__ D, const float* __restrict__ b, int H,
                                      int W, int d_s, double sx, double ox, double sy, double oy) {
    const size_t n = (size_t)H * W;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const int y = (int)(i / W), x = (int)(i - (size_t)y * W);
        const double xh = sx * x + ox, yh = sy * y + oy;
        double bg = 0.0;
        int m = 0;
        for (int t = 0; t <= d_s; ++t)
            for (int e = t; e >= 0; --e) bg += (double)b[m++] * ipow_d(xh, e) * ipow_d(yh, t - e);
        D[i] = (float)((double)D[i] + bg);
    }
}

constexpr int BG_BLOCKS = 64;

// part[block][m] = sum over the block's pixels of G P_m
__global__ __launch_bounds__(256) void bg_grad_kernel(const float* __restrict__ G, int H, int W,
                                                      int d_s, double sx, double ox, double sy,
                                                      double oy, double* __restrict__ part) {
    const int M = (d_s + 1) * (d_s + 2) / 2;
    double s[kMaxSpatialTerms];
#pragma unroll
    for (int m = 0; m < kMaxSpatialTerms; ++m) s[m] = 0.0;
    const size_t n = (size_t)H * W;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x) {
        const float g = G[i];
        if (g == 0.f) continue;
        const int y = (int)(i / W), x = (int)(i - (size_t)y * W);
        const double xh = sx * x + ox, yh = sy * y + oy;
        int m = 0;
#pragma unroll
        for (int t = 0; t <= kMaxSpatialDegree; ++t)
#pragma unroll
            for (int e = t; e >= 0; --e) {
                if (t <= d_s) s[m] += (double)g * ipow_d(xh, e) * ipow_d(yh, t - e);
                ++m;
            }
    }
    __shared__ double red[256];
    // terms are numbered per degree, so term m of degree d_s sits at the same
    // index in the full (degree kMaxSpatialDegree) numbering
#pragma unroll
    for (int m = 0; m < kMaxSpatialTerms; ++m) {
        if (m < M) {   // uniform over the workgroup
            red[threadIdx.x] = s[m];
            __syncthreads();
            for (int o = 128; o > 0; o >>= 1) {
                if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
                __syncthreads();
            }
            if (threadIdx.x == 0) part[blockIdx.x * M + m] = red[0];
            __syncthreads();
        }
    }
}

__global__ void bg_grad_final(const double* __restrict__ part, int M, double* __restrict__ gb) {
    const int m = threadIdx.x;
    if (m >= M) return;
    double s = 0.0;
    for (int b = 0; b < BG_BLOCKS; ++b) s += part[b * M + m];
    gb[m] = s;
}

static void frame_coords(const svconv_plan* p, double& sx, double& ox, double& sy, double& oy) {
    sx = ox = sy = oy = 0.0;
    if (p->Wf > 1) { sx = 2.0 / (p->Wf - 1); ox = sx * p->x0 - 1.0; }
    if (p->Hf > 1) { sy = 2.0 / (p->Hf - 1); oy = sy * p->y0 - 1.0; }
}

int launch_add_background(svconv_plan* p, const float* b, float* D) {
    double sx, ox, sy, oy;
    frame_coords(p, sx, ox, sy, oy);
    hipLaunchKernelGGL(add_background_kernel, dim3(2048), dim3(256), 0, p->stream, D, b, p->H, p->W,
                       p->d_s, sx, ox, sy, oy);
    return hip_status(hipGetLastError(), "add_background_kernel");
}

int launch_bg_grad(svconv_plan* p, const float* G, double* gb) {
    double sx, ox, sy, oy;
    frame_coords(p, sx, ox, sy, oy);
    hipLaunchKernelGGL(bg_grad_kernel, dim3(BG_BLOCKS), dim3(256), 0, p->stream, G, p->H, p->W,
                       p->d_s, sx, ox, sy, oy, p->dRed);
    int st = hip_status(hipGetLastError(), "bg_grad_kernel");
    if (st) return st;
    hipLaunchKernelGGL(bg_grad_final, dim3(1), dim3(64), 0, p->stream, p->dRed, p->M, gb);
    return hip_status(hipGetLastError(), "bg_grad_final");
}

// ------------------------------------------- preconditioned CG ----

// Scalars of the iteration, in the plan's vector scratch after the vectors.
enum { CG_RZ = 0, CG_RR = 1 };

// r = -g / 2 (g = dL/da = 2 J^T mask (J a - I)), so r = J^T mask (I - J a)
__global__ void cg_init_kernel(const double* __restrict__ g, double* __restrict__ r, int n) {
    for (int i = threadIdx.x; i < n; i += blockDim.x) r[i] = -0.5 * g[i];
}

__device__ double block_dot(const double* __restrict__ u, const double* __restrict__ v, int n,
                            double* red) {
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) s += u[i] * v[i];
    red[threadIdx.x] = s;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    const double out = red[0];
    __syncthreads();
    return out;
}

// first direction: p = z, rz = r.z
__global__ __launch_bounds__(1024) void cg_start_kernel(const double* __restrict__ r,
                                                        const double* __restrict__ z,
                                                        double* __restrict__ pv, int n,
                                                        double* __restrict__ sc) {
    __shared__ double red[1024];
    const double rz = block_dot(r, z, n, red);
    for (int i = threadIdx.x; i < n; i += 1024) pv[i] = z[i];
    if (threadIdx.x == 0) sc[CG_RZ] = rz;
}

// q2 = 2 A p (from the adjoint of the masked loss); alpha = rz / (p.A p);
// a += alpha p; r -= alpha A p; a32 = float(a); rr = r.r
__global__ __launch_bounds__(1024) void cg_step_kernel(const double* __restrict__ pv,
                                                       const double* __restrict__ q2,
                                                       double* __restrict__ a64,
                                                       float* __restrict__ a32,
                                                       double* __restrict__ r, int n,
                                                       double* __restrict__ sc) {
    __shared__ double red[1024];
    const double pq = 0.5 * block_dot(pv, q2, n, red);
    const double alpha = (pq > 0.0 && isfinite(pq)) ? sc[CG_RZ] / pq : 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) {
        const double v = a64[i] + alpha * pv[i];
        a64[i] = v;
        a32[i] = (float)v;
        r[i] -= alpha * 0.5 * q2[i];
    }
    __syncthreads();
    const double rr = block_dot(r, r, n, red);
    if (threadIdx.x == 0) sc[CG_RR] = sqrt(rr);
}

// beta = r.z / rz; p = z + beta p; rz = r.z
__global__ __launch_bounds__(1024) void cg_direction_kernel(const double* __restrict__ r,
                                                            const double* __restrict__ z,
                                                            double* __restrict__ pv, int n,
                                                            double* __restrict__ sc) {
    __shared__ double red[1024];
    const double rz_new = block_dot(r, z, n, red);
    const double rz = sc[CG_RZ];
    const double beta = (rz > 0.0 && isfinite(rz_new)) ? rz_new / rz : 0.0;
    for (int i = threadIdx.x; i < n; i += 1024) pv[i] = z[i] + beta * pv[i];
    if (threadIdx.x == 0) sc[CG_RZ] = rz_new;
}

__global__ void to_float_kernel(const double* __restrict__ v, float* __restrict__ out, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = (float)v[i];
}

// g = dL/d(a, b) of L = sum_mask D^2 for the D already in `D`, into g[n]
static int loss_gradient(svconv_plan* p, const float* R, float* D, const unsigned char* mask,
                         double* g) {
    int st = launch_loss_grad(p, D, mask, p->dGrad, nullptr);
    if (!st) st = launch_adjoint_a(p, R, p->dGrad, g);
    if (!st && p->bg) st = launch_bg_grad(p, p->dGrad, g + (size_t)p->N * p->M);
    return st;
}

}  // namespace svc

using namespace svc;

extern "C" {

int svconv_stamp_mask(svconv_plan* p, const float* R, double sky, double threshold, double frac,
                      int r_iso, int margin, int stamp_half, unsigned char* mask, int* n_centres) {
    if (!p || !R || !mask) return fail(SVCONV_EINVAL, "NULL argument");
    if (!std::isfinite(sky) || !std::isfinite(threshold)) return fail(SVCONV_EINVAL, "sky and threshold must be finite");
    if (!(frac > 0.0) || !std::isfinite(frac)) return fail(SVCONV_EINVAL, "frac must be positive");
    if (r_iso < 1 || r_iso > 64) return fail(SVCONV_EINVAL, "r_iso must be in [1, 64]");
    if (stamp_half < 0 || stamp_half > 64) return fail(SVCONV_EINVAL, "stamp_half must be in [0, 64]");
    if (margin < 0) return fail(SVCONV_EINVAL, "margin < 0");
    // one bit per pixel, rows of whole 32-bit words: at most the 4 H W bytes of dGrad
    unsigned* bits = reinterpret_cast<unsigned*>(p->dGrad);
    const int wpr = (p->W + 31) / 32;
    int* count = reinterpret_cast<int*>(p->dRed);
    const int cx = (p->W + CENTRE_TX - 1) / CENTRE_TX, cy = (p->H + CENTRE_TY - 1) / CENTRE_TY;
    const int halo = (r_iso > CENTRE_WHOLE ? CENTRE_NEAR : r_iso) + 1;
    const size_t lds = (size_t)(CENTRE_TX + 2 * halo) * (CENTRE_TY + 2 * halo) * sizeof(float);   // <= 37 KB
    const bool far = r_iso > CENTRE_WHOLE;
    const bool few = (long)cx * cy <= (r_iso > CENTRE_NEAR && !far ? 4L : 2L) * p->cus;
    auto kernel = few ? (far ? centre_kernel<16, true> : centre_kernel<16, false>)
                      : (far ? centre_kernel<4, true> : centre_kernel<4, false>);
    hipLaunchKernelGGL(kernel, dim3((unsigned)cx * cy), dim3(few ? 1024 : 256), lds, p->stream, R, p->H, p->W, sky,
                       threshold, frac, r_iso, margin, bits, wpr, cx, count);
    int st = hip_status(hipGetLastError(), "centre_kernel");
    if (st) return st;
    const int sx = (wpr + STAMP_WORDS - 1) / STAMP_WORDS, sy = (p->H + STAMP_ROWS - 1) / STAMP_ROWS;
    hipLaunchKernelGGL(stamp_kernel, dim3((unsigned)sx * sy), dim3(256), 0, p->stream, bits, p->H, p->W, wpr,
                       stamp_half, sx, mask, count);
    st = hip_status(hipGetLastError(), "stamp_kernel");
    if (st || !n_centres) return st;
    int parts[COUNT_SLOTS * COUNT_STRIDE], total = 0;
    st = hip_status(hipMemcpyAsync(parts, count, sizeof(parts), hipMemcpyDeviceToHost, p->stream), "copy count");
    if (!st) st = hip_status(hipStreamSynchronize(p->stream), "hipStreamSynchronize");
    if (st) return st;
    for (int i = 0; i < COUNT_SLOTS; ++i) total += parts[i * COUNT_STRIDE];
    *n_centres = total;
    return SVCONV_OK;
}

int svconv_plan_set_background(svconv_plan* p, int enable) {
    if (!p) return fail(SVCONV_EINVAL, "plan is NULL");
    if (enable != 0 && enable != 1) return fail(SVCONV_EINVAL, "enable must be 0 or 1");
    if (enable && (p->N + 1 > kMaxFilters || (p->N + 1) * p->M > kMaxCoefficients))
        return fail(SVCONV_EUNSUPPORTED, "background needs N + 1 <= 64 and (N + 1) M <= 1024");
    p->bg = enable;
    return SVCONV_OK;
}

int svconv_add_background(svconv_plan* p, const float* b, float* D) {
    if (!p || !b || !D) return fail(SVCONV_EINVAL, "NULL argument");
    return launch_add_background(p, b, D);
}

int svconv_pcg_fit(svconv_plan* p, const float* R, const float* I, const unsigned char* mask,
                   const double* L, int iters, double* a64, float* a32, float* D,
                   double* host_residuals) {
    if (!p || !R || !I || !L || !a64 || !a32 || !D) return fail(SVCONV_EINVAL, "NULL argument");
    if ((const void*)D == (const void*)R || (const void*)D == (const void*)I)
        return fail(SVCONV_EINVAL, "D aliases R or I");
    if (iters < 0 || iters > 10000) return fail(SVCONV_EINVAL, "iters must be in [0, 10000]");
    const int NK = p->N * p->M;
    const int n = NK + p->bg * p->M;
    double* r = p->dVec;
    double* z = r + n;
    double* pv = z + n;
    double* q = pv + n;
    double* sc = q + n;                                    // 8 scalars
    float* p32 = reinterpret_cast<float*>(sc + 8);         // n floats
    const dim3 vec_grid((n + 255) / 256);
    // r = J^T mask (I - J a), z = M^-1 r, p = z
    hipLaunchKernelGGL(to_float_kernel, vec_grid, dim3(256), 0, p->stream, a64, a32, n);
    int st = hip_status(hipGetLastError(), "to_float_kernel");
    if (!st) st = run_forward(p, R, I, a32, D);
    if (!st && p->bg) st = launch_add_background(p, a32 + NK, D);
    if (!st) st = loss_gradient(p, R, D, mask, q);
    if (!st) {
        hipLaunchKernelGGL(cg_init_kernel, dim3(1), dim3(1024), 0, p->stream, q, r, n);
        st = hip_status(hipGetLastError(), "cg_init_kernel");
    }
    if (!st) st = launch_cholesky_solve(p, L, r, z, n);
    if (!st) {
        hipLaunchKernelGGL(cg_start_kernel, dim3(1), dim3(1024), 0, p->stream, r, z, pv, n, sc);
        st = hip_status(hipGetLastError(), "cg_start_kernel");
    }
    for (int it = 0; it < iters && !st; ++it) {
        // q = 2 J^T mask J p: forward of the direction without I, then the
        // adjoint of the masked loss at that image
        hipLaunchKernelGGL(to_float_kernel, vec_grid, dim3(256), 0, p->stream, pv, p32, n);
        st = hip_status(hipGetLastError(), "to_float_kernel");
        if (!st) st = run_forward(p, R, nullptr, p32, D);
        if (!st && p->bg) st = launch_add_background(p, p32 + NK, D);
        if (!st) st = loss_gradient(p, R, D, mask, q);
        if (!st) {
            hipLaunchKernelGGL(cg_step_kernel, dim3(1), dim3(1024), 0, p->stream, pv, q, a64, a32,
                               r, n, sc);
            st = hip_status(hipGetLastError(), "cg_step_kernel");
        }
        if (!st && host_residuals)
            st = hip_status(hipMemcpyAsync(host_residuals + it, sc + CG_RR, sizeof(double),
                                           hipMemcpyDeviceToHost, p->stream), "copy residual");
        if (!st) st = launch_cholesky_solve(p, L, r, z, n);
        if (!st) {
            hipLaunchKernelGGL(cg_direction_kernel, dim3(1), dim3(1024), 0, p->stream, r, z, pv, n,
                               sc);
            st = hip_status(hipGetLastError(), "cg_direction_kernel");
        }
    }
    // D at the final coefficients
    if (!st) st = run_forward(p, R, I, a32, D);
    if (!st && p->bg) st = launch_add_background(p, a32 + NK, D);
    if (!st && host_residuals) st = hip_status(hipStreamSynchronize(p->stream), "hipStreamSynchronize");
    return st;
}

}  // extern "C"
