// Noise residuals W(I) = I - F(I) (Sec. 2, before Eq. (2)) with the wavelet denoiser
// the paper cites, on the device.
//
//   k_dwt_fwd   one level of the periodic orthonormal 2-D wavelet transform with the
//               8-tap Daubechies filter: an LDS tile of the input (with the filter's
//               reach), the horizontal lowpass/highpass at even offsets, then the
//               vertical ones; the approximation goes to a plane of its own, the three
//               detail subbands to their quadrants of the coefficient plane.  Level 1
//               reads the caller's image and extends it by mirroring past its last row
//               and column (to a multiple of 16 on each side).
//   k_dwt_inv   one level of the Wiener step and the inverse transform.  Per detail
//               subband: the windowed means of c^2 over 3x3, 5x5, 7x7 and 9x9 (zero
//               outside the subband), the smallest minus s0^2 clipped at zero as the
//               signal variance v, and the part the Wiener estimate removes,
//               c s0^2 / (v + s0^2).  From those and the approximation (zero at the
//               coarsest level: the residual keeps none of it) the adjoint transform
//               (periodic); level 1 writes the cropped residual.
//
// All arithmetic is fp32.  Every kernel is a streaming pass whose outputs are written once.
// The forward reads its input tile and halo once; a wave of the inverse reads the 8 halo
// rows of its run of coefficient rows itself (17 rows for 9 results in tiles of 64 rows, 13
// for 5 in tiles of 32; the neighbouring run's waves leave them in cache).
#include <type_traits>

#include "kernels.hpp"

namespace prnu {

namespace {

// Daubechies' orthonormal 8-tap lowpass filter (4 vanishing moments, minimum phase),
// sum sqrt(2); the highpass is its quadrature mirror g[k] = (-1)^k h[7 - k].
__constant__ float kH[8] = {0.2303778133088964f,  0.7148465705529154f,  0.6308807679298587f,
                            -0.0279837694168599f, -0.1870348117190931f, 0.0308413818355607f,
                            0.0328830116668852f,  -0.0105974017850690f};
__constant__ float kG[8] = {-0.0105974017850690f, -0.0328830116668852f, 0.0308413818355607f,
                            0.1870348117190931f,  -0.0279837694168599f, -0.6308807679298587f,
                            0.7148465705529154f,  -0.2303778133088964f};

// i mod n in [0, n).  The tiles reach at most one period past either end except on the
// smallest levels, so the division is the rare path.
__device__ __forceinline__ int wrap(int i, int n) {
  if (i >= 0 && i < n) return i;
  if (i >= n && i < 2 * n) return i - n;
  if (i < 0 && i >= -n) return i + n;
  i %= n;
  return i < 0 ? i + n : i;
}

// ---------------------------------------------------------------------------
// Forward level.  Output tile: FY rows x FX columns of each subband.  512 threads: the
// deep levels' few tiles are bound by the length of a thread's work, one call of 3 images
// of 333 x 501 6 us shorter than on 256, and the large levels are no slower.

constexpr int FY = 16, FX = 32, FT = 512;
constexpr int FIY = 2 * FY + 6, FIX = 2 * FX + 6;  // input tile with the filter's reach

// in: level input plane of rows x cols (row stride in_rs, image stride in_is); at level 1
// the caller's M x N image, extended by mirroring to rows x cols.  ll: approximation
// plane (rows/2 x cols/2, stride ll_rs, image stride ll_is) or null.  det: coefficient
// plane of the image (stride det_rs, image stride det_is); the level's details go to its
// quadrants: (0, cols/2) horizontal high, (rows/2, 0) vertical high, (rows/2, cols/2) both.
__global__ __launch_bounds__(FT) void k_dwt_fwd(const float* __restrict__ in, int64_t in_is, int64_t in_rs, int rows,
                                                int cols, int M, int N, float* __restrict__ ll, int64_t ll_is,
                                                int64_t ll_rs, float* __restrict__ det, int64_t det_is,
                                                int64_t det_rs) {
  __shared__ float tile[FIY][FIX + 1];
  __shared__ float lo[FIY][FX + 1], hi[FIY][FX + 1];
  const int img = blockIdx.z;
  const int n0 = blockIdx.y * FY, m0 = blockIdx.x * FX;
  const float* src = in + (int64_t)img * in_is;
  {
    // every load of the tile issued before the first LDS store
    constexpr int NL = (FIY * FIX + FT - 1) / FT;
    float v[NL];
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int i = threadIdx.x + k * FT;
      if (i < FIY * FIX) {
        const int r = i / FIX, c = i % FIX;
        int y = wrap(2 * n0 + r, rows), x = wrap(2 * m0 + c, cols);
        if (y >= M) y = 2 * (M - 1) - y;  // mirror past the last row (level 1 only)
        if (x >= N) x = 2 * (N - 1) - x;
        v[k] = src[(int64_t)y * in_rs + x];
      }
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      const int i = threadIdx.x + k * FT;
      if (i < FIY * FIX) tile[i / FIX][i % FIX] = v[k];
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < FIY * FX; i += FT) {
    const int r = i / FX, m = i % FX;
    float a = 0.f, b = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float v = tile[r][2 * m + k];
      a = fmaf(kH[k], v, a);
      b = fmaf(kG[k], v, b);
    }
    lo[r][m] = a;
    hi[r][m] = b;
  }
  __syncthreads();
  const int ro = rows / 2, co = cols / 2;
  float* d = det + (int64_t)img * det_is;
  for (int i = threadIdx.x; i < FY * FX; i += FT) {
    const int n = i / FX, m = i % FX;
    const int yo = n0 + n, xo = m0 + m;
    if (yo >= ro || xo >= co) continue;
    float s_ll = 0.f, s_lh = 0.f, s_hl = 0.f, s_hh = 0.f;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      const float l = lo[2 * n + k][m], h = hi[2 * n + k][m];
      s_ll = fmaf(kH[k], l, s_ll);
      s_lh = fmaf(kG[k], l, s_lh);
      s_hl = fmaf(kH[k], h, s_hl);
      s_hh = fmaf(kG[k], h, s_hh);
    }
    if (ll) ll[(int64_t)img * ll_is + (int64_t)yo * ll_rs + xo] = s_ll;
    d[(int64_t)(yo + ro) * det_rs + xo] = s_lh;        // horizontal low, vertical high
    d[(int64_t)yo * det_rs + xo + co] = s_hl;          // horizontal high, vertical low
    d[(int64_t)(yo + ro) * det_rs + xo + co] = s_hh;
  }
}

// ---------------------------------------------------------------------------
// Wiener step and inverse level.  Output tile IY x IX of the level's rows x cols plane:
// it takes CY x CX coefficients of each subband (the filter's reach is 3 back).  A wave
// takes one subband and a run of coefficient rows, a raw coefficient column per lane: the
// rows come straight from memory into registers, the windows' horizontal sums from the
// neighbouring lanes, the vertical ones from the last nine rows; only the results go to
// LDS.
//
// Level 1 of 16 1080p images (coefficients 176 MB in, residuals 133 MB out): 106 us, bound
// by its vector instructions (issue slots 76% busy: 18 per raw coefficient, 38 per
// result), where the variances as a pass of their own took 88 us and wrote and read
// 200 MB more, and the inverse after it 88 us.  64 x 96: a raw column per lane with both
// halos (59 of 64 lanes, 51 of them results); 32 rows where a level has few tiles
// (launch_residuals).  A CU holds two workgroups of 12 waves (68 VGPRs, 55 kB of LDS
// each at 64 rows).  With the raw tile in LDS and nine reads per coefficient and row the
// kernel took 115 us, two columns per thread 140 us (106 VGPRs).
constexpr int IX = 96;
constexpr int CX = IX / 2 + 3;
constexpr int WH = 4;       // the 9 x 9 window's reach
constexpr int WN = 4;       // runs of rows per subband
constexpr int IT = 3 * WN * 64;
constexpr int VS = CX | 1;  // LDS row stride of the vertical synthesis (read at every second column)
static_assert(9 * CX <= IT && 9 * (64 / 2 + 3) <= IT, "wrapped places of short subbands: one per thread");
static_assert(CX + 2 * WH <= 64 && 7 + WH + IX / 2 + WH <= 64, "a raw column per lane, wrapped ones too");

// v of the previous (next) lane, zero into the first (last).
__device__ __forceinline__ float lane_prev(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, true));  // wave_shr:1
}
__device__ __forceinline__ float lane_next(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, true));  // wave_shl:1
}

// The removed part of a coefficient c whose windows' sums of c^2 are t3, t5, t7, t9.
__device__ __forceinline__ float removed(float c, float t3, float t5, float t7, float t9, float s2) {
  const float m = fminf(fminf(t3 * (1.f / 9.f), t5 * (1.f / 25.f)), fminf(t7 * (1.f / 49.f), t9 * (1.f / 81.f)));
  const float v = fmaxf(0.f, m - s2);
  return s2 > 0.f ? c * (s2 / (v + s2)) : 0.f;
}

// The removed parts of R rows of one subband (column x of its first row at src, row
// stride rs), rows n.. (n < 0: the far end's last rows, n + ro..).  Raw rows outside the
// subband, and lanes that hold no column of it (xin false), count as zero.  The results
// of the first `rows` rows go to out (LDS, row stride CX) where put.
template <int R>
__device__ __forceinline__ void wiener_rows(const float* src, int64_t rs, unsigned x, bool xin, int n, int ro, int rows,
                                            float s2, float* out, bool put) {
  // the squares rounded before they are summed, whatever R: a coefficient's part is the
  // same bits in every tile and run it may fall in
#pragma clang fp contract(off)
  const int first = n < 0 ? -ro : 0;  // the subband's first row in the run's numbering
  float v[R + 8], h[4][R + 8];
#pragma unroll
  for (int k = 0; k < R + 8; ++k) {
    const int y = n - WH + k - first;
    v[k] = src[(int64_t)(y >= 0 && y < ro ? y : 0) * rs + x];
  }
#pragma unroll
  for (int k = 0; k < R + 8; ++k) {
    const int y = n - WH + k - first;
    v[k] = xin && y >= 0 && y < ro ? v[k] : 0.f;
    const float q = v[k] * v[k];
    float l = lane_prev(q), r = lane_next(q);
    h[0][k] = l + q + r;
#pragma unroll
    for (int w = 1; w < 4; ++w) {
      l = lane_prev(l);
      r = lane_next(r);
      h[w][k] = h[w - 1][k] + l + r;
    }
    if (k >= 8) {
      const int j = k - 8, m = j + WH;
      // sums of two and four rows, each formed once for the outputs that share it
      auto two = [&](int w, int i) { return h[w][i] + h[w][i + 1]; };
      auto four = [&](int w, int i) { return two(w, i) + two(w, i + 2); };
      const float t3 = two(0, m - 1) + h[0][m + 1];
      const float t5 = four(1, m - 2) + h[1][m + 2];
      const float t7 = four(2, m - 3) + (two(2, m + 1) + h[2][m + 3]);
      const float t9 = (four(3, m - 4) + four(3, m)) + h[3][m + 4];
      const float g = removed(v[m], t3, t5, t7, t9, s2);
      if (put && j < rows) out[j * CX] = g;
    }
  }
}

typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));

// ll: approximation plane (ro x co, stride ll_rs, image stride ll_is) or null (zero: the
// residual keeps none of the coarsest); det: coefficient planes, quadrants as in
// k_dwt_fwd.  out: rows x cols plane (stride out_rs, image stride out_is), only its first
// M rows and N columns written.
template <int IY>
__global__ __launch_bounds__(IT, 6) void k_dwt_inv(const float* __restrict__ ll, int64_t ll_is, int64_t ll_rs,
                                                     const float* __restrict__ det, int64_t det_is, int64_t det_rs,
                                                     int rows, int cols, int M, int N, float s2,
                                                     float* __restrict__ out, int64_t out_is, int64_t out_rs) {
  constexpr int CY = IY / 2 + 3;
  constexpr int WR = (CY + WN - 1) / WN;             // rows of a run
  constexpr int WRE = (IY / 2 + WN - 2) / (WN - 1);  // rows of a run in a tile of the first rows
  __shared__ float s[3][CY][CX], a[CY][CX];  // removed parts (LH, HL, HH) and LL
  __shared__ float vl[IY][VS], vh[IY][VS];   // vertical synthesis
  const int img = blockIdx.z, tid = threadIdx.x;
  const int ro = rows / 2, co = cols / 2;
  const int y0 = blockIdx.y * IY, x0 = blockIdx.x * IX;
  const int n0 = y0 / 2 - 3, m0 = x0 / 2 - 3;
  // A subband shorter than 7 (then the level is one tile in that direction): the far end's
  // last seven would hold a column twice, so each is computed once and the wrapped places
  // are copied afterwards (a call of one 96 x 96 image 74 us, of 640 x 16 74, of 112 x 112
  // 74; with every place of the tile summed element by element 116 and 166).
  const bool few_rows = ro < 3 + WH, few_cols = co < 3 + WH;
  {
    // the wave's index, and with it every row's address, in scalar registers
    const int lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* d = det + (int64_t)img * det_is;
    // LL rows, requested first
    constexpr int NC = (CY + 3 * WN - 1) / (3 * WN);
    float va[NC];
    const unsigned xa = lane < CX ? (unsigned)wrap(m0 + lane, co) : 0u;
#pragma unroll
    for (int k = 0; k < NC; ++k)
      va[k] = ll ? (ll + (int64_t)img * ll_is + (int64_t)wrap(n0 + w + k * 3 * WN, ro) * ll_rs)[xa] : 0.f;
    const int band = w / WN, run = w % WN;
    const float* src = d + (band == 1 ? 0 : (int64_t)ro * det_rs) + (band == 0 ? 0 : co);
    float* sb = &s[band][0][0];
    // The lane's column.  In a tile of the first columns, lanes 0..6 hold the far end's
    // last seven (the synthesis is periodic, the windows are not), four lanes zeros; of a
    // subband of fewer columns each is held once.
    int m = m0 - WH + lane;
    bool in = m < co && lane < CX + 2 * WH, res = lane >= WH && lane < WH + CX;
    if (few_cols) {
      m = lane - WH;
      in = res = m >= 0 && m < co;
    } else if (m0 < 0) {
      const bool far = lane < 7;
      m = far ? lane - 7 : lane - 7 - WH;
      in = far || (m >= 0 && m < co && m < IX / 2 + WH);
      res = far ? m >= -3 : m >= 0 && m < IX / 2;
    }
    const unsigned x = in ? (unsigned)(m < 0 ? m + co : m) : 0u;
    float* o = sb + (res ? m - m0 : 0);
    if (n0 < 0) {
      // a tile of the first rows: the far end's last three are a run of their own
      if (run > 0)
        wiener_rows<WRE>(src, det_rs, x, in, (run - 1) * WRE, ro, min(WRE, IY / 2 - (run - 1) * WRE), s2,
                         o + (3 + (run - 1) * WRE) * CX, res);
      else if (!few_rows)
        wiener_rows<3>(src, det_rs, x, in, -3, ro, 3, s2, o, res);
    } else {
      wiener_rows<WR>(src, det_rs, x, in, n0 + run * WR, ro, min(WR, CY - run * WR), s2, o + run * WR * CX, res);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
      const int r = w + k * 3 * WN;
      if (lane < CX && r < CY) a[r][lane] = va[k];
    }
  }
  __syncthreads();
  if (few_rows || few_cols) {
    // the places before the first row or column, from the subband's last three (or fewer)
    auto col = [&](int c) { return few_cols && c < 3 ? 3 + wrap(c - 3, co) : c; };
    if (few_rows && tid < 9 * CX) {
      const int b = tid / (3 * CX), r = tid / CX % 3, c = tid % CX;
      s[b][r][c] = s[b][3 + wrap(r - 3, ro)][col(c)];
    }
    if (few_cols && tid < 9 * CY) {
      const int b = tid / (3 * CY), r = tid / 3 % CY, c = tid % 3;
      if (!few_rows || r >= 3) s[b][r][c] = s[b][r][col(c)];
    }
    __syncthreads();
  }
  // vertical: output row y takes coefficient rows y/2 - j (j = 0..3) with taps y%2 + 2j
  // (y0 is even).  A thread takes one coefficient column and 8 output rows, which
  // need 7 coefficient rows of each subband: read into registers once.
  static_assert(IY % 8 == 0, "whole vertical work items");
  for (int i = tid; i < (IY / 8) * CX; i += IT) {
    const int c = i % CX, g = i / CX;
    float q[4][7];
#pragma unroll
    for (int t = 0; t < 7; ++t) q[0][t] = a[4 * g + t][c];
#pragma unroll
    for (int b = 0; b < 3; ++b)
#pragma unroll
      for (int t = 0; t < 7; ++t) q[b + 1][t] = s[b][4 * g + t][c];
#pragma unroll
    for (int rr = 0; rr < 8; ++rr) {
      const int p = rr & 1, nb = rr / 2 + 3;  // local coefficient row of j = 0, minus 4g
      float L = 0.f, H = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int k = p + 2 * j;
        L = fmaf(kH[k], q[0][nb - j], fmaf(kG[k], q[1][nb - j], L));
        H = fmaf(kH[k], q[2][nb - j], fmaf(kG[k], q[3][nb - j], H));
      }
      vl[8 * g + rr][c] = L;
      vh[8 * g + rr][c] = H;
    }
  }
  __syncthreads();
  // horizontal: four outputs of a row per thread, from five columns of each half
  float* o = out + (int64_t)img * out_is;
  const int yend = min(rows, M), xend = min(cols, N);
  for (int i = tid; i < IY * IX / 4; i += IT) {
    const int r = i / (IX / 4), c = i % (IX / 4) * 4;
    const int y = y0 + r, x = x0 + c;
    if (y >= yend || x >= xend) continue;
    float l[5], h[5], v[4];
#pragma unroll
    for (int t = 0; t < 5; ++t) l[t] = vl[r][c / 2 + t], h[t] = vh[r][c / 2 + t];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int p = t & 1, mb = t / 2 + 3;
      v[t] = 0.f;
#pragma unroll
      for (int j = 0; j < 4; ++j) v[t] = fmaf(kH[p + 2 * j], l[mb - j], fmaf(kG[p + 2 * j], h[mb - j], v[t]));
    }
    float* po = o + (int64_t)y * out_rs + x;
    if (x + 4 <= xend) {
      *reinterpret_cast<f4u*>(po) = f4u{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
      for (int t = 0; t < 4; ++t)
        if (x + t < xend) po[t] = v[t];
    }
  }
}

}  // namespace

int residual_padded(int n) { return (n + 15) / 16 * 16; }

size_t residual_workspace_floats(int M, int N) {
  const size_t M2 = (size_t)residual_padded(M), N2 = (size_t)residual_padded(N);
  return M2 * N2 + (M2 / 2) * (N2 / 2) + (M2 / 4) * (N2 / 4);
}

hipError_t launch_residuals(const float* in, int64_t in_is, int64_t in_rs, int L, int M, int N, float sigma0,
                            float* ws, float* out, int64_t out_is, int64_t out_rs, hipStream_t s) {
  if (L <= 0) return hipSuccess;
  const int M2 = residual_padded(M), N2 = residual_padded(N);
  const int64_t P = (int64_t)M2 * N2;
  const int64_t per = (int64_t)residual_workspace_floats(M, N);
  // per image: coefficient plane C, approximation planes T1, T2
  float* C = ws;
  float* T1 = ws + P;
  float* T2 = T1 + (int64_t)(M2 / 2) * (N2 / 2);
  constexpr int kLevels = 4;
  // forward: level l reads a rows x cols plane and writes rows/2 x cols/2 subbands
  for (int l = 1; l <= kLevels; ++l) {
    const int rows = M2 >> (l - 1), cols = N2 >> (l - 1);
    const float* src;
    int64_t sis, srs;
    int mm, nn;
    if (l == 1) {
      src = in, sis = in_is, srs = in_rs, mm = M, nn = N;
    } else {
      src = (l % 2 == 0) ? T1 : T2;  // level l-1 wrote its approximation there
      sis = per, srs = cols, mm = rows, nn = cols;
    }
    float* dst_ll = l == kLevels ? nullptr : ((l % 2 == 1) ? T1 : T2);
    dim3 grid((unsigned)((cols / 2 + FX - 1) / FX), (unsigned)((rows / 2 + FY - 1) / FY), (unsigned)L);
    k_dwt_fwd<<<grid, FT, 0, s>>>(src, sis, srs, rows, cols, mm, nn, dst_ll, per, cols / 2, C, per, N2);
  }
  const float s2 = sigma0 * sigma0;
  // inverse: level l rebuilds the rows x cols plane from its rows/2 x cols/2 subbands.
  // Approximations: level 4 starts from zero and writes T1, level 3 reads T1 and writes
  // T2, level 2 reads T2 and writes T1, level 1 reads it and writes the cropped residual.
  for (int l = kLevels; l >= 1; --l) {
    const int rows = M2 >> (l - 1), cols = N2 >> (l - 1);
    const float* src_ll = l == kLevels ? nullptr : (l % 2 == 1 ? T1 : T2);
    float* dst = out;
    int64_t dis = out_is, drs = out_rs;
    int mm = M, nn = N;
    if (l > 1) {
      dst = l % 2 == 0 ? T1 : T2;
      dis = per, drs = cols, mm = rows, nn = cols;
    }
    // A level of at most one tile of 64 rows per CU takes tiles of 32, whose work is half
    // as long on twice the CUs: a call of 3 images of 333 x 501 84 -> 76 us.  Everywhere
    // they would cost 16 images of 1080 x 1920 270 -> 302 us (more halo).
    auto inv = [&](auto iy) {
      constexpr int IY = decltype(iy)::value;
      dim3 grid((unsigned)((cols + IX - 1) / IX), (unsigned)((rows + IY - 1) / IY), (unsigned)L);
      k_dwt_inv<IY><<<grid, IT, 0, s>>>(src_ll, per, cols / 2, C, per, N2, rows, cols, mm, nn, s2, dst, dis, drs);
    };
    if ((int64_t)((cols + IX - 1) / IX) * ((rows + 63) / 64) * L <= 256)
      inv(std::integral_constant<int, 32>());
    else
      inv(std::integral_constant<int, 64>());
  }
  return hipGetLastError();
}

}  // namespace prnu
