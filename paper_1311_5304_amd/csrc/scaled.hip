// Scaled decoding (1/2, 1/4, 1/8 output) in one pass: reduced dequantise +
// IDCT -> chroma upsampling -> YCbCr->RGB (or gray samples) -> output rows.
//
// The block's top-left N x N coefficients (N = 8 / scale) go through the
// N-point IDCT with the 8-point normalisation, in islow-style fixed point
// (x0 * 2^13 + sum round(2^13 sqrt(2) cos((2m+1) u pi / 2N)) x_u, pass 1
// descaled by 11, pass 2 by 18, +128); upsampling and colour are those of the
// full-size path at the reduced size.
//
// A workgroup decodes a tile of 64 or more MCUs, one block per lane, and each
// wave takes one block position of 64 MCUs: component, quant table and sample
// plane are the wave's, so the lanes' address arithmetic is a few shifts.
// All of a tile's loads are in flight at once and the samples never leave the
// LDS; where the triangle filter reads chroma across the tile's edge, one or
// two more waves decode the neighbour MCUs' chroma blocks again, from lines
// that the neighbour tile of the same XCD has just fetched.
//
// Measured, kernel spacing in a graph (4096x3072, fancy): 4:2:0 at 1/2 17.1 us
// as two launches with the samples in memory between them, 10.0 us here (47 MB
// of whole lines and output: 8.6 us at the copy kernel's rate); 6000x4000
// 4:2:2 at 1/8 20.1 -> 15.4 us (96 MB of lines).  Two or four blocks a lane,
// or loads past the caches, were no faster (15.5 and 16.6 us at 1/8).
#include "mjd_internal.h"

namespace mjd {
namespace scaled {

struct View {
  const int16_t* coef;
  const uint16_t* qt;
  uint8_t* out;
  uint32_t pitch;
  int width, height;  // of the output
  int mcus_x, mcus_y;
  int comp_w, comp_h;  // the chroma components' true size at the output scale
  int tiles_x;
  uint32_t n_tiles;
  int qsel[3];
};

// Two 32-bit words of coefficients, at the alignment a coefficient row has;
// four quant table entries at any 2-byte address (unaligned access mode).
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef uint32_t v2u2 __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t u32a2 __attribute__((aligned(2)));
typedef __attribute__((address_space(3))) v2u lds64;

// The tile of a scale (N samples a block side), luma sampling HF x VF,
// NC components, with the triangle filter or without.
template <int N_, int HF_, int VF_, bool FANCY_, int NC_>
struct Tile {
  static constexpr int N = N_, HF = HF_, VF = VF_, NC = NC_;
  // the triangle filter serves factors of 2; the rest replicate
  static constexpr bool FH = NC == 3 && FANCY_ && HF == 2;
  static constexpr bool FV = NC == 3 && FANCY_ && VF == 2 && HF <= 2;
  static constexpr int LUMA = HF * VF, BPM = NC == 1 ? 1 : LUMA + 2;
  // GROUPS x 64 MCUs, TX x TY: 4:2:0 and 4:1:1 fill eight or six waves with
  // 64; more where an MCU has fewer blocks
  static constexpr int GROUPS = NC == 1 ? 8 : BPM == 6 ? 1 : 2;
  static constexpr int TX = NC == 1 ? 64 : BPM == 6 || VF == 2 ? 16 : 32;
  static constexpr int TY = 64 * GROUPS / TX;
  // with the neighbours whose chroma the filter reads; HALO of them
  static constexpr int EX = TX + (FH ? 2 : 0), EY = TY + (FV ? 2 : 0);
  static constexpr int HALO = EX * EY - TX * TY;
  static_assert(HALO <= 64, "a wave per component");
  static constexpr int CORE_WAVES = GROUPS * BPM, WAVES = CORE_WAVES + (2 * HALO + 63) / 64;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int YW = TX * HF * N, YH = TY * VF * N;  // luma samples, bytes in LDS
  static constexpr int CW = EX * N, CH = EY * N;            // chroma samples, Cb | Cr << 16 in LDS
  static_assert(YW % 4 == 0 && YH % 2 == 0, "whole units of 4 x 2 pixels");
  static constexpr int SPB = N == 4 ? 10 : 3;  // dwords between blocks of the transposition (no bank conflicts)
};

// 1-D transforms, `bias` added; every sum wraps in 32 bits, so the order of
// the terms does not matter.  4 points: K = 2^13 sqrt(2) cos((2m+1) u pi / 8),
// which is +-2^13 for u = 2; 2 points: +-2^13.
constexpr int kRed1 = 10703;  // round(2^13 sqrt(2) cos(pi/8))
constexpr int kRed3 = 4433;   // round(2^13 sqrt(2) cos(3 pi/8))
template <bool SMALL>  // every input in 24 bits
__device__ __forceinline__ int mul_red(int x, int k) {
  return SMALL ? mul24(x, k) : static_cast<int>(static_cast<uint32_t>(x) * static_cast<uint32_t>(k));
}
template <int N, bool SMALL>
__device__ __forceinline__ void red_1d(const int x[N], int y[N], int bias) {
  if constexpr (N == 4) {
    const int e0 = ((x[0] + x[2]) << 13) + bias, e1 = ((x[0] - x[2]) << 13) + bias;
    const int o0 = mul_red<SMALL>(x[1], kRed1) + mul_red<SMALL>(x[3], kRed3);
    const int o1 = mul_red<SMALL>(x[1], kRed3) - mul_red<SMALL>(x[3], kRed1);
    y[0] = e0 + o0;
    y[1] = e1 + o1;
    y[2] = e1 - o1;
    y[3] = e0 - o0;
  } else {
    y[0] = ((x[0] + x[1]) << 13) + bias;
    y[1] = ((x[0] - x[1]) << 13) + bias;
  }
}

// One block: the rows' words -> the samples.  SMALL: the dequantised values
// fit in 24 bits (table entries of 8 bits), where a product takes one pass of
// the multiplier instead of four.
template <int N, bool SMALL>
__device__ __forceinline__ void red_block(const uint32_t cw[N][2], const uint32_t qw[N][2], uint32_t px[N][N]) {
  auto coef = [&](int u, int v) { return static_cast<int>(cw[u][v >> 1] << (16 * (1 - (v & 1)))) >> 16; };
  auto quant = [&](int u, int v) { return static_cast<int>((qw[u][v >> 1] >> (16 * (v & 1))) & 0xFFFFu); };
  if constexpr (N == 1) {
    px[0][0] = static_cast<uint32_t>(clamp255i((mul24(coef(0, 0), quant(0, 0)) * 32768 + (1 << 17) + (128 << 18)) >> 18));
  } else {
    int ws[N][N];
#pragma unroll
    for (int v = 0; v < N; ++v) {  // pass 1: column v
      int x[N], y[N];
#pragma unroll
      for (int u = 0; u < N; ++u) x[u] = mul24(coef(u, v), quant(u, v));
      red_1d<N, SMALL>(x, y, 1 << 10);
#pragma unroll
      for (int m = 0; m < N; ++m) ws[m][v] = y[m] >> 11;  // 21 bits
    }
#pragma unroll
    for (int m = 0; m < N; ++m) {  // pass 2: row m
      int z[N];
      red_1d<N, true>(ws[m], z, (1 << 17) + (128 << 18));
#pragma unroll
      for (int n = 0; n < N; ++n) px[m][n] = static_cast<uint32_t>(clamp255i(z[n] >> 18));
    }
  }
}

// N samples as one store, to the LDS or to the output at any byte address.
template <int N>
__device__ __forceinline__ void store_row(lds8* d, const uint32_t px[N]) {
  if constexpr (N == 4) *reinterpret_cast<lds32*>(d) = px[0] | (px[1] << 8) | (px[2] << 16) | (px[3] << 24);
  else if constexpr (N == 2) *reinterpret_cast<ldsu16*>(d) = static_cast<uint16_t>(px[0] | (px[1] << 8));
  else d[0] = static_cast<uint8_t>(px[0]);
}
template <int N>
__device__ __forceinline__ void store_row(gbl8* d, const uint32_t px[N]) {
  if constexpr (N == 4) *reinterpret_cast<gbl32u*>(d) = px[0] | (px[1] << 8) | (px[2] << 16) | (px[3] << 24);
  else if constexpr (N == 2) *reinterpret_cast<gbl16u*>(d) = static_cast<uint16_t>(px[0] | (px[1] << 8));
  else d[0] = static_cast<uint8_t>(px[0]);
}

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 pair(uint32_t w) { return __builtin_bit_cast(u16x2, w); }
__device__ __forceinline__ uint32_t word(u16x2 p) { return __builtin_bit_cast(uint32_t, p); }

// The chroma of the 4 x 2 pixels at column x (a multiple of 4) and row y
// (even) of the tile, less 128: Cb and Cr travel as the 16-bit halves of one
// word, every biased sum in 16 bits, and one bit-field extract shifts and
// unpacks it.  (gx, gy): the pixels in the image.
template <class T>
struct Chroma {
  static constexpr int SH = T::FH && T::FV ? 4 : T::FH || T::FV ? 2 : 0;
  uint32_t c[2][4];
  __device__ __forceinline__ Chroma(const lds32* ch, int x, int y, int gx, int gy, const View& v) {
    constexpr int N = T::N;
    const lds32* row = ch + (y / T::VF + (T::FV ? N : 0)) * T::CW + (x / T::HF + (T::FH ? N : 0));
    const u16x2 three = {3, 3};
    if constexpr (T::FH || T::FV) {
      // the horizontal filter reads the samples kx-1 .. kx+2
      constexpr int FIRST = T::FH ? -1 : 0;
      u16x2 s[2][4];
#pragma unroll
      for (int i = 0; i < 4; ++i) s[0][i] = pair(row[FIRST + i]);
      if constexpr (T::FV) {
        // 3:1 sums with the row above (even) and below (odd), the sample's
        // own past the component's ends
        const int ky = gy >> 1;
        const int up = ky > 0 ? -T::CW : 0, down = ky + 1 <= v.comp_h - 1 ? T::CW : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const u16x2 t = s[0][i] * three;
          s[0][i] = t + pair(row[FIRST + i + up]);
          s[1][i] = t + pair(row[FIRST + i + down]);
        }
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) s[1][i] = pair(row[T::CW + FIRST + i]);
      }
      constexpr unsigned short EVEN = (SH == 4 ? 8 : 1) - (128 << SH), ODD = (SH == 4 ? 7 : 2) - (128 << SH);
      const u16x2 even = {EVEN, EVEN}, odd = {ODD, ODD};
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if constexpr (T::FH) {
          const int kx = gx >> 1;
          const u16x2 l = kx == 0 ? s[r][1] : s[r][0];
          const u16x2 m = kx + 1 > v.comp_w - 1 ? s[r][1] : s[r][2], e = kx + 2 > v.comp_w - 1 ? s[r][2] : s[r][3];
          c[r][0] = word(s[r][1] * three + (l + even));
          c[r][1] = word(s[r][1] * three + (m + odd));
          c[r][2] = word(s[r][2] * three + (s[r][1] + even));
          c[r][3] = word(s[r][2] * three + (e + odd));
        } else {
#pragma unroll
          for (int i = 0; i < 4; ++i) c[r][i] = word(s[r][i] + (r ? odd : even));
        }
      }
    } else {
      const u16x2 bias = {static_cast<unsigned short>(-128), static_cast<unsigned short>(-128)};
#pragma unroll
      for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < 4; ++i) c[r][i] = word(pair(row[(r / T::VF) * T::CW + i / T::HF]) + bias);
    }
  }
  __device__ __forceinline__ int cb(int r, int i) const { return __builtin_amdgcn_sbfe(static_cast<int>(c[r][i]), SH, 16 - SH); }
  __device__ __forceinline__ int cr(int r, int i) const { return static_cast<int>(c[r][i]) >> (16 + SH); }
};

// A grayscale block's rows, cropped, into the output.
template <int N>
__device__ __forceinline__ void gray_rows(const uint32_t px[N][N], int mx, int my, const View& v) {
  const int x0 = mx * N, n = min(N, v.width - x0);
  gbl8* dst = (gbl8*)(v.out + static_cast<size_t>(my) * N * v.pitch + x0);
#pragma unroll
  for (int m = 0; m < N; ++m) {
    if (my * N + m >= v.height) break;
    if (n == N) {
      store_row<N>(dst, px[m]);
    } else {
#pragma unroll
      for (int i = 0; i < N - 1; ++i)
        if (i < n) dst[i] = static_cast<uint8_t>(px[m][i]);
    }
    dst += v.pitch;
  }
}

// 4 pixels of an output row: 12 bytes, or the 3, 6 or 9 inside the image.
__device__ __forceinline__ void rgb_row(gbl8* dst, const uint32_t w[3], int n) {
  if (n == 4) {
    gbl32u* d = reinterpret_cast<gbl32u*>(dst);
    d[0] = w[0];
    d[1] = w[1];
    d[2] = w[2];
  } else {
    for (int k = 0; k < n; ++k) {
      // pixel k: bytes 3k .. 3k + 2 of the words
      const uint32_t p = k == 0 ? w[0] : k == 1 ? __builtin_amdgcn_alignbyte(w[1], w[0], 3) : __builtin_amdgcn_alignbyte(w[2], w[1], 2);
      *reinterpret_cast<gbl16u*>(dst) = static_cast<uint16_t>(p);
      dst[2] = static_cast<uint8_t>(p >> 16);
      dst += 3;
    }
  }
}

template <int N, int HF, int VF, bool FANCY, int NC>
__global__ __launch_bounds__((Tile<N, HF, VF, FANCY, NC>::THREADS)) void scaled_tile(const View v) {
  using T = Tile<N, HF, VF, FANCY, NC>;
  __shared__ __align__(16) uint32_t turn[N == 1 ? 1 : T::THREADS * T::SPB];
  __shared__ __align__(16) uint8_t ys[NC == 1 ? 16 : T::YW * T::YH];
  __shared__ __align__(16) uint32_t cs[NC == 1 ? 1 : T::CW * T::CH];
  // the grid is a multiple of 8 dealt to the XCDs round-robin: each takes a
  // contiguous run of tiles, whose shared neighbours meet in its L2
  const uint32_t tile = (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  if (tile >= v.n_tiles) return;
  const int tyi = static_cast<int>(tile / static_cast<uint32_t>(v.tiles_x));
  const int mx0 = (static_cast<int>(tile) - tyi * v.tiles_x) * T::TX, my0 = tyi * T::TY;
  const int t = static_cast<int>(threadIdx.x), lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

  // the lane's block: block j of the MCU (tx, ty) of the tile, or of a
  // neighbour MCU
  int tx, ty, j;
  bool valid = true;
  if (wave < T::CORE_WAVES) {
    j = wave / T::GROUPS;
    tx = lane % T::TX;
    ty = lane / T::TX + (wave % T::GROUPS) * (64 / T::TX);
  } else {
    // the MCUs of the rows above and below, then those left and right
    int p = T::HALO > 32 ? lane : lane & 31;
    j = T::LUMA + (T::HALO > 32 ? wave - T::CORE_WAVES : lane >> 5);
    tx = ty = 0;
    valid = p < T::HALO;
    if constexpr (T::FV) {
      if (p < 2 * T::EX) {
        const int r = p >= T::EX ? 1 : 0;
        ty = r ? T::TY : -1;
        tx = p - r * T::EX - (T::FH ? 1 : 0);
      }
      p -= 2 * T::EX;
    }
    if constexpr (T::FH) {
      if (p >= 0) {
        tx = p & 1 ? T::TX : -1;
        ty = p >> 1;
      }
    }
  }
  const int mx = mx0 + tx, my = my0 + ty;
  valid = valid && mx >= 0 && mx < v.mcus_x && my >= 0 && my < v.mcus_y;
  const int comp = NC == 1 || j < T::LUMA ? 0 : j - T::LUMA + 1;
  // a lane without a block reads one of the tile's first MCU and drops it:
  // loads without branches go out together
  const uint32_t blk = (static_cast<uint32_t>(valid ? my : my0) * static_cast<uint32_t>(v.mcus_x) +
                        static_cast<uint32_t>(valid ? mx : mx0)) * T::BPM + static_cast<uint32_t>(j);
  const uint16_t* q = v.qt + 64 * (comp == 0 ? v.qsel[0] : comp == 1 ? v.qsel[1] : v.qsel[2]);

  uint32_t cw[N][2], qw[N][2], px[N][N];
  if constexpr (N == 1) {
    cw[0][0] = static_cast<uint16_t>(v.coef[static_cast<size_t>(blk) * 64]);
    qw[0][0] = q[0];
    red_block<N, true>(cw, qw, px);
  } else {
    // A wave's N loads take N-th parts of its blocks, all rows of a block in
    // one load (one pass over the line in the L1), and the rows meet their
    // lane through the LDS.
    constexpr int PER = 64 / N;  // blocks a load
#pragma unroll
    for (int k = 0; k < N; ++k) {
      const uint32_t from = static_cast<uint32_t>(__shfl(static_cast<int>(blk), lane / N + PER * k));
      const int16_t* src = v.coef + (static_cast<size_t>(from) * 64 + 8 * (lane % N));
      if constexpr (N == 4) {
        const v2u w = *reinterpret_cast<const v2u*>(src);
        cw[k][0] = w.x;
        cw[k][1] = w.y;
      } else {
        cw[k][0] = *reinterpret_cast<const uint32_t*>(src);
      }
    }
    uint32_t odd = 0;  // the entries that are multiplied on: rows 1 and 3
#pragma unroll
    for (int u = 0; u < N; ++u) {
      if constexpr (N == 4) {
        const v2u2 w = *reinterpret_cast<const v2u2*>(q + 8 * u);
        qw[u][0] = w.x;
        qw[u][1] = w.y;
        if (u & 1) odd |= w.x | w.y;
      } else {
        qw[u][0] = *reinterpret_cast<const u32a2*>(q + 8 * u);
      }
    }
    uint32_t* mine = turn + (t & ~63) * T::SPB;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      uint32_t* d = mine + (lane / N + PER * k) * T::SPB + (lane % N) * (N / 2);
      if constexpr (N == 4) *reinterpret_cast<v2u*>(d) = v2u{cw[k][0], cw[k][1]};
      else d[0] = cw[k][0];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const uint32_t* s = mine + lane * T::SPB + u * (N / 2);
      if constexpr (N == 4) {
        const v2u w = *reinterpret_cast<const v2u*>(s);
        cw[u][0] = w.x;
        cw[u][1] = w.y;
      } else {
        cw[u][0] = s[0];
      }
    }
    // N == 2 multiplies by powers of two alone
    if (N == 2 || __all((odd & 0xFF00FF00u) == 0)) red_block<N, true>(cw, qw, px);
    else red_block<N, false>(cw, qw, px);
  }

  if constexpr (NC == 1) {
    if (valid) gray_rows<N>(px, mx, my, v);
  } else {
    if (valid) {
      if (comp == 0) {
        const int jy = j / HF, jx = j - jy * HF;
        uint8_t* d = ys + (ty * VF + jy) * N * T::YW + (tx * HF + jx) * N;
#pragma unroll
        for (int m = 0; m < N; ++m) {
          store_row<N>((lds8*)d, px[m]);
          d += T::YW;
        }
      } else {
        uint16_t* d = reinterpret_cast<uint16_t*>(cs) +
                      2 * ((ty + (T::FV ? 1 : 0)) * N * T::CW + (tx + (T::FH ? 1 : 0)) * N) + (comp - 1);
#pragma unroll
        for (int m = 0; m < N; ++m) {
#pragma unroll
          for (int n = 0; n < N; ++n) d[2 * n] = static_cast<uint16_t>(px[m][n]);
          d += 2 * T::CW;
        }
      }
    }
    __syncthreads();

    // 4 x 2 pixels a lane: 12 contiguous bytes a row, a wave's stores without gaps
    constexpr int UPR = T::YW / 4, UNITS = UPR * (T::YH / 2);
    const int gx0 = mx0 * HF * N, gy0 = my0 * VF * N;
#pragma unroll
    for (int base = 0; base < UNITS; base += T::THREADS) {
      const int i = base + t;
      if (UNITS % T::THREADS != 0 && i >= UNITS) break;
      const int y = i / UPR * 2, x = i % UPR * 4;
      const int gx = gx0 + x, gy = gy0 + y;
      if (gx >= v.width || gy >= v.height) continue;
      const Chroma<T> c((const lds32*)cs, x, y, gx, gy, v);
      gbl8* dst = (gbl8*)(v.out + static_cast<size_t>(gy) * v.pitch + static_cast<size_t>(gx) * 3);
      const int n = min(4, v.width - gx);
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if (gy + r >= v.height) break;
        const uint32_t yd = *reinterpret_cast<const uint32_t*>(ys + (y + r) * T::YW + x);
        RGBWide p[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) p[k] = ycc_wide(y16_of(yd, k), c.cb(r, k), c.cr(r, k));
        uint32_t w[3];
        pack_rgb4(p, w);
        rgb_row(dst, w, n);
        dst += v.pitch;
      }
    }
  }
}

template <int N, int HF, int VF, bool FANCY, int NC>
hipError_t launch_tiles(View v, hipStream_t s) {
  using T = Tile<N, HF, VF, FANCY, NC>;
  v.tiles_x = (v.mcus_x + T::TX - 1) / T::TX;
  v.n_tiles = static_cast<uint32_t>(v.tiles_x) * static_cast<uint32_t>((v.mcus_y + T::TY - 1) / T::TY);
  hipLaunchKernelGGL((scaled_tile<N, HF, VF, FANCY, NC>), dim3((v.n_tiles + 7u) & ~7u), dim3(T::THREADS), 0, s, v);
  return hipGetLastError();
}

template <int N>
hipError_t launch_n(const View& v, int ncomp, int hf, int vf, bool fancy, hipStream_t s) {
  if (ncomp == 1) return launch_tiles<N, 1, 1, false, 1>(v, s);
  if (hf == 4) return launch_tiles<N, 4, 1, false, 3>(v, s);
  if (hf == 2 && vf == 2) return fancy ? launch_tiles<N, 2, 2, true, 3>(v, s) : launch_tiles<N, 2, 2, false, 3>(v, s);
  if (hf == 2) return fancy ? launch_tiles<N, 2, 1, true, 3>(v, s) : launch_tiles<N, 2, 1, false, 3>(v, s);
  if (vf == 2) return fancy ? launch_tiles<N, 1, 2, true, 3>(v, s) : launch_tiles<N, 1, 2, false, 3>(v, s);
  return launch_tiles<N, 1, 1, false, 3>(v, s);
}

}  // namespace scaled

hipError_t launch_scaled(const mjd_variant& vr, const mjd_geometry& g, const int16_t* coef, const uint16_t* qt,
                         uint8_t* out, uint32_t pitch, hipStream_t s) {
  const int sc = static_cast<int>(vr.scale), nc = static_cast<int>(vr.ncomp);
  scaled::View v{};
  v.coef = coef;
  v.qt = qt;
  v.out = out;
  v.pitch = pitch;
  v.width = (static_cast<int>(vr.frame.width) + sc - 1) / sc;
  v.height = (static_cast<int>(vr.frame.height) + sc - 1) / sc;
  v.mcus_x = static_cast<int>(g.mcus_x);
  v.mcus_y = static_cast<int>(g.mcus_y);
  v.comp_w = static_cast<int>(g.comp_w[1]);
  v.comp_h = static_cast<int>(g.comp_h[1]);
  for (int c = 0; c < nc; ++c) v.qsel[c] = vr.frame.qsel[c];
  const int hf = nc == 3 ? vr.frame.h[0] : 1, vf = nc == 3 ? vr.frame.v[0] : 1;
  const bool fancy = vr.upsample == MJD_UPSAMPLE_FANCY;
  switch (sc) {
    case 2: return scaled::launch_n<4>(v, nc, hf, vf, fancy, s);
    case 4: return scaled::launch_n<2>(v, nc, hf, vf, fancy, s);
    default: return scaled::launch_n<1>(v, nc, hf, vf, fancy, s);
  }
}

}  // namespace mjd
