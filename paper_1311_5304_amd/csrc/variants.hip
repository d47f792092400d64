// Decoder variants: the IDCT methods libjpeg offers beside islow (the paper
// notes AAN-based and integer-or-float IDCTs, Sec. 2 and Sec. 3), the
// samplings beyond 4:4:4 / 4:2:2 / 4:2:0 (the paper decodes the others the
// same way, Sec. 4.2) and grayscale.  Full-size colour images run the fused
// segment kernel and scaled output the tile kernel of scaled.hip; the kernel
// here is var_gray: full-size grayscale, one block per lane, the fused
// kernels' dequantise + IDCT of each method, straight into the output rows.
// IDCT methods:
//   islow  LL&M in 13-bit fixed point (the fused kernel's arithmetic);
//   ifast  the transposed AAN flowgraph in fixed point: multipliers
//          q * 2^6 / (s(u) s(v)) (s(0) = 1, s(k) = sqrt(2) cos(k pi/16)),
//          9-bit constants with truncating products, ((v + 2^8) >> 9) + 128;
//   float  the same flowgraph in IEEE single precision, multipliers
//          fp32(q / (8 s(u) s(v))), one rounding per operation in a fixed
//          order (no contraction), floor(v + 128.5).
#include <math.h>

#include <mutex>

#include "aan.h"
#include "mjd_internal.h"

// The float method rounds once per operation, in the order written: no
// contraction into fused multiply-adds (the file is also built with
// -ffp-contract=off).
#pragma clang fp contract(off)

namespace mjd {
// Scale factors and constants of the AAN methods (aan.h), from the C
// library's cos, once.
const AanConsts& aan_consts() {
  static AanConsts k;
  static std::once_flag once;
  std::call_once(once, [] {
    double s[8];
    s[0] = 1.0;
    for (int i = 1; i < 8; ++i) s[i] = sqrt(2.0) * cos(i * M_PI / 16.0);
    for (int u = 0; u < 8; ++u)
      for (int v = 0; v < 8; ++v) {
        const double p = s[u] * s[v];
        k.ss8[8 * u + v] = 8.0 * p;
        k.a14[8 * u + v] = static_cast<int32_t>(llround(16384.0 / p));
      }
    const double c[4] = {cos(M_PI / 4.0), cos(3.0 * M_PI / 8.0), cos(M_PI / 8.0) - cos(3.0 * M_PI / 8.0),
                         cos(M_PI / 8.0) + cos(3.0 * M_PI / 8.0)};
    for (int i = 0; i < 4; ++i) {
      k.ki[i] = static_cast<int32_t>(llround(c[i] * (1 << kIfastConstBits)));
      k.kf[i] = static_cast<float>(c[i]);
    }
  });
  return k;
}

namespace var {


struct View {
  const int16_t* coef;
  const uint16_t* qt;
  uint8_t* out;
  uint64_t n_blocks;
  uint32_t pitch;
  int width, height, mcus_x, qsel;
};

// --- grayscale, one block per lane ---------------------------------------------
// A grayscale MCU is one block, so the blocks lie in raster order.  Each lane
// takes one, its 8 coefficient rows straight into registers, through the fused
// kernels' dequantise + IDCT of the method (islow: the dot-product passes;
// ifast, float: the AAN flowgraph on one lane), and out as 8-byte sample rows
// at any byte address (unaligned access mode), cropped at the image's right
// and bottom edges.  Bound by memory: 4093x3070 takes 8.8 us (37.7 MB, 6.9 at
// the copy kernel's rate).  One run of 64 blocks per wave: waves that loaded
// the next run while they transformed one held twice the registers, two
// instead of four of them to a SIMD, and half had two runs and half one (9.6
// us); through LDS by whole lines it took 9.9.
constexpr int kGrayThreads = 256;
constexpr int kGrayWaves = kGrayThreads / 64;

template <int M>
__global__ __launch_bounds__(kGrayThreads) void var_gray(const View v, const AanConsts k) {
  // islow: the table as uint16 pairs, and times 16 (the scaled pass 1
  // reads it); ifast, float: the 64 AAN multipliers
  __shared__ __align__(16) uint32_t qs[64];
  __shared__ __align__(16) uint32_t qs16[32];
  const int t = static_cast<int>(threadIdx.x);
  const uint16_t* qt = v.qt + 64 * v.qsel;
  if constexpr (M == MJD_IDCT_ISLOW) {
    if (t < 32) {
      const uint32_t lo = qt[2 * t], hi = qt[2 * t + 1];
      qs[t] = lo | (hi << 16);
      qs16[t] = ((lo << 4) & 0xFFFFu) | (((hi << 4) & 0xFFFFu) << 16);
    }
  } else {
    if (t < 64)
      qs[t] = static_cast<uint32_t>(M == MJD_IDCT_IFAST ? aan_ifast_mult(qt[t], t, k) : aan_float_mult(qt[t], t, k));
  }
  const lds32* q = (const lds32*)qs;
  const lds32* q16 = (const lds32*)qs16;
  const uint32_t n_blocks = static_cast<uint32_t>(v.n_blocks);
  const uint32_t lane = static_cast<uint32_t>(t & 63);
  const uint32_t mcx = static_cast<uint32_t>(v.mcus_x);
  const uint32_t b = (blockIdx.x * kGrayWaves + static_cast<uint32_t>(t >> 6)) * 64 + lane;
  v4i rows[8];
  {
    const v4i* src = reinterpret_cast<const v4i*>(v.coef) + static_cast<size_t>(b < n_blocks ? b : n_blocks - 1) * 8;
#pragma unroll
    for (int r = 0; r < 8; ++r) rows[r] = src[r];
  }
  __syncthreads();  // the table
  uint32_t out[16];
  if constexpr (M == MJD_IDCT_ISLOW) idct_block_fast(rows, q, q16, out);  // every lane (a wave-wide range test)
  else aan_block<M>(rows, reinterpret_cast<const ldsi*>(q), k, out);
  if (b >= n_blocks) return;
  const uint32_t by = b / mcx, bx = b - by * mcx;
  const int px0 = static_cast<int>(bx) * 8;
  const int n = min(8, v.width - px0);
  // the output as a global (not flat) pointer: the store instructions
  gbl8* dst = (gbl8*)(v.out + static_cast<size_t>(by) * 8 * v.pitch + px0);
#pragma unroll
  for (int r = 0; r < 8; ++r) {
    if (static_cast<int>(by) * 8 + r >= v.height) break;
    if (n == 8) {
      gbl32u* d = reinterpret_cast<gbl32u*>(dst);
      __builtin_nontemporal_store(out[2 * r], &d[0]);
      __builtin_nontemporal_store(out[2 * r + 1], &d[1]);
    } else {
      // n = 1..7: a whole dword if n >= 4, then a 16-bit and a byte store
      if (n >= 4) *reinterpret_cast<gbl32u*>(dst) = out[2 * r];
      const uint32_t last = n >= 4 ? out[2 * r + 1] : out[2 * r];
      gbl8* tail = dst + (n & 4);
      if (n & 2) *reinterpret_cast<gbl16u*>(tail) = static_cast<uint16_t>(last);
      if (n & 1) tail[n & 2] = static_cast<uint8_t>(last >> (8 * (n & 2)));
    }
    dst += v.pitch;
  }
}

// Grayscale: a wave per run of 64 blocks.
template <int M>
hipError_t launch_gray(const View& v, const AanConsts& k, hipStream_t s) {
  const uint64_t runs = (v.n_blocks + 63) / 64;
  const unsigned grid = static_cast<unsigned>((runs + kGrayWaves - 1) / kGrayWaves);
  hipLaunchKernelGGL(var_gray<M>, dim3(grid), dim3(kGrayThreads), 0, s, v, k);
  return hipGetLastError();
}

}  // namespace var

}  // namespace mjd

extern "C" {

int mjd_decode_variant(mjd_ctx* ctx, const mjd_variant* variant, const int16_t* d_coef, const uint16_t* d_qt,
                       uint8_t* d_out, size_t pitch, void* d_work, uint64_t work_bytes, void* stream) {
  using namespace mjd;
  if (!ctx) return fail(MJD_EINVAL, "null context");
  mjd_geometry g;
  uint64_t need = 0;
  int rc = variant_geometry(variant, &g, &need);
  if (rc != MJD_OK) return rc;
  if (!d_coef || !d_qt || !d_out) return fail(MJD_EINVAL, "null device buffer");
  if (reinterpret_cast<uintptr_t>(d_coef) % 16) return fail(MJD_EINVAL, "coefficient buffer not 16-byte aligned");
  if (reinterpret_cast<uintptr_t>(d_qt) % 2) return fail(MJD_EINVAL, "quant table buffer not 2-byte aligned");
  const int nc = static_cast<int>(variant->ncomp);
  const uint32_t scale = variant->scale ? variant->scale : 1;
  const uint32_t out_w = (variant->frame.width + scale - 1) / scale;
  const uint64_t row_bytes = static_cast<uint64_t>(nc) * out_w;
  if (pitch < row_bytes) return fail(MJD_EINVAL, "pitch %zu < %u*width", pitch, nc);
  if (pitch >= (1ull << 31)) return fail(MJD_EINVAL, "pitch %zu not below 2^31 bytes", pitch);
  const bool fused = nc == 3 && scale == 1;
  if (fused) {
    // full-size colour images: the fused segment kernel of the sampling and
    // IDCT method, one launch, no sample planes in memory
    if (pitch >= (1ull << 24)) return fail(MJD_EINVAL, "pitch %zu not below 2^24 bytes", pitch);
    ImageView im{};
    im.coef = d_coef;
    im.qt = d_qt;
    im.rgb = d_out;
    im.pitch = static_cast<uint32_t>(pitch);
    im.width = static_cast<int>(variant->frame.width);
    im.height = static_cast<int>(variant->frame.height);
    im.mcus_x = static_cast<int>(g.mcus_x);
    im.mcus_y = static_cast<int>(g.mcus_y);
    im.chroma_w = static_cast<int>(g.comp_w[1]);
    im.chroma_h = static_cast<int>(g.comp_h[1]);
    im.qsel0 = static_cast<int>(variant->frame.qsel[0]);
    im.qsel1 = static_cast<int>(variant->frame.qsel[1]);
    im.qsel2 = static_cast<int>(variant->frame.qsel[2]);
    int cur = 0;
    if (hipGetDevice(&cur) != hipSuccess || cur != ctx->device) {
      if (hipSetDevice(ctx->device) != hipSuccess) return fail(MJD_EDEVICE, "hipSetDevice(%d) failed", ctx->device);
    }
    const hipError_t e = launch_variant(im, static_cast<int>(variant->frame.h[0]), static_cast<int>(variant->frame.v[0]),
                                        variant->upsample == MJD_UPSAMPLE_FANCY, variant->idct, ctx->cu_count, ctx->tuning,
                                        static_cast<hipStream_t>(stream));
    if (cur != ctx->device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return fail(MJD_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
    return MJD_OK;
  }
  if (nc == 3) {  // scaled: no kernel reads the workspace any more, but the call's contract stands
    if (!d_work) return fail(MJD_EINVAL, "null workspace");
    if (reinterpret_cast<uintptr_t>(d_work) % 16) return fail(MJD_EINVAL, "workspace not 16-byte aligned");
    if (work_bytes < need) return fail(MJD_EINVAL, "workspace of %llu bytes below the %llu needed",
                                       static_cast<unsigned long long>(work_bytes), static_cast<unsigned long long>(need));
  }
  int cur = 0;
  if (hipGetDevice(&cur) != hipSuccess || cur != ctx->device) {
    if (hipSetDevice(ctx->device) != hipSuccess) return fail(MJD_EDEVICE, "hipSetDevice(%d) failed", ctx->device);
  }
  const hipStream_t s = static_cast<hipStream_t>(stream);
  hipError_t e;
  if (scale > 1) {
    e = launch_scaled(*variant, g, d_coef, d_qt, d_out, static_cast<uint32_t>(pitch), s);
  } else {  // full-size grayscale (colour returned above)
    var::View v{};
    v.coef = d_coef;
    v.qt = d_qt;
    v.out = d_out;
    v.n_blocks = g.n_blocks;
    v.pitch = static_cast<uint32_t>(pitch);
    v.width = static_cast<int>(out_w);
    v.height = static_cast<int>(variant->frame.height);
    v.mcus_x = static_cast<int>(g.mcus_x);
    v.qsel = variant->frame.qsel[0];
    const AanConsts& k = aan_consts();
    switch (variant->idct) {
      case MJD_IDCT_ISLOW: e = var::launch_gray<MJD_IDCT_ISLOW>(v, k, s); break;
      case MJD_IDCT_IFAST: e = var::launch_gray<MJD_IDCT_IFAST>(v, k, s); break;
      default: e = var::launch_gray<MJD_IDCT_FLOAT>(v, k, s); break;
    }
  }
  if (cur != ctx->device) (void)hipSetDevice(cur);
  if (e != hipSuccess) return fail(MJD_EDEVICE, "kernel launch failed: %s", hipGetErrorString(e));
  return MJD_OK;
}

}  // extern "C"
