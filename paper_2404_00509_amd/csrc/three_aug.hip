// Gaussian blur and colour jitter of the finetuning augmentation "3 Aug" / "3 Aug+" (Sec. 3 finetuning
// recipe, Sec. 4.4 "Data Augmentation", Sec. 5.2 Table 7).  Per image one of grayscale / solarisation /
// Gaussian blur is drawn; the first two are pointwise and run as the epilogue of the resampling
// kernel, which leaves the rounded 8-bit resized crop of the blur images in patch order
// ([B, L, D] bytes, the layout of `target`), and with "3 Aug+" also those of the others, after their
// operation.  aug_blur_kernel blurs the former, applies the colour jitter of "3 Aug+", normalises and
// writes `target` / `visible`; aug_jitter_kernel, at the end of the file, does the same for the
// others without the blur.
//
// aug_blur_band_kernel, for patches of 16 and 32 pixels: on the matrix cores (see there).
// aug_blur_kernel, for other even patch sizes: one workgroup per image, row of patches and column part of
// whole patches; it leaves at once when its image drew another operation.
//  * Staging.  The bytes of the part's rows and of R more rows above and below, over the part's
//    patches and the neighbouring patch on either side, are copied into LDS in image order (all
//    loads of a thread issued before the first is stored).  Rows beyond the image repeat its
//    border row.
//  * Vertical pass.  A thread takes one value column and a run of rows: it converts the bytes it
//    needs once and applies the 2 R + 1 taps to each row of its run; columns beyond the image
//    repeat the border column.  The result (fp32) goes to a second LDS array with R pixels more
//    on either side of the part.
//  * Horizontal pass, folded into the walk over the part in output order: a lane reads the
//    4 + 2 R pixels around its four with aligned 16-byte LDS reads and applies the taps.
// R is the smallest of 2, 4, 6 that holds the image's radius ceil(3 sigma), so that an image with
// a small sigma does not pay for 13 taps.  The taps themselves come with the image's draws from
// the parameter kernel (one record per image) and sit in scalar registers.
// The contrast step needs the mean luma of the whole image after the brightness step: with jitter
// on, a first launch of the same kernel (kReduce) only accumulates that sum per part in double
// precision, and the second launch adds the partial sums of its image in fixed order.  Where the
// brightness factor is at most 1 nothing is clamped and the blur is linear: the sum is then one over the
// bytes (band_luma_sum).
#include "aug_device.hpp"
#include "mae_device.hpp"
#include "mae_kernels.hpp"

namespace mae {

constexpr int kAugThreads = 256;
constexpr int kMaxRadius = 6;  // ceil(3 * 2.0)

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_a4 __attribute__((aligned(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef u32x3 u32x3_a4 __attribute__((aligned(4)));

// A lane's kPx neighbouring pixels are 3 kPx floats = three pieces of kPx floats.
template <int kPx>
struct BlurPiece;
template <>
struct BlurPiece<4> {
  typedef f32x4 type;
};
template <>
struct BlurPiece<2> {
  typedef f32x2 type;
};

// floor(n / d) for 0 <= n < 2^22 and small d, from the float reciprocal (inv = 1 / d)
__device__ static inline int fast_div(int n, float inv) { return (int)(((float)n + 0.5f) * inv); }

// Mean luma after the brightness step, from the partial sums of the reduction launch.
__device__ static inline float image_mean(const AugArgs& a, int b) {
  // one slot per (row of patches, column part of the blur kernel); unused slots hold zero
  const int slots = a.G * a.blur_parts;
  double sum = 0.0;
  for (int g = 0; g < slots; ++g) sum += a.partials[(int64_t)b * slots + g];
  return (float)(sum / ((double)a.S * (double)a.S));
}

// Sum over the workgroup in a fixed order (lanes by butterfly, wavefronts in index order).
template <int kThreads>
__device__ static inline void store_band_sum(const AugArgs& a, int b, int slot, float lsum,
                                             double* red) {
  double s = (double)lsum;
  for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
  const int tid = threadIdx.x;
  if ((tid % kWave) == 0) red[tid / kWave] = s;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    for (int w = 0; w < kThreads / kWave; ++w) t += red[w];
    a.partials[(int64_t)b * a.G * a.blur_parts + slot] = t;
  }
}

// ---- Gaussian blur ---------------------------------------------------------------------------------
// Patches staged on either side of the part: enough for the largest radius.
__host__ __device__ static inline int halo_patches(int p) { return (kMaxRadius + p - 1) / p; }

// Copies `rows` image rows (first y_first, clamped into the image) of patches gxa .. gxa + nseg - 1
// from the patch-order bytes `img` into `dst` in image order, in pieces of type T (wseg pieces per
// patch row).  A wavefront takes whole rows, a lane one piece of the row, so that everything that
// depends on the row is the same for all lanes and a piece costs one address addition; a lane
// issues four loads (four rows) before it stores the first.
template <typename T>
__device__ static inline void stage_rows(uint8_t* dst, const uint8_t* img, int rows, int nseg,
                                         int wseg, int y_first, int S, int p, int G, int gxa,
                                         int D) {
  T* out = reinterpret_cast<T*>(dst);
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int pitch = nseg * wseg;
  const float inv_wseg = 1.0f / (float)wseg, inv_p = 1.0f / (float)p;
  constexpr int kBatch = 4, kWaves = kAugThreads / kWave;
  for (int l0 = 0; l0 < pitch; l0 += kWave) {
    const bool have = l0 + lane < pitch;
    const int l = have ? l0 + lane : pitch - 1;
    const int seg = fast_div(l, inv_wseg);
    const uint32_t piece = (uint32_t)(__mul24(gxa + seg, D) + (int)sizeof(T) * (l - seg * wseg));
    for (int j0 = wave; j0 < rows; j0 += kBatch * kWaves) {
      T v[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = min(j0 + u * kWaves, rows - 1);
        const int yy = min(max(y_first + j, 0), S - 1);
        const int gyy = fast_div(yy, inv_p);
        const uint32_t row = (uint32_t)(__mul24(__mul24(gyy, G), D) + (yy - gyy * p) * 3 * p);
        v[u] = *reinterpret_cast<const T*>(img + (row + piece));
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int j = j0 + u * kWaves;
        if (j < rows && have) out[j * pitch + l] = v[u];
      }
    }
  }
}

// Vertical pass: kRows output rows of one value column per item.
template <int R, int kRows>
__device__ static inline void blur_vertical(const uint8_t* sbytes, float* vbuf, const float* wt,
                                            int p, int S, int x_lo, int xs0, int Wp, int pitchb,
                                            int vpitch) {
  const int ncols = (Wp + 2 * R) * 3;
  const int chunks = p / kRows;
  for (int it = threadIdx.x; it < ncols * chunks; it += kAugThreads) {
    const int yc = fast_div(it, 1.0f / (float)ncols);
    const int vx = it - yc * ncols;
    const int px = fast_div(vx, 1.0f / 3.0f);
    const int c = vx - 3 * px;
    const int xa = min(max(x_lo - R + px, 0), S - 1);  // border column repeated
    // (32-bit offsets, stepped row by row: no multiplication per row)
    uint32_t at = (uint32_t)(__mul24(yc * kRows, pitchb) + (xa - xs0) * 3 + c);
    float in[kRows + 2 * R];
#pragma unroll
    for (int j = 0; j < kRows + 2 * R; ++j) {
      in[j] = (float)sbytes[at];
      at += (uint32_t)pitchb;
    }
#pragma unroll
    for (int y = 0; y < kRows; ++y) {
      float acc = 0.f;
#pragma unroll
      for (int k = 0; k <= 2 * R; ++k) acc += wt[k] * in[y + k];
      vbuf[(yc * kRows + y) * vpitch + vx] = acc;
    }
  }
}

// kPx: pixels per lane in the horizontal pass, 4 when p is a multiple of 4, else 2 (p even).
template <int R, bool kReduce, bool kBf16, int kPx>
__device__ static void blur_part(const AugArgs& a, const AugParams& ap, int b, int gy, int part,
                                 int gx0, int npatch, float* vbuf, uint8_t* scratch,
                                 double* red) {
  typedef typename BlurPiece<kPx>::type piece_t;
  constexpr int kVals = 3 * kPx;
  const int S = a.S, p = a.p, G = a.G;
  const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
  const int Wp = npatch * p, x_lo = gx0 * p, y0 = gy * p;
  const int hp = halo_patches(p);
  const int gxa = max(gx0 - hp, 0), gxb = min(gx0 + npatch - 1 + hp, G - 1);
  const int nseg = gxb - gxa + 1, xs0 = gxa * p;
  const int pitchb = nseg * 3 * p;  // bytes per staged row
  const int rows = p + 2 * R;
  const float inv_p = 1.0f / (float)p;
  const uint8_t* img = a.u8 + (int64_t)b * a.L * a.D;  // patch order

  // ---- staging: rows y0 - R .. y0 + p - 1 + R (clamped), patches gxa .. gxb ----------------------
  // in pieces of 16 bytes when a patch row is a multiple of that (p = 16, 32), else of 4 bytes,
  // else (p even, no multiple of 4) of 2 bytes
  if constexpr (kPx == 4) {
    if ((p & 15) == 0)
      stage_rows<u32x4>(scratch, img, rows, nseg, (3 * p) >> 4, y0 - R, S, p, G, gxa, a.D);
    else
      stage_rows<uint32_t>(scratch, img, rows, nseg, (3 * p) >> 2, y0 - R, S, p, G, gxa, a.D);
  } else {
    stage_rows<uint16_t>(scratch, img, rows, nseg, (3 * p) >> 1, y0 - R, S, p, G, gxa, a.D);
  }
  // taps -R .. R of this image's kernel as the parameter kernel left them (zero beyond the
  // image's radius); the record is the same for the whole workgroup
  float wt[2 * R + 1];
#pragma unroll
  for (int k = 0; k <= 2 * R; ++k) wt[k] = ap.tap[k < R ? R - k : k - R];
  __syncthreads();

  const int vpitch = (Wp + 2 * R) * 3;  // a multiple of kPx floats
  if constexpr (kPx == 4) {
    if ((p & 7) == 0)
      blur_vertical<R, 8>(scratch, vbuf, wt, p, S, x_lo, xs0, Wp, pitchb, vpitch);
    else
      blur_vertical<R, 4>(scratch, vbuf, wt, p, S, x_lo, xs0, Wp, pitchb, vpitch);
  } else {
    blur_vertical<R, 2>(scratch, vbuf, wt, p, S, x_lo, xs0, Wp, pitchb, vpitch);
  }
  // noise rank of each patch of the part, one per lane (read back with a shuffle at the stores)
  const int l0 = gy * G + gx0;
  const int my_rank = lane < npatch ? a.ids_restore[(int64_t)b * a.L + l0 + lane] : 0x7fffffff;
  __syncthreads();  // the staged bytes are dead from here on: their space serves as the strips

  const float mean = (!kReduce && a.mode == 2) ? image_mean(a, b) : 0.0f;
  const int gpp = (p * p) / kPx;
  const float inv_gpp = 1.0f / (float)gpp;
  const int ngroups = npatch * gpp;
  float* strip = reinterpret_cast<float*>(scratch) + wave * (kWave * kVals);
  float* target_image = a.target ? a.target + (int64_t)b * a.L * a.D : nullptr;
  void* visible_image =
      kBf16 ? static_cast<void*>(static_cast<uint16_t*>(a.visible) + (int64_t)b * a.K * a.D)
            : static_cast<void*>(static_cast<float*>(a.visible) + (int64_t)b * a.K * a.D);
  // one piece of a patch row of `target` / `visible` (element offsets inside the image)
  auto store_piece = [&](uint32_t target_off, int rank, uint32_t visible_off, piece_t t) {
    if (a.target) *reinterpret_cast<piece_t*>(target_image + target_off) = t;
    if (rank < a.K) {
      if (kBf16) {
        uint16_t* dst = static_cast<uint16_t*>(visible_image) + visible_off;
        if constexpr (kPx == 4)
          *reinterpret_cast<u32x2*>(dst) = u32x2{pack_bf16x2(t[0], t[1]), pack_bf16x2(t[2], t[3])};
        else
          *reinterpret_cast<uint32_t*>(dst) = pack_bf16x2(t[0], t[1]);
      } else {
        *reinterpret_cast<piece_t*>(static_cast<float*>(visible_image) + visible_off) = t;
      }
    }
  };
  float lsum = 0.0f;
  // patches of 16 x 16 or 32 x 32 pixels: the 64 groups of a wavefront's step lie in one patch
  const bool whole = kPx == 4 && (p & 15) == 0;
  const int gsh = __builtin_ctz(gpp), psh = __builtin_ctz(p);  // used when `whole`
  for (int i0 = wave * kWave; i0 < ngroups; i0 += kAugThreads) {
    bool have;
    int gxl, q, py;
    if (whole) {
      have = true;
      gxl = i0 >> gsh;  // uniform
      q = 4 * ((i0 & (gpp - 1)) + lane);
      py = q >> psh;
    } else {
      have = i0 + lane < ngroups;
      const int i = have ? i0 + lane : ngroups - 1;
      gxl = fast_div(i, inv_gpp);
      q = kPx * (i - gxl * gpp);
      py = fast_div(q, inv_p);
    }
    const int x = gxl * p + (q - py * p);  // pixel inside the part
    // pixels x - R .. x + kPx - 1 + R of the row: (kPx + 2 R) * 3 floats, aligned to a piece
    constexpr int kIn = (kPx + 2 * R) * 3;
    const piece_t* src = reinterpret_cast<const piece_t*>(vbuf + py * vpitch + 3 * x);
    float n[kIn];
#pragma unroll
    for (int j = 0; j < kIn / kPx; ++j) {
      const piece_t t = src[j];
#pragma unroll
      for (int e = 0; e < kPx; ++e) n[kPx * j + e] = t[e];
    }
    float v[kVals];
#pragma unroll
    for (int h = 0; h < kPx; ++h) {
      float r = 0.f, g = 0.f, bl = 0.f;
#pragma unroll
      for (int k = 0; k <= 2 * R; ++k) {
        r += wt[k] * n[3 * (h + k)];
        g += wt[k] * n[3 * (h + k) + 1];
        bl += wt[k] * n[3 * (h + k) + 2];
      }
      v[3 * h] = r;
      v[3 * h + 1] = g;
      v[3 * h + 2] = bl;
      if (a.mode == 2) {
        const float lum = jitter_pixel<kReduce>(ap, mean, v[3 * h], v[3 * h + 1], v[3 * h + 2]);
        lsum += have ? lum : 0.0f;
      }
    }
    if (kReduce) continue;

    // normalise, then through the wavefront's strip: every store instruction writes 1 KiB (512
    // bytes with two pixels per lane) of contiguous memory; piece k of the strip belongs to
    // group k / 3
    piece_t o[3];
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
      for (int e = 0; e < kPx; ++e) {
        const int idx = kPx * k + e;
        o[k][e] = v[idx] * a.nscale[idx % 3] + a.nbias[idx % 3];
      }
    piece_t* mine = reinterpret_cast<piece_t*>(strip + kVals * lane);
    __builtin_amdgcn_wave_barrier();
    mine[0] = o[0];
    mine[1] = o[1];
    mine[2] = o[2];
    __builtin_amdgcn_wave_barrier();
    if (whole) {
      // one patch, 768 consecutive floats of its row from element 12 (i0 mod gpp) on
      const int gxs = __builtin_amdgcn_readfirstlane(gxl);
      const int rank = __builtin_amdgcn_readlane(my_rank, gxs);
      const uint32_t e0 = 12u * (uint32_t)(i0 & (gpp - 1)) + 4u * (uint32_t)lane;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const piece_t t = reinterpret_cast<const piece_t*>(strip)[k * kWave + lane];
        const uint32_t eo = e0 + 4u * kWave * k;
        store_piece((uint32_t)((l0 + gxs) * a.D) + eo, rank, (uint32_t)(rank * a.D) + eo, t);
      }
      continue;
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int piece = k * kWave + lane;
      const int g = i0 + fast_div(piece, 1.0f / 3.0f);
      const piece_t t = reinterpret_cast<const piece_t*>(strip)[piece];
      const int pgx = fast_div(min(g, ngroups - 1), inv_gpp);
      const int rank = __shfl(my_rank, pgx, kWave);
      if (g >= ngroups) continue;
      const int eo = kVals * (g - __mul24(pgx, gpp)) + kPx * (piece - 3 * (g - i0));
      store_piece((uint32_t)(__mul24(l0 + pgx, a.D) + eo), rank,
                  (uint32_t)(__mul24(rank, a.D) + eo), t);
    }
  }
  if (kReduce) store_band_sum<kAugThreads>(a, b, gy * a.blur_parts + part, lsum, red);
}

// Dynamic LDS: [ vbuf: p rows of 3 (W + 12) floats, W = widest part in pixels | scratch: the
// staged bytes ((p + 12) rows of the part's patches and their neighbours), later the four
// wavefronts' strips ].
template <bool kReduce, bool kBf16, int kPx>
__global__ __launch_bounds__(kAugThreads) void aug_blur_kernel(AugArgs a) {
  extern __shared__ __attribute__((aligned(16))) float vals[];
  __shared__ double red[kAugThreads / kWave];

  const int p = a.p, G = a.G, parts = a.blur_parts;
  const uint32_t tile = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t band_id = tile / (uint32_t)parts;
  const int part = (int)(tile - band_id * (uint32_t)parts);
  const int b = (int)(band_id / (uint32_t)G);
  const int gy = (int)(band_id - (uint32_t)b * (uint32_t)G);
  const int gx0 = part * G / parts, gx1 = (part + 1) * G / parts;
  const int npatch = gx1 - gx0;
  const bool valid = reinterpret_cast<const CropRec*>(a.workspace + kWorkspaceHeader)[b].valid != 0;
  if (!valid || npatch <= 0) return;
  const AugParams ap = static_cast<const AugParams*>(a.aug_recs)[b];
  if (ap.op != kOpBlur) return;

  const int radius = ap.radius;
  float* vbuf = vals;
  uint8_t* scratch = reinterpret_cast<uint8_t*>(
      vals + p * 3 * (a.blur_part_patches * p + 2 * kMaxRadius));
  if (radius <= 2)
    blur_part<2, kReduce, kBf16, kPx>(a, ap, b, gy, part, gx0, npatch, vbuf, scratch, red);
  else if (radius <= 4)
    blur_part<4, kReduce, kBf16, kPx>(a, ap, b, gy, part, gx0, npatch, vbuf, scratch, red);
  else
    blur_part<6, kReduce, kBf16, kPx>(a, ap, b, gy, part, gx0, npatch, vbuf, scratch, red);
}

// ---- Gaussian blur on the matrix cores ----------------------------------------------------------------
// Patches whose side is a multiple of 16 (16 and 32).  Both passes are products with a band matrix of
// taps (v_mfma_f32_16x16x32_bf16), so the vector ALUs, which bound the kernel above at 26 multiply-adds
// per value, are left with the operands' conversion and the epilogue.  Nothing is lost by the 16-bit
// operands: a byte is exact in bf16, a tap is the sum of three bf16 values of 8 bits each, and so is,
// to its last bit or half of it, a value between the passes.  All products of the parts that reach 2^-24
// of the result are taken, the smallest first, and added in fp32.
// (The fp32 form of the instruction, v_mfma_f32_16x16x4f32, needs no parts but runs no faster than the
// vector ALUs and not beside them: 355 us for the outputs and 267 for all sums of the launch below.)
//
// A wavefront takes 16 rows of an image, or a part of them, and walks along x in steps of 16 pixels;
// nothing is shared, so there is no barrier and no LDS.
//  * Vertical: V[x, y] = sum over 32 rows r of X[x, r] T[r, y], a channel at a time, for the 16 pixels from
//    16 j - 8 on.  The rows come straight from memory: lane (x, g) loads the dwords that end with its
//    pixel's three bytes of rows 8 g .. 8 g + 7 (rows and columns beyond the image: the border's), the
//    next tile's while this one is multiplied.
//  * Horizontal: O[y, x] = sum over x' of V[y, x'] T[x', x] with the two tiles that hold the 16 pixels
//    and eight more on either side.  The instruction leaves V with x' = 4 g + e in register e of lane
//    group g and takes eight consecutive indices of the sum from a lane group: the registers of the two
//    tiles as they are, with the taps in the same order.
// The 16 rows go through the columns of V in the order 0, 4, 8, 12, 1, ..: a lane then ends with pixel x of
// rows g, 4 + g, 8 + g, 12 + g, and a store instruction covers four whole rows of the tile.
// 4096 images of 224 pixels ("3 Aug+", a third of them blurred): 322 us for the outputs and 125 for the luma
// sums (518 and 358 us by the kernel above); 1024 images of 160 pixels, "3 Aug": 37 us (65).  Bound by the
// vector instructions of the epilogue and of the splits, and by the stores (0.8 GB).
typedef uint32_t u32_a1 __attribute__((aligned(1)));
typedef float f32x3 __attribute__((ext_vector_type(3)));
typedef f32x3 f32x3_a4 __attribute__((aligned(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
constexpr int kBandRows = 16;

// Pairs of values as three pairs of bf16 that add up to them.
__device__ static inline void split3(float x, float y, uint32_t& hi, uint32_t& mid, uint32_t& lo) {
  hi = pack_bf16x2(x, y);
  x -= bf16_lo(hi);
  y -= bf16_hi(hi);
  mid = pack_bf16x2(x, y);
  lo = pack_bf16x2(x - bf16_lo(mid), y - bf16_hi(mid));
}
__device__ static inline f32x4 mfma_bf16(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// A wavefront's rows of an image's bytes (patch order): the lane's pixel 16 j + shift + lane % 16 of kRows
// rows, row i of which is first + stride i, as dwords whose upper three bytes are its channels.
template <int kRows>
struct BandPixels {
  const uint8_t* img;
  uint32_t row[kRows];
  int psh, p, D, S, shift;
  __device__ inline void open(const AugArgs& a, int b, int first, int stride, int shift_) {
    p = a.p;
    psh = __builtin_ctz(p);  // (16 or 32)
    D = a.D;
    S = a.S;
    shift = shift_ + (int)(threadIdx.x & 15);
    img = a.u8 + (int64_t)b * a.L * D - 1;  // (the workspace begins further in front)
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
      const int y = min(max(first + stride * i, 0), S - 1);
      row[i] = (uint32_t)((y >> psh) * a.G * D + (y & (p - 1)) * 3 * p);
    }
  }
  __device__ inline void load(int j, uint32_t* px) const {
    const int x = min(max(16 * j + shift, 0), S - 1);
    const uint32_t column = (uint32_t)((x >> psh) * D + (x & (p - 1)) * 3);
#pragma unroll
    for (int i = 0; i < kRows; ++i) px[i] = *reinterpret_cast<const u32_a1*>(img + (row[i] + column));
  }
};
__device__ static inline float channel_of(uint32_t px, int c) {
  return (float)((px >> (8 * c + 8)) & 0xFFu);
}

__device__ static inline void store_luma_sum(const AugArgs& a, int b, int slot, float lsum) {
  double sum = (double)lsum;  // lanes by butterfly
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
  if (threadIdx.x % kWave == 0)
    a.partials[(int64_t)b * (a.S / kBandRows) * a.band_parts + slot] = sum;
}

// The luma sum after the brightness step where nothing is clamped by it (a factor of at most 1): the blur
// is linear, so the sum over the blurred image is one over the bytes, weighted with what every pixel
// contributes: the sum of the taps in x and in y, of which those beyond the border fall to its pixel.
__device__ static void band_luma_sum(const AugArgs& a, const AugParams& ap, int b, int y0, int tile0,
                                     int tile1, int slot) {
  const int lane = threadIdx.x % kWave, g = lane >> 4;
  const float taps = static_cast<const AugParams*>(a.aug_recs)[b].tap[lane & 7];
  float half = 0.0f, near = 0.0f, edge = 0.0f;  // taps 0 .. 6; 1 .. lane; sum of (d + 1) tap[d]
#pragma unroll
  for (int d = 0; d <= kMaxRadius; ++d) {
    const float t = __shfl(taps, d, kWave);
    half += t;
    near += d >= 1 && d <= lane ? t : 0.0f;
    edge += (float)(d + 1) * t;
  }
  // lane q: the weight of a pixel q pixels off the nearest border (6: or more)
  const float weights = lane == 0 ? edge : half + near;
  const auto weight = [&](int at) { return __shfl(weights, min(min(at, a.S - 1 - at), kMaxRadius), kWave); };
  BandPixels<4> rows;
  rows.open(a, b, y0 + g, 4, 0);
  float wy[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) wy[e] = weight(y0 + 4 * e + g);
  float lsum = 0.0f;
  uint32_t px[4], next[4];
  rows.load(tile0, px);
  for (int j = tile0; j < tile1; ++j) {
    rows.load(min(j + 1, tile1 - 1), next);
    const float wx = weight(16 * j + (lane & 15));
    float sum = 0.0f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sum += wy[e] * luma(channel_of(px[e], 0), channel_of(px[e], 1), channel_of(px[e], 2));
      px[e] = next[e];
    }
    lsum += wx * sum;
  }
  store_luma_sum(a, b, slot, lsum * ap.brightness);
}

template <bool kReduce, bool kBf16>
__device__ static void blur_band(const AugArgs& a, const AugParams& ap, int b, int y0, int tile0,
                                 int tile1, int slot) {
  const int lane = threadIdx.x % kWave, lx = lane & 15, g = lane >> 4;
  const int S = a.S, p = a.p, D = a.D;
  const int psh = __builtin_ctz(p);
  BandPixels<8> rows;
  rows.open(a, b, y0 - 8 + 8 * g, 1, -8);
  uint32_t px[8];
  rows.load(tile0, px);

  const float taps = static_cast<const AugParams*>(a.aug_recs)[b].tap[lane & 7];
  const auto tap = [&](int d) { return __shfl(taps, min(abs(d), 7), kWave); };  // ([7] is zero)
  u32x4 tv[3], th[3];  // parts of the vertical and the horizontal taps
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int dy = 2 * i + 8 * g - 8 - (4 * (lx & 3) + (lx >> 2));
    const int dx = (i < 2 ? 2 * i - 8 : 2 * i + 4) + 4 * g - lx;
    uint32_t hi, mid, lo;
    split3(tap(dy), tap(dy + 1), hi, mid, lo);
    tv[0][i] = hi;
    tv[1][i] = mid;
    tv[2][i] = lo;
    split3(tap(dx), tap(dx + 1), hi, mid, lo);
    th[0][i] = hi;
    th[1][i] = mid;
    th[2][i] = lo;
  }

  // noise rank of the patch of tile (tile0 + lane), and the mean luma after the brightness step
  const int l0 = (y0 >> psh) * a.G;
  const int my_tile = min(tile0 + lane, tile1 - 1);
  const int my_rank =
      kReduce ? 0 : a.ids_restore[(int64_t)b * a.L + l0 + ((16 * my_tile) >> psh)];
  float mean = 0.0f;
  if (!kReduce && a.mode == 2) {
    const int slots = (S / kBandRows) * a.band_parts;
    double sum = 0.0;
    for (int i = lane; i < slots; i += kWave) sum += a.partials[(int64_t)b * slots + i];
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_xor(sum, off, kWave);
    mean = (float)(sum / ((double)S * (double)S));
  }

  float* target_image = a.target ? a.target + (int64_t)b * a.L * D : nullptr;
  const int64_t visible_base = (int64_t)b * a.K * D;
  const uint32_t in_patch_row = (uint32_t)((y0 & (p - 1)) + g) * (uint32_t)(3 * p) + 3u * (uint32_t)lx;
  float lsum = 0.0f;
  // parts of V, the two tiles of the horizontal pass: [channel][part], registers 0, 1 the left tile's
  u32x4 v[3][3];
  for (int j = tile0; j <= tile1; ++j) {
    f32x4 cur[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      u32x4 x;
#pragma unroll
      for (int i = 0; i < 4; ++i)  // (whole numbers below 256: the upper halves of the floats)
        x[i] = __builtin_amdgcn_perm(__float_as_uint(channel_of(px[2 * i + 1], c)),
                                     __float_as_uint(channel_of(px[2 * i], c)), 0x07060302u);
      cur[c] = f32x4{0.f, 0.f, 0.f, 0.f};
      cur[c] = mfma_bf16(x, tv[2], cur[c]);
      cur[c] = mfma_bf16(x, tv[1], cur[c]);
      cur[c] = mfma_bf16(x, tv[0], cur[c]);
    }
    if (j < tile1) rows.load(j + 1, px);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
#pragma unroll
      for (int part = 0; part < 3; ++part) {
        v[c][part][0] = v[c][part][2];
        v[c][part][1] = v[c][part][3];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        uint32_t hi, mid, lo;
        split3(cur[c][2 * i], cur[c][2 * i + 1], hi, mid, lo);
        v[c][0][2 + i] = hi;
        v[c][1][2 + i] = mid;
        v[c][2][2 + i] = lo;
      }
    }
    if (j == tile0) continue;
    f32x4 out[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      out[c] = f32x4{0.f, 0.f, 0.f, 0.f};
      out[c] = mfma_bf16(v[c][2], th[0], out[c]);
      out[c] = mfma_bf16(v[c][0], th[2], out[c]);
      out[c] = mfma_bf16(v[c][1], th[1], out[c]);
      out[c] = mfma_bf16(v[c][1], th[0], out[c]);
      out[c] = mfma_bf16(v[c][0], th[1], out[c]);
      out[c] = mfma_bf16(v[c][0], th[0], out[c]);
    }
    const int tile = j - 1;
    const int rank = __builtin_amdgcn_readlane(my_rank, tile - tile0);
    const int l = l0 + ((16 * tile) >> psh);
    const uint32_t at0 = in_patch_row + (uint32_t)(3 * ((16 * tile) & (p - 1)));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float v0 = out[0][e], v1 = out[1][e], v2 = out[2][e];
      if (a.mode == 2) {
        const float lum = jitter_pixel<kReduce>(ap, mean, v0, v1, v2);
        lsum += lum;
      }
      if constexpr (!kReduce) {
        v0 = v0 * a.nscale[0] + a.nbias[0];
        v1 = v1 * a.nscale[1] + a.nbias[1];
        v2 = v2 * a.nscale[2] + a.nbias[2];
        const uint32_t at = at0 + (uint32_t)(12 * e * p);
        if (a.target)
          *reinterpret_cast<f32x3_a4*>(target_image + ((uint32_t)(l * D) + at)) = f32x3{v0, v1, v2};
        if (rank < a.K) {
          const int64_t vo = visible_base + ((uint32_t)(rank * D) + at);
          if constexpr (kBf16) {
            // two pixels are three dwords: two from the left one's lane, one from the right one's
            const float next = __uint_as_float((uint32_t)__builtin_amdgcn_mov_dpp(
                (int)__float_as_uint(v0), 0xF5 /* quad_perm 1, 1, 3, 3 */, 0xF, 0xF, true));
            uint16_t* dst = static_cast<uint16_t*>(a.visible) + vo;
            if (lane & 1)
              *reinterpret_cast<uint32_t*>(dst + 1) = pack_bf16x2(v1, v2);
            else
              *reinterpret_cast<u32x2_a4*>(dst) = u32x2{pack_bf16x2(v0, v1), pack_bf16x2(v2, next)};
          } else {
            *reinterpret_cast<f32x3_a4*>(static_cast<float*>(a.visible) + vo) = f32x3{v0, v1, v2};
          }
        }
      }
    }
  }
  if constexpr (kReduce) store_luma_sum(a, b, slot, lsum);
}

template <bool kReduce, bool kBf16>
__global__ __launch_bounds__(kAugThreads) void aug_blur_band_kernel(AugArgs a, int parts) {
  const int bands = a.S / kBandRows, slots = bands * parts;
  const uint32_t task = xcd_remap(blockIdx.x, gridDim.x) * (kAugThreads / kWave) +
                        (uint32_t)__builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int b = (int)(task / (uint32_t)slots);
  if (b >= a.B) return;
  const int slot = (int)(task - (uint32_t)b * (uint32_t)slots);
  const bool valid = reinterpret_cast<const CropRec*>(a.workspace + kWorkspaceHeader)[b].valid != 0;
  if (!valid) return;
  const AugParams ap = static_cast<const AugParams*>(a.aug_recs)[b];
  if (ap.op != kOpBlur) return;
  const int band = slot / parts, part = slot - band * parts;
  const int tile0 = part * bands / parts, tile1 = (part + 1) * bands / parts;  // (as many tiles as bands)
  if (tile0 == tile1) {
    if (kReduce && threadIdx.x % kWave == 0) a.partials[(int64_t)b * slots + slot] = 0.0;
    return;
  }
  if (kReduce && ap.brightness <= 1.0f)
    band_luma_sum(a, ap, b, band * kBandRows, tile0, tile1, slot);
  else
    blur_band<kReduce, kBf16>(a, ap, b, band * kBandRows, tile0, tile1, slot);
}

// Bytes of dynamic LDS of the blur kernel for parts of n patches: the vertically blurred rows,
// then the staged bytes (or the four wavefronts' strips, whichever is larger).
static size_t blur_lds_bytes(int p, int n) {
  const size_t vbuf = (size_t)p * 3 * (n * p + 2 * kMaxRadius) * 4;
  const size_t staged = (size_t)(p + 2 * kMaxRadius) * (n + 2 * halo_patches(p)) * 3 * p;
  const size_t strips = (size_t)kAugThreads * 12 * 4;
  return vbuf + (staged > strips ? staged : strips);
}

// Column parts of the blur kernel: the fewest (whole patches each) whose LDS stays within 40 KiB,
// so that four workgroups share a compute unit.
AugPlan three_aug_plan(int S, int p) {
  const int G = S / p;
  AugPlan plan;
  for (int parts = 1;; ++parts) {
    const int n = (G + parts - 1) / parts;
    const size_t lds = blur_lds_bytes(p, n);
    if (lds <= 40 * 1024 || parts >= G) {
      plan.parts = parts;
      plan.part_patches = n;
      plan.lds_bytes = lds;
      return plan;
    }
  }
}

// Column parts of a band of the matrix kernel, by the size of the image alone: the same for every batch, as an
// image's sum is added up in the same order in a batch and in a shard of it.  Patches of 16: eight tiles in a
// part or fewer; of 32: four or five, of which eight as well take longer (calls of "3 Aug+", 600 images -> 128
// 96.8 -> 107.6 us, 150 -> 256 83 -> 92, 64 -> 224 50.1 -> 52.0; nothing gets faster by it).
int blur_band_parts(int S, int p) { return p == 16 ? (S + 127) / 128 : max(1, S / 64); }
// Luma sums per image: one per row of patches and column part, or per band and its part.
int blur_luma_slots(int S, int p) {
  return (p & 15) == 0 ? S / kBandRows * blur_band_parts(S, p) : S / p * three_aug_plan(S, p).parts;
}

// The blur images of a batch.  reduce: only the luma sums after the brightness step ("3 Aug+").
hipError_t launch_aug_blur(const AugArgs& a, bool reduce, hipStream_t stream) {
  dim3 block(kAugThreads);
  if ((a.p & 15) == 0) {
    // (outputs: whole bands where they fill the chip, as a part has one more tile of V to make; as many
    // parts as give every SIMD a wavefront, of a third of the images, where they do not: calls of
    // "3 Aug", 192 pixels, bf16, 16 images: 24.5 -> 20.6 us, 100 images 38.9 -> 35.9)
    const int bands = a.S / kBandRows;
    int parts = a.band_parts;
    if (!reduce && (int64_t)a.B * bands >= 12288) parts = 1;
    while (!reduce && 2 * parts <= bands && (int64_t)a.B * bands * parts < 3072) parts *= 2;
    const uint64_t tasks = (uint64_t)a.B * (uint64_t)(bands * parts);
    constexpr int kPerBlock = kAugThreads / kWave;
    dim3 grid((uint32_t)((tasks + kPerBlock - 1) / kPerBlock));
    if (reduce)
      hipLaunchKernelGGL((aug_blur_band_kernel<true, false>), grid, block, 0, stream, a, parts);
    else if (a.visible_bf16)
      hipLaunchKernelGGL((aug_blur_band_kernel<false, true>), grid, block, 0, stream, a, parts);
    else
      hipLaunchKernelGGL((aug_blur_band_kernel<false, false>), grid, block, 0, stream, a, parts);
    return hipGetLastError();
  }
  dim3 bgrid((uint32_t)a.B * (uint32_t)a.G * (uint32_t)a.blur_parts);
  const size_t lds = blur_lds_bytes(a.p, a.blur_part_patches);
  // four pixels per lane when they tile a patch row, else two (even patch sizes)
#define MAE_BLUR_LAUNCH(RED, BF)                                                           \
  do {                                                                                     \
    if ((a.p & 3) == 0)                                                                    \
      hipLaunchKernelGGL((aug_blur_kernel<RED, BF, 4>), bgrid, block, lds, stream, a);     \
    else                                                                                   \
      hipLaunchKernelGGL((aug_blur_kernel<RED, BF, 2>), bgrid, block, lds, stream, a);     \
  } while (0)
  if (reduce) MAE_BLUR_LAUNCH(true, false);
  else if (a.visible_bf16) MAE_BLUR_LAUNCH(false, true);
  else MAE_BLUR_LAUNCH(false, false);
#undef MAE_BLUR_LAUNCH
  return hipGetLastError();
}

// ---- colour jitter of the images without the blur ("3 Aug+") -----------------------------------------
// The resampling kernel has left these images' bytes (operation applied, patch order) and their luma
// sums; here they are jittered, normalised and written.  A pointwise stream: 1 byte in, 4 out (8
// with a target) per value, bound by HBM.  Groups of four consecutive pixels of a patch row of bytes
// are dealt to the lanes (p even: a patch is a whole number of them), a wavefront has kJitterRuns
// loads of 768 contiguous bytes in flight, and the values go through its strip of LDS so that every
// store covers 1 KiB of contiguous memory.  4096 images of 224 pixels, tokens only: the call takes
// 1.72 ms; with a second run of the resampling kernel (0.49 ms, bound by vector instructions) in
// this one's place it took 1.82 ms.
constexpr int kJitterRuns = 4;   // loads in flight per wavefront
constexpr int kJitterSteps = 8;  // runs of 64 groups per wavefront of a workgroup

template <bool kBf16>
__global__ __launch_bounds__(kAugThreads) void aug_jitter_kernel(AugArgs a, int blocks_per_image) {
  __shared__ int ranks[kMaxPatches];
  __shared__ __attribute__((aligned(16))) float strips[kAugThreads * 12];
  const uint32_t tile = xcd_remap(blockIdx.x, gridDim.x);
  const int b = (int)(tile / (uint32_t)blocks_per_image);
  const int part = (int)(tile - (uint32_t)b * (uint32_t)blocks_per_image);
  const bool valid = reinterpret_cast<const CropRec*>(a.workspace + kWorkspaceHeader)[b].valid != 0;
  if (!valid) return;  // (its neutral outputs are written by the resampling kernel)
  const AugParams ap = static_cast<const AugParams*>(a.aug_recs)[b];
  if (ap.op == kOpBlur) return;
  const int tid = threadIdx.x, lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  for (int l = tid; l < a.L; l += kAugThreads) ranks[l] = a.ids_restore[(int64_t)b * a.L + l];
  double sum = 0.0;  // in the order of the rows and parts
  for (int g = 0; g < a.luma_slots; ++g) sum += a.luma_partials[(int64_t)b * a.luma_slots + g];
  const float mean = (float)(sum / ((double)a.S * (double)a.S));
  __syncthreads();

  const int D = a.D, d4 = D >> 2;
  const float inv_d4 = 1.0f / (float)d4;
  const int ngroups = (a.S * a.S) >> 2;
  const bool gray = ap.op == kOpGray;
  const uint8_t* image = a.u8 + (int64_t)b * a.L * D;
  float* target_image = a.target ? a.target + (int64_t)b * a.L * D : nullptr;
  const int64_t visible_base = (int64_t)b * a.K * D;
  f32x4* strip = reinterpret_cast<f32x4*>(strips + wave * (kWave * 12));
  constexpr int kWaves = kAugThreads / kWave;
  const int first = part * (kJitterSteps * kAugThreads);

  for (int s0 = 0; s0 < kJitterSteps; s0 += kJitterRuns) {
    u32x3 in[kJitterRuns];
#pragma unroll
    for (int u = 0; u < kJitterRuns; ++u) {
      const int i = first + ((s0 + u) * kWaves + wave) * kWave + lane;
      in[u] = *reinterpret_cast<const u32x3_a4*>(image + 12 * (uint32_t)min(i, ngroups - 1));
    }
#pragma unroll
    for (int u = 0; u < kJitterRuns; ++u) {
      const int i0 = first + ((s0 + u) * kWaves + wave) * kWave;
      if (i0 >= ngroups) break;
      float v[12];
#pragma unroll
      for (int e = 0; e < 12; ++e) v[e] = (float)((in[u][e >> 2] >> (8 * (e & 3))) & 0xFFu);
      if (gray) {
        // equal channels stay equal under the jitter: one channel's arithmetic, and the saturation
        // step leaves it as it is (the luma weights add up to one)
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          const float g = clamp255(v[3 * h] * ap.brightness);
          v[3 * h] = v[3 * h + 1] = v[3 * h + 2] =
              clamp255(ap.contrast * g + (1.0f - ap.contrast) * mean);
        }
      } else {
#pragma unroll
        for (int h = 0; h < 4; ++h)
          jitter_pixel<false>(ap, mean, v[3 * h], v[3 * h + 1], v[3 * h + 2]);
      }
      f32x4 o[3];
#pragma unroll
      for (int e = 0; e < 12; ++e) o[e >> 2][e & 3] = v[e] * a.nscale[e % 3] + a.nbias[e % 3];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int k = 0; k < 3; ++k) strip[3 * lane + k] = o[k];
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const f32x4 t = strip[k * kWave + lane];
        const int piece = 3 * i0 + k * kWave + lane;  // four values each, inside the image
        if (piece >= 3 * ngroups) continue;
        const int l = fast_div(piece, inv_d4);
        const int rank = ranks[l];
        if (a.target) reinterpret_cast<f32x4*>(target_image)[piece] = t;
        if (rank < a.K) {
          const int64_t vo = visible_base + (uint32_t)(__mul24(rank, D) + 4 * (piece - __mul24(l, d4)));
          if (kBf16)
            *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(a.visible) + vo) =
                u32x2{pack_bf16x2(t.x, t.y), pack_bf16x2(t.z, t.w)};
          else
            *reinterpret_cast<f32x4*>(static_cast<float*>(a.visible) + vo) = t;
        }
      }
    }
  }
}

hipError_t launch_aug_jitter(const AugArgs& a, hipStream_t stream) {
  const int ngroups = (a.S * a.S) >> 2;
  const int per_block = kJitterSteps * kAugThreads;
  const int blocks = (ngroups + per_block - 1) / per_block;
  dim3 grid((uint32_t)a.B * (uint32_t)blocks), block(kAugThreads);
  if (a.visible_bf16)
    hipLaunchKernelGGL(aug_jitter_kernel<true>, grid, block, 0, stream, a, blocks);
  else
    hipLaunchKernelGGL(aug_jitter_kernel<false>, grid, block, 0, stream, a, blocks);
  return hipGetLastError();
}

}  // namespace mae
