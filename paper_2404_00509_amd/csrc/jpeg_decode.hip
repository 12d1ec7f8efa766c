// Crop decode (Sec. 4.1 "Crop Decode"): the loader's images are JPEG files, and only the region
// that the random crop needs is decoded.  Baseline sequential DCT (ITU-T T.81), 8 bits, three
// components (JFIF YCbCr), luma sampled 1x1 or 2x2 against 1x1 chroma, tables as found in the file,
// any restart interval.  The rows of MCUs above and below the crop are not transformed, a row is
// entropy-decoded only up to the crop's right edge, and the inverse transform runs only for the
// MCUs inside it.  With one restart interval per row of MCUs (a choice of the dataset writer) the
// rows are independent and those outside the crop are never touched; in any other file the
// entropy-coded data is one chain, or several that are no rows, and a first kernel walks it (symbol
// lengths only) to find where each of the crop's rows starts.
//
//  * jpeg_header_kernel: one lane per file walks the marker segments and leaves a record (size,
//    sampling, restart interval, where the tables and the entropy-coded data start) plus the
//    image's height and width for the crop-parameter kernel.
//  * jpeg_tables_kernel: one wavefront per image builds what the decoder needs and leaves it in
//    the workspace: the Huffman tables (the code ranges of Annex C plus a direct table for codes
//    of up to 10 bits), the quantiser steps in zig-zag order, the crop's rows and columns of
//    MCUs, and, for files with a restart interval per row, the restart markers (16 bytes per lane
//    and step, positions ranked with a prefix sum) = the states at which the rows start.  The
//    crop record is rewritten relative to the decoded region.
//  * jpeg_sync_kernel (files without restart markers): one wavefront per file enters the chain in
//    64 places at once and finds the states at which the crop's rows start.
//  * jpeg_scan_kernel (what is left: intervals that are no rows, files too large for the memory of
//    the parallel walk): one lane per file, two files per wavefront with their
//    tables in LDS, decodes code lengths and DC differences only, handles restart markers where
//    they come, and records the state of the bit reader and the DC predictors at the start of
//    each of the crop's rows of MCUs.
//  * jpeg_entropy_kernel: one wavefront per group of up to four images, a lane per row of MCUs that
//    a crop touches (or per piece of such a row where the parallel walk has found the pieces'
//    states); the coefficients go to the plane buffer as 16-bit values, those of 4:4:4 crops of more
//    than half a slot in part to the region buffer.
//  * jpeg_decode_kernel (what is left: restart intervals that end inside a row, and crops of the
//    whole slot with 4:4:4 sampling and more than 64 MCUs in a row): rows dealt to the lanes in the
//    same way.  A lane's file bytes come through its column of a ring in LDS that is fed at the
//    start of every block, where all lanes are at the same instruction; the bit buffer takes four
//    bytes at a time unless one of them is 0xFF.  Per block: DC difference, AC symbols with one
//    table look-up each (code and value bits out of the same 32-bit peek), de-quantisation on
//    insertion, fixed-point separable inverse DCT in LDS, eight 8-byte stores into the image's Y,
//    Cb or Cr plane.
//  * jpeg_idct_kernel: coefficients (inverse transform) or planes -> interleaved RGB rows of the
//    region (repeated chroma, fixed-point JFIF colour matrix), which is what the resampling kernel
//    reads.
//
// The integer arithmetic of the inverse DCT and of the colour conversion is part of the
// definition of the output (a decoder is only specified up to that): 13-bit cosines, first pass
// kept with 3 fractional bits, both passes' inputs clamped to +-32767, floor after adding one half.
//
// Every read of file bytes is clamped into the file, every table index is masked, and every loop
// has a fixed bound, so a corrupt file gives wrong pixels or a sample flagged invalid, nothing else.
#include "mae_device.hpp"
#include "mae_kernels.hpp"

namespace mae {

constexpr int kJpegThreads = 64;  // one wavefront per workgroup
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__constant__ uint8_t kZigzag[64] = {
    0,  1,  8,  16, 9,  2,  3,  10, 17, 24, 32, 25, 18, 11, 4,  5,  12, 19, 26, 33, 40, 48,
    41, 34, 27, 20, 13, 6,  7,  14, 21, 28, 35, 42, 49, 56, 57, 50, 43, 36, 29, 22, 15, 23,
    30, 37, 44, 51, 58, 59, 52, 45, 38, 31, 39, 46, 53, 60, 61, 54, 47, 55, 62, 63};

// C(u) cos((2x+1) u pi / 16) * 2^13 rounded, C(0) = 1/sqrt 2: row x, column u
__constant__ __attribute__((aligned(16))) int16_t kBasis[64] = {
    5793, 8035,  7568,  6811,  5793,  4551,  3135,  1598,   //
    5793, 6811,  3135,  -1598, -5793, -8035, -7568, -4551,  //
    5793, 4551,  -3135, -8035, -5793, 1598,  7568,  6811,   //
    5793, 1598,  -7568, -4551, 5793,  6811,  -3135, -8035,  //
    5793, -1598, -7568, 4551,  5793,  -6811, -3135, 8035,   //
    5793, -4551, -3135, 8035,  -5793, -1598, 7568,  -6811,  //
    5793, -6811, 3135,  1598,  -5793, 8035,  -7568, 4551,   //
    5793, -8035, 7568,  -6811, 5793,  -4551, 3135,  -1598};

__device__ static inline int be16(const uint8_t* p) { return ((int)p[0] << 8) | (int)p[1]; }

// ---- header ----------------------------------------------------------------------------------------
__global__ __launch_bounds__(kJpegThreads) void jpeg_header_kernel(JpegArgs a) {
  const int b = (int)(blockIdx.x * kJpegThreads + threadIdx.x);
  if (b >= a.B) return;
  JpegRec rec;
  memset(&rec, 0, sizeof(rec));
  int H = 1, W = 1;  // what the crop-parameter kernel sees for an unusable file
  const int64_t off = a.offsets[b];
  const int64_t n = (int64_t)a.sizes[b];
  bool ok = off >= 0 && n >= 4 && off + n <= a.files_bytes;
  if (ok) {
    const uint8_t* d = a.files + off;
    ok = d[0] == 0xFF && d[1] == 0xD8;
    int64_t pos = 2;
    bool have_frame = false, have_scan = false;
    int tq[3] = {0, 0, 0}, cid[3] = {0, 0, 0};
    int q_off[4] = {0, 0, 0, 0}, dc_off[4] = {0, 0, 0, 0}, ac_off[4] = {0, 0, 0, 0};
    for (int seg = 0; seg < 64 && ok && !have_scan; ++seg) {
      if (pos + 4 > n || d[pos] != 0xFF) {
        ok = false;
        break;
      }
      const int m = d[pos + 1];
      if (m == 0xFF) {
        ++pos;
        continue;
      }
      const int len = be16(d + pos + 2);
      if (len < 2 || pos + 2 + len > n) {
        ok = false;
        break;
      }
      const uint8_t* s = d + pos + 4;
      const int body = len - 2;
      if (m == 0xDB) {
        for (int o = 0; o + 65 <= body; o += 65) {
          const int pq = s[o] >> 4, t = s[o] & 15;
          if (pq != 0 || t > 3) {
            ok = false;
            break;
          }
          q_off[t] = (int)(pos + 4 + o + 1);
        }
      } else if (m == 0xC0) {
        if (body < 15 || s[0] != 8 || s[5] != 3) {
          ok = false;
          break;
        }
        H = be16(s + 1);
        W = be16(s + 3);
        int hs[3], vs[3];
        for (int c = 0; c < 3; ++c) {
          cid[c] = s[6 + 3 * c];
          hs[c] = s[7 + 3 * c] >> 4;
          vs[c] = s[7 + 3 * c] & 15;
          tq[c] = s[8 + 3 * c] & 3;
        }
        ok = H >= 1 && W >= 1 && hs[1] == 1 && vs[1] == 1 && hs[2] == 1 && vs[2] == 1 &&
             ((hs[0] == 1 && vs[0] == 1) || (hs[0] == 2 && vs[0] == 2));
        rec.hs = hs[0];
        have_frame = true;
      } else if (m >= 0xC1 && m <= 0xCF && m != 0xC4 && m != 0xC8 && m != 0xCC) {
        ok = false;
      } else if (m == 0xC4) {
        int o = 0;
        for (int t = 0; t < 8 && o + 17 <= body; ++t) {
          const int tc = s[o] >> 4, th = s[o] & 15;
          int total = 0;
          for (int i = 0; i < 16; ++i) total += s[o + 1 + i];
          if (tc > 1 || th > 3 || total > 256 || o + 17 + total > body) {
            ok = false;
            break;
          }
          (tc ? ac_off : dc_off)[th] = (int)(pos + 4 + o + 1);
          o += 17 + total;
        }
      } else if (m == 0xDD) {
        rec.restart = body >= 2 ? be16(s) : 0;
      } else if (m == 0xDA) {
        if (!have_frame || body < 10 || s[0] != 3 || s[7] != 0 || s[8] != 63) {
          ok = false;
          break;
        }
        for (int c = 0; c < 3; ++c) {
          const int td = s[2 + 2 * c] >> 4, ta = s[2 + 2 * c] & 15;
          if (s[1 + 2 * c] != cid[c] || td > 3 || ta > 3 || !dc_off[td] || !ac_off[ta] ||
              !q_off[tq[c]])
            ok = false;
          // luma tables first, the two chroma components share theirs in files we accept
          if (c < 2) {
            rec.dc_off[c] = dc_off[td & 3];
            rec.ac_off[c] = ac_off[ta & 3];
            rec.q_off[c] = q_off[tq[c]];
          } else if (dc_off[td & 3] != rec.dc_off[1] || ac_off[ta & 3] != rec.ac_off[1] ||
                     q_off[tq[c]] != rec.q_off[1]) {
            ok = false;
          }
        }
        rec.scan_off = (int)(pos + 2 + len);
        have_scan = true;
      } else if (m == 0xD9) {
        ok = false;
      }
      pos += 2 + len;
    }
    ok = ok && have_scan;
  }
  if (ok) {
    const int mcu = 8 * rec.hs;
    rec.mcux = (W + mcu - 1) / mcu;
    rec.mcuy = (H + mcu - 1) / mcu;
    // the image has to fit its slot of the region buffer
    ok = rec.mcux * mcu <= a.slot_side && rec.mcuy * mcu <= a.slot_side;
  }
  if (!ok) {
    H = 1;
    W = 1;
  }
  rec.H = H;
  rec.W = W;
  rec.size = ok ? (int)n : 0;
  rec.valid = ok ? 1 : 0;
  a.recs[b] = rec;
  a.heights[b] = H;
  a.widths[b] = W;
  a.region_offsets[b] = (int64_t)b * a.slot_side * a.slot_side * 3;
  a.region_widths[b] = 1;
}

// ---- entropy decoding ------------------------------------------------------------------------------
// File bytes reach a lane through its column of a ring in LDS (128 bytes per lane, dword i of lane
// l at ring[i][l], so that every access of a wavefront is free of bank conflicts).  The ring is fed
// at points that all lanes pass together, the start of every block: the 32 bytes loaded at the
// previous such point are written to the ring, and the next 32 are requested if the ring has
// room.  The wait for memory is then one block of decoding long, whichever lanes asked.  A lane
// that runs dry inside a block loads and waits on the spot.
constexpr int kRingBytes = 128;
constexpr int kRingStep = 32;  // bytes per load point: two 16-byte chunks
typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));

struct BitReader {
  const uint8_t* chunks;  // 8-byte aligned start of the file's first chunk (at or before the file)
  int64_t chunks_bytes;   // bytes from there to the end of the buffer of files
  uint32_t* ring;         // this lane's column: dword i at ring[i * kJpegThreads]
  int skew;               // file position pos is byte pos + skew from `chunks`
  int n;                  // file size
  int pos;                // next byte of the file
  int have;               // the ring holds the bytes before this one (from `chunks`, multiple of 32)
  bool pending;           // `next` holds the 32 bytes at `have`, not yet in the ring
  u32x4_a8 next[2];
  uint64_t acc;  // the low nbits bits are the unread ones, oldest on top
  int nbits;
  int zeros;   // bits put into acc behind the end of the data
  bool ended;  // a marker was reached: zero bits from here on
};

// The 16 bytes at `base + at` (8-byte aligned) of a buffer of `bytes` bytes; bytes beyond its end
// read as zero.
__device__ static inline u32x4_a8 load_chunk(const uint8_t* base, int64_t bytes, int64_t at) {
  if (__builtin_expect(at + 16 <= bytes, 1)) return *reinterpret_cast<const u32x4_a8*>(base + at);
  // the last bytes of the buffer of files: a rolled loop, this code is inlined in many places
  uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll 1
  for (int j = 0; j < 4; ++j) {
    uint32_t v = 0;
#pragma unroll 1
    for (int i = 0; i < 4; ++i)
      if (at + 4 * j + i < bytes) v |= (uint32_t)base[at + 4 * j + i] << (8 * i);
    w[j] = v;
  }
  return u32x4_a8{w[0], w[1], w[2], w[3]};
}
__device__ static __forceinline__ void request_bytes(BitReader& r) {
  r.next[0] = load_chunk(r.chunks, r.chunks_bytes, r.have);
  r.next[1] = load_chunk(r.chunks, r.chunks_bytes, r.have + 16);
  r.pending = true;
}
__device__ static __forceinline__ void accept_bytes(BitReader& r) {
  const int i = (r.have & (kRingBytes - 1)) >> 2;  // 32 bytes never wrap: both are powers of two
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    r.ring[(i + j) * kJpegThreads] = r.next[0][j];
    r.ring[(i + 4 + j) * kJpegThreads] = r.next[1][j];
  }
  r.have += kRingStep;
  r.pending = false;
}
// The point all lanes pass together (start of a block).
__device__ static __forceinline__ void feed_ring(BitReader& r) {
  if (r.pending) accept_bytes(r);
  // room: the 32 bytes to come replace those 128 bytes back, which must have been read
  if (!r.ended && r.have - (r.pos + r.skew) <= kRingBytes - kRingStep && r.have < r.n + r.skew)
    request_bytes(r);
}
// Makes the `count` <= 4 bytes at file position pos available in the ring.
__device__ static __forceinline__ void need_bytes(BitReader& r, int pos, int count) {
  while (pos + r.skew + count > r.have) {
    if (!r.pending) request_bytes(r);
    accept_bytes(r);
  }
}
__device__ static __forceinline__ void open_reader(BitReader& r, int start) {
  r.pos = start;
  r.have = (start + r.skew) & ~(kRingStep - 1);
  r.pending = false;
  r.acc = 0;
  r.nbits = 0;
  r.zeros = 0;
  if (!r.ended) {
    need_bytes(r, start, 4);
    request_bytes(r);
  }
}
__device__ static inline uint32_t ring_dword(const BitReader& r, int i) {
  return r.ring[(i & (kRingBytes / 4 - 1)) * kJpegThreads];
}
// Byte `pos` of the file (pos < n).
__device__ static __forceinline__ uint32_t file_byte(BitReader& r, int pos) {
  need_bytes(r, pos, 1);
  const int q = pos + r.skew;
  return (ring_dword(r, q >> 2) >> (8 * (q & 3))) & 0xFFu;
}

// Tops the bit buffer up to at least 33 bits: enough for the longest code (16) together with the
// longest value (15).  0xFF00 stands for a data byte 0xFF; any other marker ends the data of this
// row, and zero bits are supplied from there on.  Four bytes without a 0xFF among them, the usual
// case, go in at once.
// The four bytes at the read position, as they would go into the bit buffer at once; `usable`
// says whether they may (inside the file and the ring, no 0xFF among them).  Reading them early
// costs nothing: the position only moves when the buffer is topped up.
struct NextFour {
  uint32_t bits;   // first byte on top
  bool usable;
  bool in_reach;   // the four bytes are inside the file and in the ring (they may hold a 0xFF)
};
__device__ static inline NextFour next_four(const BitReader& r) {
  const int q = r.pos + r.skew;
  const uint32_t x = __builtin_amdgcn_alignbyte(ring_dword(r, (q >> 2) + 1), ring_dword(r, q >> 2),
                                                (uint32_t)(q & 3));
  const uint32_t inv = ~x;  // a byte 0xFF of x is a zero byte here
  NextFour f;
  f.bits = __builtin_bswap32(x);
  // (no short-circuit: straight-line code lets the reads above overlap the table look-up)
  f.in_reach = (int)!r.ended & (int)(r.pos + 4 <= r.n) & (int)(q + 4 <= r.have);
  f.usable = (int)f.in_reach & (int)(((inv - 0x01010101u) & ~inv & 0x80808080u) == 0u);
  return f;
}
__device__ static __forceinline__ void fill_bytewise(BitReader& r);
__device__ static __forceinline__ void fill(BitReader& r, const NextFour& f) {
  if (r.nbits > 32) return;
  if (f.usable) {
    r.acc = (r.acc << 32) | (uint64_t)f.bits;
    r.nbits += 32;
    r.pos += 4;
    return;
  }
  if (f.in_reach) {
    // a 0xFF among the four: byte by byte out of the register.  0xFF00 is a data byte 0xFF, any
    // other follower a marker; a 0xFF in the last place waits for its follower.
    bool skip = false, stop = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t b = (f.bits >> (24 - 8 * i)) & 0xFFu;
      const uint32_t follower = i < 3 ? (f.bits >> (16 - 8 * i)) & 0xFFu : 1u;
      const bool data = !skip && !stop && (b != 0xFFu || (i < 3 && follower == 0u));
      const bool marker = !skip && !stop && b == 0xFFu && i < 3 && follower != 0u;
      stop = stop || (!skip && b == 0xFFu && (i == 3 || follower != 0u));
      r.ended = r.ended || marker;
      const bool stuffed = data && b == 0xFFu;
      if (data) {
        r.acc = (r.acc << 8) | b;
        r.nbits += 8;
        r.pos += stuffed ? 2 : 1;
      }
      skip = stuffed;
    }
    if (r.nbits > 32) return;
  }
  fill_bytewise(r);
}
__device__ static __forceinline__ void fill(BitReader& r) {
  if (r.nbits > 32) return;
  if (!r.ended && r.pos + 4 <= r.n) need_bytes(r, r.pos, 4);
  fill(r, next_four(r));
}
__device__ static __forceinline__ void fill_bytewise(BitReader& r) {
  while (r.nbits <= 32) {
    uint32_t byte = 0;
    if (!r.ended && r.pos < r.n) {
      byte = file_byte(r, r.pos);
      if (byte == 0xFF) {
        if (r.pos + 1 < r.n && file_byte(r, r.pos + 1) == 0x00) {
          r.pos += 2;
        } else {
          r.ended = true;
          byte = 0;
          r.zeros += 8;
        }
      } else {
        r.pos += 1;
      }
    } else {
      r.zeros += 8;
    }
    r.acc = (r.acc << 8) | byte;
    r.nbits += 8;
  }
}
// Whether a row of MCUs can start where `left` bits of its data are unread, the last of them in
// `last`: a marker that ends the data comes behind up to seven one-bits of padding (T.81 F.1.2.3),
// and no code consists of ones alone, so such a rest holds none.
__device__ static inline bool row_can_start(int left, uint32_t last) {
  const uint32_t rest = (1u << (left & 7)) - 1u;
  return left >= 8 || (left > 0 && (last & rest) != rest);
}
// At a restart boundary: what is left of the interval (the padding of its last byte, fill bytes)
// is dropped, the marker skipped and the reader opened behind it.  Returns false when no restart
// marker follows within a few bytes.
__device__ static __forceinline__ bool restart_reader(BitReader& r) {
  int p = r.pos;  // the reader never loads a marker: it is at or behind this byte
  bool found = false;
  for (int i = 0; i < 16 && !found; ++i) {
    if (p + 1 >= r.n) break;
    if (file_byte(r, p) == 0xFFu && (file_byte(r, p + 1) & 0xF8u) == 0xD0u) found = true;
    else ++p;
  }
  r.ended = !found;
  open_reader(r, found ? p + 2 : r.pos);
  return found;
}

// The next 32 bits (after fill()), the oldest on top.
__device__ static inline uint32_t peek32(const BitReader& r) {
  return (uint32_t)(r.acc >> (r.nbits - 32));
}

// `size` >= 1 value bits that follow a code of `len` bits in `top`, as the signed value they stand
// for (T.81 F.2.2.1: the lower half of the range is the negative numbers).
__device__ static inline int value_bits(uint32_t top, int len, int size) {
  const int v = (int)((top << len) >> (32 - size));
  return v < (1 << (size - 1)) ? v - (1 << size) + 1 : v;
}

// Canonical code (Annex C) in the form the decoder wants.  With every code left-aligned in 16
// bits, the codes of one length are a range, and the ranges follow each other with the length:
// range[l].limit is the end of the range of length l + 1, so the length of the code that starts
// the 16 bits x is one more than the number of limits that x has reached.  range[l].delta turns
// the leading l + 1 bits into the index of the symbol.
struct CodeRange {
  uint32_t limit;
  int32_t delta;
};
struct alignas(16) HuffDc {
  CodeRange range[16];
  uint8_t symbols[16];  // categories 0..11
};
constexpr int kFastBits = 10;
struct alignas(16) HuffAc {
  CodeRange range[16];
  uint8_t symbols[256];
  uint16_t fast[1 << kFastBits];  // per 10-bit prefix: length << 8 | symbol, 0 = a longer code
};

// The code that starts the 16 bits x, looking at lengths above kFrom only: index (length - 1) of
// its length, 16 = none, and through `index` the position of its symbol in the table.
template <int kFrom>
__device__ static inline int find_code(const CodeRange* range, uint32_t x, int& index) {
  int len = kFrom, delta = range[kFrom].delta;
#pragma unroll
  for (int l = kFrom; l < 16; ++l) {
    if (x >= range[l].limit) {
      len = l + 1;
      delta = l + 1 < 16 ? range[l + 1].delta : 0;
    }
  }
  index = delta + (int)(x >> (15 - min(len, 15)));
  return len;
}

// Sum over eight 16-bit values times one row of the basis, two products per instruction; the
// sums stay below 2^31 (the row's absolute values add up to 43284, the values are at most 32767).
typedef short s16x2 __attribute__((ext_vector_type(2)));
__device__ static inline int basis_dot(const s16x2 v[4], int row) {
  const s16x2* basis = reinterpret_cast<const s16x2*>(kBasis) + row * 4;
  int acc = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) acc = __builtin_amdgcn_sdot2(v[i], basis[i], acc, false);
  return acc;
}

// One row of the second pass of the inverse DCT below.
__device__ static inline void idct_row(const int16_t* coef, int y, int out[8]) {
  s16x2 t[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    t[i] = s16x2{coef[(y * 8 + 2 * i) * kJpegThreads], coef[(y * 8 + 2 * i + 1) * kJpegThreads]};
#pragma unroll
  for (int x = 0; x < 8; ++x)
    out[x] = min(max(((basis_dot(t, x) + (1 << 16)) >> 17) + 128, 0), 255);
}

// Dequantised coefficients (natural order, 16-bit) -> 64 samples, in two passes.  The coefficients
// live in LDS with the lane as the fastest index (element k of this lane at coef[k * 64]): the
// lanes of a wavefront then touch neighbouring addresses instead of one bank.  The first pass
// overwrites each column with its transform (the clamped values fit 16 bits); the second gives
// the samples row by row.
__device__ static inline void idct_columns(int16_t* coef) {
  for (int u = 0; u < 8; ++u) {
    s16x2 c[4];
    int t[8];
#pragma unroll
    for (int i = 0; i < 4; ++i)
      c[i] = s16x2{coef[(2 * i * 8 + u) * kJpegThreads], coef[((2 * i + 1) * 8 + u) * kJpegThreads]};
#pragma unroll
    for (int y = 0; y < 8; ++y)
      t[y] = min(max((basis_dot(c, y) + (1 << 10)) >> 11, -32767), 32767);
#pragma unroll
    for (int y = 0; y < 8; ++y) coef[(y * 8 + u) * kJpegThreads] = (int16_t)t[y];
  }
}

__device__ static inline uint32_t ycc_to_rgbx(int y, int cb, int cr) {
  const int b = cb - 128, r = cr - 128;
  const int R = min(max(y + ((91881 * r + 32768) >> 16), 0), 255);
  const int G = min(max(y - ((22554 * b + 46802 * r + 32768) >> 16), 0), 255);
  const int B = min(max(y + ((116130 * b + 32768) >> 16), 0), 255);
  return (uint32_t)R | ((uint32_t)G << 8) | ((uint32_t)B << 16);
}

// Images per workgroup of the decode kernel (template parameter kGroup: 4, 2 or 1): their rows of
// MCUs share the 64 lanes.  A lane gets at most kGroup rows (an image has at most 64).

constexpr int kBlockBytes = 128;  // a block of coefficients in the plane buffer
// 0: the sample takes no part
constexpr int kLivePlanes = 1, kLiveCoefs = 2, kLivePieces = 3, kLiveSpill = 4;

// What the wavefront keeps per image of its group.
struct JpegImage {
  HuffDc dc[2];  // luma, chroma
  HuffAc ac[2];
  uint16_t qz[2][64];  // per zig-zag position: natural position << 8 | quantiser step
  int my0, mx0, mx1, nrows, region_w, hs, size, scan_off;
  // kLivePlanes: decoded to planes, kLiveCoefs: by jpeg_entropy_kernel to coefficients,
  // kLivePieces: the same, and the states of pieces of its rows are known, kLiveSpill: to
  // coefficients that its slot of the plane buffer does not hold alone (spilled_rows)
  int live;
  int restart, mcux;  // restart interval in MCUs (0 = none), MCUs per row of the image
  // bytes of entropy-coded data in the image's slot of the region buffer, byte stuffing removed
  // (see jpeg_unstuff), + kCutShort where the file ends without a marker behind them; -1 = not there
  int clean_bytes;
  int64_t origin, region_off;
};

// What the table kernel hands to the decode kernel per image (through the workspace).
struct alignas(16) JpegPrepared {
  JpegImage im;
};
static_assert(sizeof(JpegPrepared) % 16 == 0, "copied in 16-byte pieces");

// Where the entropy-coded data of one of the crop's rows of MCUs starts: the bit reader's state
// and the DC predictors at that point (workspace; max_rows of them per image).
struct alignas(16) RowState {
  int32_t pos;        // next byte of the file that goes into the bit buffer; -1 = not known
  int32_t nbits;      // unread bits in acc
  uint64_t acc;
  int16_t pred[3];    // Y, Cb, Cr
  uint16_t rst_left;  // MCUs from here to the next restart marker (unused without an interval)
  int32_t pad;
};
static_assert(sizeof(RowState) == 32, "32 bytes per row");

template <int kGroup>
struct JpegLds {
  JpegPrepared img[kGroup];
  // one block per lane, the lane is the fastest index; row 64 takes the stores of skipped blocks
  int16_t coef[65][kJpegThreads];
  uint32_t ring[kRingBytes / 4][kJpegThreads];  // file bytes on their way to the lanes
};

// A file's entropy-coded data without its byte stuffing lies in the image's slot of the region
// buffer until jpeg_idct_kernel writes the region there: the bytes at the start of the slot, and
// behind them (clean_map_offset) the file position of every 16th of them.  The slot's size does
// not depend on the file's, so a file may be too large for it; such a file is walked by
// jpeg_scan_kernel.
__device__ static inline int64_t clean_map_offset(int size, int scan_off) {
  return ((int64_t)(size - scan_off) + 31) & ~(int64_t)15;
}
__device__ static inline bool clean_fits(const JpegArgs& a, int size, int scan_off) {
  const int64_t raw = (int64_t)size - scan_off;
  return raw < (1 << 27) && clean_map_offset(size, scan_off) + 4 * (raw / 16 + 2) <=
                                (int64_t)a.slot_side * a.slot_side * 3;
}
constexpr int kCleanStep = kJpegThreads * 16;  // bytes of the file per step
constexpr int kCutShort = 1 << 30;             // (beyond any number of bytes that fits)

// The walk over a file that is one chain of codes can also tell where each of several pieces of the
// crop's rows starts, so that a row is several lanes' work: as many pieces as fill a wavefront (four
// at most), from the crop's first MCU on.  Their states lie at the end of the image's slot of the
// region buffer until the region is written.
constexpr int kMaxPieces = 4, kPieceBytes = kJpegThreads * 32;
__device__ static inline int pieces_per_row(int nrows, int ncols) {
  return max(1, min(min(kMaxPieces, kJpegThreads / max(nrows, 1)), ncols));
}
__device__ static inline RowState* piece_states(const JpegArgs& a, int64_t region_off) {
  return reinterpret_cast<RowState*>(a.regions + region_off +
                                     (int64_t)a.slot_side * a.slot_side * 3 - kPieceBytes);
}
__device__ static inline bool pieces_fit(const JpegArgs& a, int size, int scan_off, int nrows) {
  const int64_t raw = (int64_t)size - scan_off;
  return nrows <= kJpegThreads && clean_map_offset(size, scan_off) + 4 * (raw / 16 + 2) + kPieceBytes <=
                                      (int64_t)a.slot_side * a.slot_side * 3;
}

// The two passes over a file's bytes below take 16 of them per lane and step, four at a time: bit 7 of
// every byte of x that is 0xFF, or zero, and bit i of a mask for byte i of a lane's 16.
__device__ static inline uint32_t ff_bytes(uint32_t x) {
  return ((x & 0x7F7F7F7Fu) + 0x01010101u) & x & 0x80808080u;
}
__device__ static inline uint32_t zero_bytes(uint32_t x) {
  return ~(((x & 0x7F7F7F7Fu) + 0x7F7F7F7Fu) | x | 0x7F7F7F7Fu);
}
__device__ static inline uint32_t byte_mask(uint32_t m0, uint32_t m1, uint32_t m2, uint32_t m3) {
  const uint32_t lo = __builtin_amdgcn_udot4(m1 >> 7, 0x80402010u,
                                             __builtin_amdgcn_udot4(m0 >> 7, 0x08040201u, 0u, false), false);
  const uint32_t hi = __builtin_amdgcn_udot4(m3 >> 7, 0x80402010u,
                                             __builtin_amdgcn_udot4(m2 >> 7, 0x08040201u, 0u, false), false);
  return lo | (hi << 8);
}
// Bits n and up / below n, of 16 (any n).
__device__ static inline uint32_t mask_from(int n) { return (0xFFFFu << min(max(n, 0), 16)) & 0xFFFFu; }
__device__ static inline uint32_t mask_below(int n) { return ~mask_from(n) & 0xFFFFu; }
// Sum of the lanes' x (below 32) over the lanes in front of this one, and over all of them.
__device__ static inline int lanes_before(int x, int& total) {
  int before = 0;
  total = 0;
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    const uint64_t has = __builtin_amdgcn_ballot_w64((x >> k) & 1);
    before += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32),
                                             __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u)) << k;
    total += __popcll(has) << k;
  }
  return before;
}

// Entropy-coded data from scan_off to the first marker, byte stuffing removed, into `clean`, with
// the file position of every 16th byte in `map`; returns how many bytes, + kCutShort when the file
// ends before a marker does it (whole wavefront).  The file is read in aligned 16-byte pieces, one
// per lane, the next two steps' on their way (a step looks at the first byte of the next one); a prefix
// sum gives each piece its place in the LDS buffer, which leaves in 1-KiB stores.  What bounds it is
// a wavefront's chain of latencies per step, 1.2 us: with single bytes looked at and stored, prefix sums through
// LDS and one step's pieces on their way, which the look at the next one waited for, it was 2.9 us.  The
// whole kernel, 1024 files of 256 pixels 92 -> 56 us, 512 files of 500 pixels 254 -> 115 us; 4096 files whose
// restart markers it looks for 158 -> 131 us.
__device__ static int jpeg_unstuff(const JpegArgs& a, int64_t origin, int scan_off, int n,
                                   uint8_t* stage, uint8_t* clean, int32_t* map) {
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  typedef u32x4 u32x4_a1 __attribute__((aligned(1)));
  typedef uint64_t u64_a1 __attribute__((aligned(1)));
  typedef uint32_t u32_a1 __attribute__((aligned(1)));
  typedef uint16_t u16_a1 __attribute__((aligned(1)));
  const int lane = threadIdx.x;
  const int64_t first = (origin + scan_off) & ~(int64_t)15;
  const int64_t end = origin + n;
  int done = 0, fill = 0;  // bytes stored / bytes waiting in `stage`
  uint32_t carry = 0;      // the last byte of the step before was 0xFF
  int cut = kCutShort;
  u32x4_a8 cur = load_chunk(a.files, a.files_bytes, first + lane * 16);
  u32x4_a8 next = load_chunk(a.files, a.files_bytes, first + lane * 16 + kCleanStep);
  for (int64_t base = first; base < end; base += kCleanStep) {
    const int64_t at = base + lane * 16;
    const u32x4_a8 later = load_chunk(a.files, a.files_bytes, at + 2 * kCleanStep);
    const int p0 = (int)(at - origin);
    const uint32_t ff = byte_mask(ff_bytes(cur.x), ff_bytes(cur.y), ff_bytes(cur.z), ff_bytes(cur.w));
    const uint32_t zero =
        byte_mask(zero_bytes(cur.x), zero_bytes(cur.y), zero_bytes(cur.z), zero_bytes(cur.w));
    // the byte in front of the piece is 0xFF; the one behind it is zero
    const uint64_t last_ff = __builtin_amdgcn_ballot_w64(ff >> 15 != 0u);
    const uint64_t first_zero = __builtin_amdgcn_ballot_w64((zero & 1u) != 0u);
    const uint64_t wrap = (uint64_t)((__builtin_amdgcn_readfirstlane((int)next.x) & 0xFF) == 0);
    const uint32_t prev = (uint32_t)(((last_ff << 1) | carry) >> lane) & 1u;
    const uint32_t follow = (uint32_t)(((first_zero >> 1) | (wrap << 63)) >> lane) & 1u;
    const uint32_t inside = mask_from(scan_off - p0) & mask_below(n - p0);
    const uint32_t stuffing = zero & ((ff << 1) | prev) & mask_from(scan_off + 1 - p0);
    const uint32_t marker = ff & inside & ~(((zero >> 1) | (follow << 15)) & mask_below(n - 1 - p0));
    uint32_t keep = inside & ~stuffing;
    const uint64_t stops = __builtin_amdgcn_ballot_w64(marker != 0u);
    if (stops) {  // (of the first piece with a marker, what comes before it)
      const int who = __builtin_ctzll(stops);
      keep &= lane < who ? 0xFFFFu : (lane == who ? (marker & (0u - marker)) - 1u : 0u);
    }
    const int cnt = __popc(keep);
    int total;
    const int place = fill + lanes_before(cnt, total);
    // the kept bytes next to each other, and where the one was that is the 16th of the data
    uint64_t lo = (uint64_t)cur.x | ((uint64_t)cur.y << 32), hi = (uint64_t)cur.z | ((uint64_t)cur.w << 32);
    const int mapped = -(done + place) & 15;
    int from = mapped;
    uint32_t drop = keep ? ~keep & ((1u << (31 - __clz((int)keep))) - 1u) : 0u;
    for (int gone = 0; drop; ++gone) {
      const int q = __builtin_ctz(drop);
      from += q + gone <= from ? 1 : 0;
      const uint64_t low = q < 8 ? ~(uint64_t)0 << (8 * q) : 0u;         // bytes q .. 7
      const uint64_t high = q < 8 ? ~(uint64_t)0 : ~(uint64_t)0 << (8 * (q - 8));
      lo = (lo & ~low) | (((lo >> 8) | (hi << 56)) & low);
      hi = (hi & ~high) | ((hi >> 8) & high);
      drop = (drop & (drop - 1u)) >> 1;
    }
    uint8_t* dst = stage + place;
    if (cnt == 16) {
      *reinterpret_cast<u32x4_a1*>(dst) =
          u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    } else {
      if (cnt & 8) {
        *reinterpret_cast<u64_a1*>(dst) = lo;
        lo = hi;
        dst += 8;
      }
      if (cnt & 4) {
        *reinterpret_cast<u32_a1*>(dst) = (uint32_t)lo;
        lo >>= 32;
        dst += 4;
      }
      if (cnt & 2) {
        *reinterpret_cast<u16_a1*>(dst) = (uint16_t)lo;
        lo >>= 16;
        dst += 2;
      }
      if (cnt & 1) *dst = (uint8_t)lo;
    }
    if (mapped < cnt) map[(done + place + mapped) >> 4] = p0 + from;
    fill += total;
    __syncthreads();
    if (fill >= kCleanStep) {
      u32x4* src = reinterpret_cast<u32x4*>(stage);
      reinterpret_cast<u32x4*>(clean + done)[lane] = src[lane];
      const u32x4 rest = src[kJpegThreads + lane];
      __syncthreads();
      src[lane] = rest;
      done += kCleanStep;
      fill -= kCleanStep;
      __syncthreads();
    }
    if (stops) {
      cut = 0;
      break;
    }
    carry = (uint32_t)(last_ff >> 63);
    cur = next;
    next = later;
  }
  if (lane * 16 < fill)
    reinterpret_cast<u32x4*>(clean + done)[lane] = reinterpret_cast<u32x4*>(stage)[lane];
  return done + fill + cut;
}

// Coefficients with 4:4:4 sampling take twice the slot for a crop that fills it.  As many of the
// crop's last rows of MCUs as the image's slot of the plane buffer holds go there; the first rows,
// of which this is the number, go to the end of its slot of the region buffer.  One workgroup of
// jpeg_idct_kernel then takes the rows in order (with such crops by jpeg_decode_kernel to planes,
// beside others by coefficients, a batch waited for one and the other: 512 files of 256 pixels,
// 4:4:4, a restart interval per row: 3.94 -> 1.10 ms; 4096 files 5.85 -> 3.77; all of them by
// planes 3.19 and 3.98): the pixels of rows 0 .. r need (r + 1) half rows of coefficients from the
// slot's start on, and the rows of coefficients behind r start at or behind that, as all that are
// there (never more than the slot, whose side is a multiple of two MCUs) end with it.
__device__ static inline int spilled_rows(int64_t slot_bytes, int64_t row_bytes, int nrows) {
  return max(0, nrows - (int)(slot_bytes / row_bytes));
}

// Tables, crop geometry and restart-marker positions of image b into slot `im` (whole wavefront).
__device__ static void jpeg_prepare_image(const JpegArgs& a, int b, JpegImage& im,
                                          uint8_t* stage) {
  const int lane = threadIdx.x;
  const JpegRec rec = a.recs[b];
  CropRec* crop = reinterpret_cast<CropRec*>(a.workspace + kWorkspaceHeader) + b;
  CropRec cr = *crop;
  RowState* states = reinterpret_cast<RowState*>(a.row_states) + (int64_t)b * a.max_rows;
  __syncthreads();  // everybody has read the record before lane 0 rewrites it
  if (a.whole_image) {
    // index run: the "crop" is the whole image, and every row of the index gets a defined value
    // whatever becomes of the file
    cr.top = 0;
    cr.left = 0;
    cr.ch = rec.H;
    cr.cw = rec.W;
    cr.flip = 0;
    cr.valid = 1;
    RowState none;
    none.pos = -1;
    none.nbits = 0;
    none.acc = 0;
    none.pred[0] = none.pred[1] = none.pred[2] = 0;
    none.rst_left = 0;
    none.pad = 0;
    for (int i = lane; i < a.max_rows; i += kJpegThreads) states[i] = none;
    __syncthreads();
  }
  if (!rec.valid) {
    if (lane == 0) {
      crop->valid = 0;
      if (a.crop_out) a.crop_out[(int64_t)b * 6 + 5] = 0;
      im.live = 0;
      im.nrows = 0;
    }
    return;
  }
  if (!cr.valid) {
    if (lane == 0) {
      im.live = 0;
      im.nrows = 0;
    }
    return;
  }
  const uint8_t* d = a.files + a.offsets[b];
  const int n = rec.size;
  const int mcu = 8 * rec.hs;
  // rows and columns of MCUs that the crop touches
  const int my0 = cr.top / mcu, my1 = min((cr.top + cr.ch - 1) / mcu, rec.mcuy - 1);
  const int mx0 = cr.left / mcu, mx1 = min((cr.left + cr.cw - 1) / mcu, rec.mcux - 1);
  // Blocks as 64 coefficients of 16 bits: the slot of the plane buffer (3 bytes per pixel) holds
  // those of any crop with 4:2:0 sampling and of a crop of up to half the slot with 4:4:4; of a larger
  // one the slot of the region buffer takes the rest.  A restart boundary may only fall between rows
  // of MCUs.
  const int64_t slot_bytes = (int64_t)a.slot_side * a.slot_side * 3;
  const int nrows = my1 - my0 + 1, ncols = mx1 - mx0 + 1;
  const int64_t row_bytes = (int64_t)ncols * (rec.hs * rec.hs + 2) * kBlockBytes;
  const int spilled = spilled_rows(slot_bytes, row_bytes, nrows);
  // (a row that jpeg_idct_kernel takes in several steps, half of it written before all is read: only
  // where the spilled rows leave half a row free, which all crops but one of the whole slot do)
  const bool dense = rec.restart % rec.mcux == 0 && !a.whole_image &&
                     (spilled == 0 || ncols <= kWave || spilled * row_bytes + row_bytes / 2 <= slot_bytes);
  if (dense) {  // most coefficients are zero: only the others will be written
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4* coef = reinterpret_cast<u32x4*>(a.planes + a.region_offsets[b]);
    const int pieces = (int)((nrows - spilled) * row_bytes / 16);  // (spilled rows: jpeg_entropy_kernel)
    for (int i = lane; i < pieces; i += kJpegThreads) coef[i] = u32x4{0u, 0u, 0u, 0u};
  }
  if (lane == 0) {
    im.my0 = my0;
    im.mx0 = mx0;
    im.mx1 = mx1;
    im.nrows = my1 - my0 + 1;
    im.region_w = (mx1 - mx0 + 1) * mcu;
    im.hs = rec.hs;
    im.size = n;
    im.scan_off = rec.scan_off;
    im.restart = rec.restart;
    im.mcux = rec.mcux;
    im.clean_bytes = -1;
    im.live = !dense ? kLivePlanes : (spilled ? kLiveSpill : kLiveCoefs);
    im.origin = a.offsets[b];
    im.region_off = a.region_offsets[b];
    // region geometry for jpeg_idct_kernel and the resampling kernel
    a.region_widths[b] = (mx1 - mx0 + 1) * mcu;
    a.recs[b].region_h = (my1 - my0 + 1) * mcu;
    crop->top = cr.top - my0 * mcu;
    crop->left = cr.left - mx0 * mcu;
  }

  // tables: symbols and quantiser steps by all lanes
  for (int t = 0; t < 2; ++t) {
    if (lane < 16) im.dc[t].symbols[lane] = d[min(rec.dc_off[t] + 16 + lane, n - 1)];
    for (int i = lane; i < 256; i += kJpegThreads)
      im.ac[t].symbols[i] = d[min(rec.ac_off[t] + 16 + i, n - 1)];
  }
  for (int i = lane; i < 128; i += kJpegThreads)
    im.qz[i >> 6][i & 63] =
        (uint16_t)(((int)kZigzag[i & 63] << 8) | d[min(rec.q_off[i >> 6] + (i & 63), n - 1)]);
  {  // code ranges: lane = table * 16 + (length - 1); the counts of the shorter lengths come from
     // the lanes before it (first code of a length = twice the end of the length before)
    const int tt = lane >> 4, len = lane & 15;
    const int t = tt & 1;
    const bool is_ac = tt >= 2;
    const int count = d[min((is_ac ? rec.ac_off[t] : rec.dc_off[t]) + len, n - 1)];
    int code = 0, index = 0;
    for (int j = 0; j < 15; ++j) {
      const int cj = __shfl(count, (tt << 4) + j);
      if (j < len) {
        code += cj << (len - j);
        index += cj;
      }
    }
    CodeRange* range = is_ac ? im.ac[t].range : im.dc[t].range;
    range[len].delta = index - code;
    range[len].limit = (uint32_t)(code + count) << (15 - len);
  }
  __syncthreads();
  for (int t = 0; t < 2; ++t) {
    HuffAc& h = im.ac[t];
    // direct table: the code that starts a 10-bit prefix is the one of the first length whose
    // range the prefix (followed by zeros) falls into; none = a longer code
    for (int i = lane; i < (1 << kFastBits); i += kJpegThreads) {
      const uint32_t x = (uint32_t)i << (16 - kFastBits);
      int len = kFastBits;
      for (int l = kFastBits - 1; l >= 0; --l)
        if (x < h.range[l].limit) len = l;
      uint16_t e = 0;
      if (len < kFastBits)
        e = (uint16_t)(((len + 1) << 8) |
                       h.symbols[(h.range[len].delta + (int)(x >> (15 - len))) & 255]);
      h.fast[i] = e;
    }
  }

  // the rows' states: unknown until found below or by the scan kernel
  {
    RowState none;
    none.pos = -1;
    none.nbits = 0;
    none.acc = 0;
    none.pred[0] = none.pred[1] = none.pred[2] = 0;
    none.rst_left = 0;
    none.pad = 0;
    const int nrows = min(my1 - my0 + 1, a.max_rows);
    for (int i = lane; i < nrows; i += kJpegThreads) states[i] = none;
  }
  __syncthreads();  // (these stores are complete before a row's real state is written)
  if (a.row_index) {
    // the states come from the caller's index of the file (row r of the file at entry r).  It is
    // the caller's memory: an entry that does not point into the entropy-coded data or whose bit
    // count is impossible is left unknown, which flags the sample in the decode kernel.
    const RowState* index = reinterpret_cast<const RowState*>(a.row_index) + (int64_t)b * a.max_rows;
    const int nrows = min(my1 - my0 + 1, a.max_rows);
    for (int i = lane; i < nrows; i += kJpegThreads) {
      if (my0 + i >= a.max_rows) continue;
      RowState st = index[my0 + i];
      const bool ok = st.pos >= rec.scan_off && st.pos <= n && st.nbits >= 0 && st.nbits <= 64;
      if (ok) states[i] = st;
    }
    return;
  }
  if (rec.restart == 0 && clean_fits(a, n, rec.scan_off)) {
    // one chain of codes from end to end: jpeg_sync_kernel enters it in many places at once
    uint8_t* clean = a.regions + a.region_offsets[b];
    const int bytes = jpeg_unstuff(
        a, a.offsets[b], rec.scan_off, n, stage, clean,
        reinterpret_cast<int32_t*>(clean + clean_map_offset(n, rec.scan_off)));
    if (lane == 0) im.clean_bytes = bytes;
    return;
  }
  if (rec.restart != rec.mcux) return;  // rows not independent: the scan kernel finds the states

  // restart markers: marker m (0-based) ends MCU row m; row r starts after marker r - 1.  The
  // file is scanned in aligned 16-byte pieces of the buffer, one per lane and step, the next two
  // steps' pieces on their way while this step's are examined.
  RowState start;
  start.nbits = 0;
  start.acc = 0;
  start.pred[0] = start.pred[1] = start.pred[2] = 0;
  start.rst_left = (uint16_t)rec.restart;
  start.pad = 0;
  const int64_t origin = a.offsets[b];
  const int64_t first = (origin + rec.scan_off) & ~(int64_t)15;
  const int64_t last = origin + n - 1;  // a marker starts before this byte
  int seen = 0;                         // markers before the current step
  u32x4_a8 cur = load_chunk(a.files, a.files_bytes, first + lane * 16);
  u32x4_a8 next = load_chunk(a.files, a.files_bytes, first + lane * 16 + kJpegThreads * 16);
  for (int64_t base = first; base < last && seen <= my1; base += kJpegThreads * 16) {
    const int64_t at = base + lane * 16;
    const u32x4_a8 later = load_chunk(a.files, a.files_bytes, at + 2 * kJpegThreads * 16);
    const int p0 = (int)(at - origin);  // file position of the piece (negative before the file)
    const uint32_t ff = byte_mask(ff_bytes(cur.x), ff_bytes(cur.y), ff_bytes(cur.z), ff_bytes(cur.w));
    const auto rst = [](uint32_t x) { return zero_bytes((x & 0xF8F8F8F8u) ^ 0xD0D0D0D0u); };  // 0xD0 .. 0xD7
    const uint32_t second = byte_mask(rst(cur.x), rst(cur.y), rst(cur.z), rst(cur.w));
    // the byte after this piece: the first of the next lane's, or of the next step's
    const uint64_t first_second = __builtin_amdgcn_ballot_w64((second & 1u) != 0u);
    const uint64_t wrap = (uint64_t)((__builtin_amdgcn_readfirstlane((int)next.x) & 0xF8) == 0xD0);
    const uint32_t follow = (uint32_t)(((first_second >> 1) | (wrap << 63)) >> lane) & 1u;
    // bit i: a restart marker starts at byte p0 + i
    uint32_t mask = ff & ((second >> 1) | (follow << 15)) & mask_from(rec.scan_off - p0) &
                    mask_below(n - 1 - p0);
    if (__builtin_amdgcn_ballot_w64(mask != 0u)) {
      int total;
      // the row that starts after the lane's first marker
      int row = seen + lanes_before(__popc(mask), total) + 1;
      for (; mask; mask &= mask - 1u, ++row) {
        if (row >= my0 && row <= my1 && row - my0 < a.max_rows) {
          start.pos = p0 + __builtin_ctz(mask) + 2;
          states[row - my0] = start;
        }
      }
      seen += total;
    }
    cur = next;
    next = later;
  }
  if (my0 == 0 && lane == 0) {
    start.pos = rec.scan_off;
    states[0] = start;
  }
}

// One wavefront per image: tables, crop geometry, row starts -> workspace.  Many of these fit a
// CU at once, which hides the latency of the scattered header reads and of the marker scan.
__global__ __launch_bounds__(kJpegThreads) void jpeg_tables_kernel(JpegArgs a) {
  __shared__ JpegPrepared p;
  __shared__ __attribute__((aligned(16))) uint8_t stage[2 * kCleanStep];
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const int b = (int)blockIdx.x;
  for (int i = threadIdx.x; i < (int)(sizeof(JpegPrepared) / 16); i += kJpegThreads)
    reinterpret_cast<u32x4*>(&p)[i] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  jpeg_prepare_image(a, b, p.im, stage);
  __syncthreads();
  u32x4* dst = reinterpret_cast<u32x4*>(a.prepared + (size_t)b * sizeof(JpegPrepared));
  for (int i = threadIdx.x; i < (int)(sizeof(JpegPrepared) / 16); i += kJpegThreads)
    dst[i] = reinterpret_cast<const u32x4*>(&p)[i];
}

// DC difference of the next block (T.81 F.2.2.1).  Returns false for a code that does not exist
// or a category that 8-bit data does not have (the difference is then 0).
__device__ static __forceinline__ bool decode_dc(BitReader& r, const HuffDc& h, int& diff) {
  fill(r);
  const uint32_t top = peek32(r);
  const uint32_t x = top >> 16;
  int index;
  int len = find_code<0>(h.range, x, index);
  int sym = 16;
  if (len < 16) sym = h.symbols[index & 15];
  const bool ok = sym <= 11;
  if (!ok) {
    sym = 0;
    len = -1;
  }
  diff = sym ? value_bits(top, len + 1, sym) : 0;
  r.nbits -= len + 1 + sym;
  return ok;
}

// AC coefficients of a block (F.2.2.2): a symbol is a run of zeros << 4 | size of the value.  The
// usual step -- short code, and the next four bytes ready if the buffer has to be topped up -- is
// straight-line code; everything else takes the one branch.  kStore: de-quantised values go to
// the lane's column of `coef` (natural order; row 64 takes what is skipped); otherwise only the
// symbols' lengths are followed.  Returns false for a code that does not exist or a run past the
// end of the block.
template <bool kStore>
__device__ static __forceinline__ bool decode_ac(BitReader& r, const HuffAc& h, const uint16_t* qz,
                                        int16_t* coef, bool want) {
  bool ok = true;
  fill(r);
  for (int k = 1; k < 64;) {
    const NextFour ahead = next_four(r);  // in flight while the symbol is looked up
    const uint32_t top = peek32(r);
    const int e = h.fast[top >> (32 - kFastBits)];
    int len1 = e >> 8, rs = e & 255;
    const bool top_up = r.nbits - (len1 + (rs & 15)) <= 32;
    if ((int)(e == 0) | ((int)top_up & (int)!ahead.usable)) {
      if (!e) {
        int index;
        const int len = find_code<kFastBits>(h.range, top >> 16, index);
        rs = h.symbols[index & 255];
        len1 = len + 1;
        if (len == 16) {  // no such code: flag the sample and end the block
          ok = false;
          rs = 0;
          len1 = 0;
        }
      }
      r.nbits -= len1 + (rs & 15);
      fill(r, ahead);
    } else {
      r.nbits -= len1 + (rs & 15) - (top_up ? 32 : 0);
      r.acc = top_up ? (r.acc << 32) | (uint64_t)ahead.bits : r.acc;
      r.pos += top_up ? 4 : 0;
    }
    const int run = rs >> 4, size = rs & 15;
    // size 0: sixteen zeros (run 15) or the end of the block
    k += size ? run : (run == 15 ? 16 : 64);
    ok = ok && !(size != 0 && k > 63);
    if (kStore) {  // no branch: what is not to be stored goes to the spare row 64
      const bool store = size != 0 && k <= 63;
      const int zq = qz[k & 63];
      coef[(store && want ? zq >> 8 : 64) * kJpegThreads] = (int16_t)min(
          max(value_bits(top, len1, size ? size : 1) * (zq & 255), -32767), 32767);
    }
    k += size ? 1 : 0;
  }
  return ok;
}

__device__ static __forceinline__ void reader_for(BitReader& r, const JpegArgs& a, const JpegImage& im,
                                         uint32_t* ring) {
  r.skew = (int)(im.origin & 7);
  r.chunks = a.files + (im.origin - r.skew);
  r.chunks_bytes = a.files_bytes - (im.origin - r.skew);
  r.ring = ring;
  r.n = im.size;
}
// Opens the reader in the state recorded for a row.
__device__ static __forceinline__ void open_at(BitReader& r, const RowState& st) {
  open_reader(r, st.pos);
  r.acc = st.acc;
  r.nbits = st.nbits;
}

// ---- files whose rows of MCUs are not independent: where does each of the crop's rows start? ----
// One lane per file, kScanImages files per wavefront (two: a batch then gives every SIMD two
// wavefronts to switch between, and a lane rarely waits for the other's longer block).  The lane walks
// the entropy-coded data from its start: per block the DC difference (the predictors run through
// the whole interval) and the lengths of the AC symbols; at every restart boundary the marker is
// skipped and the predictors cleared.  At the first MCU of each of the crop's rows the reader's
// state goes to the workspace.  The walk ends with the crop's last row.
constexpr int kScanImages = 2;
struct JpegScanLds {
  JpegPrepared img[kScanImages];
  uint32_t ring[kRingBytes / 4][kJpegThreads];
};

__global__ __launch_bounds__(kJpegThreads) void jpeg_scan_kernel(JpegArgs a) {
  __shared__ JpegScanLds s;
  const int lane = threadIdx.x;
  const int b0 = (int)blockIdx.x * kScanImages;
  const int nimg = min(kScanImages, a.B - b0);
  bool need = false;
  if (lane < nimg) {
    const JpegRec rec = a.recs[b0 + lane];
    const CropRec cr = reinterpret_cast<const CropRec*>(a.workspace + kWorkspaceHeader)[b0 + lane];
    need = rec.valid && (cr.valid || a.whole_image) && rec.restart != rec.mcux && !a.row_index &&
           reinterpret_cast<const JpegPrepared*>(a.prepared)[b0 + lane].im.clean_bytes < 0;
  }
  if (__builtin_amdgcn_ballot_w64(need) == 0) return;  // every file here has independent rows
  {
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4* src = reinterpret_cast<const u32x4*>(a.prepared + (size_t)b0 * sizeof(JpegPrepared));
    u32x4* dst = reinterpret_cast<u32x4*>(&s.img[0]);
    const int n16 = nimg * (int)(sizeof(JpegPrepared) / 16);
    for (int i = lane; i < n16; i += kJpegThreads) dst[i] = src[i];
  }
  __syncthreads();
  if (!need) return;  // (no barrier below)

  const JpegImage& im = s.img[lane].im;
  const int b = b0 + lane;
  RowState* states = reinterpret_cast<RowState*>(a.row_states) + (int64_t)b * a.max_rows;
  BitReader r;
  reader_for(r, a, im, &s.ring[0][lane]);
  r.ended = false;
  open_reader(r, im.scan_off);
  const int nblk = im.hs * im.hs, per_mcu = nblk + 2;
  const int rows = im.my0 + im.nrows;  // rows of MCUs down to the crop's last
  const int mcux = im.mcux, interval = im.restart;
  int pred[3] = {0, 0, 0};
  int rst_left = interval;
  bool bad = false;
  // one block per iteration (every lane is at the start of a block here); the bounds do not
  // depend on the data
  int row = 0, mx = 0, blk = 0;
  const int64_t blocks = (int64_t)rows * mcux * per_mcu;
  for (int64_t it = 0; it < blocks; ++it) {
    if (blk == 0) {  // first block of an MCU
      if (interval) {
        if (rst_left == 0) {
          bad = bad || !restart_reader(r);
          pred[0] = pred[1] = pred[2] = 0;
          rst_left = interval;
        }
      }
      if (mx == 0 && row >= im.my0 && row - im.my0 < a.max_rows) {
        RowState st;
        st.pos = r.pos;
        st.nbits = r.nbits;
        st.acc = r.acc;
        st.pred[0] = (int16_t)pred[0];
        st.pred[1] = (int16_t)pred[1];
        st.pred[2] = (int16_t)pred[2];
        st.rst_left = (uint16_t)rst_left;
        st.pad = 0;
        // (the look-ahead meets the end before the row does)
        if (r.ended && !row_can_start(r.nbits - r.zeros, (uint32_t)(r.acc >> (r.zeros & 63))))
          st.pos = -1;  // a marker ended the data before this row
        states[row - im.my0] = st;
      }
      rst_left -= interval ? 1 : 0;
    }
    const int c = blk < nblk ? 0 : blk - nblk + 1;  // component
    const int t = c ? 1 : 0;                        // table set
    feed_ring(r);
    int diff;
    bad = bad || !decode_dc(r, im.dc[t], diff);
    pred[0] += c == 0 ? diff : 0;
    pred[1] += c == 1 ? diff : 0;
    pred[2] += c == 2 ? diff : 0;
    bad = bad || !decode_ac<false>(r, im.ac[t], nullptr, nullptr, false);
    if (++blk == per_mcu) {
      blk = 0;
      if (++mx == mcux) {
        mx = 0;
        ++row;
      }
    }
  }
  if (bad) {
    reinterpret_cast<CropRec*>(a.workspace + kWorkspaceHeader)[b].valid = 0;
    if (a.crop_out) a.crop_out[(int64_t)b * 6 + 5] = 0;
  }
}

// ---- symbols by table look-up, for the two kernels that follow -------------------------------------
// A step is one AC symbol, one look-up and no branch; what only some lanes need comes every kSteps
// steps: a block's end, the next one's DC coefficient, a code that is not in the table.  A lane that
// ends its block in between waits for that point, three steps on average; without the waiting every
// step would carry the instructions for all of it (about 100 instead of 31, 20 without the value).
// A lane that waits goes through the steps with an entry that moves nothing, and not around them: a
// branch per step, even one that is never taken, costs more than it can save, since a wavefront has its
// SIMD to itself (the walk below 650 -> 576 us, entropy decoding 762 -> 718 us with the value of a
// symbol made while the next one is looked up; with a way out where all lanes wait 733 us).  Files whose blocks
// are nearly all ended by their first or second symbol pay for it: whole calls with 1024 files of 256 pixels
// without markers, gradients and discs without noise at quality 50 1122 -> 1168 us, one colour 325 -> 336 (with
// a restart interval per row 306 -> 336).  A way out after the first step gives 317 and 303 there, but 982 instead of 936
// for gradients with noise at quality 90; steps of which all but the first are left out while all lanes
// waited in the round before, 1083.
constexpr int kLongCodes = 512;  // entries for codes beyond the direct part of a table
constexpr int kDirect = 1 << kFastBits;
constexpr int kSteps = 6;    // AC symbols of at most 31 bits between two points that all lanes pass
constexpr int kRounds = 2;   // such points between two at which file bytes are taken
constexpr int kAhead = 8 * kRounds;  // dwords in the ring then: kSteps symbols and two more, twice
constexpr int kDcBits = 8;
// direct part, then (from entry limit / 64 on) one entry per value of the 16 bits from `limit` on
constexpr int kCoefAc = kDirect + kLongCodes;
constexpr int kCoefTable = 2 * kCoefAc + (2 << kDcBits);
// An entry: size of the value (bits 0-3) | how far the coefficient index moves (bits 4-9; 63 from any
// index ends the block) | 32 - bits of code and value (bits 10-15).  kMiss, for a code that is not in
// the table, uses no bits and parks the lane at the end of a block, where the code is looked up.
constexpr uint32_t kMiss = (32u << 10) | (63u << 4);
constexpr uint32_t kNoStep = 32u << 10;  // no bits, no coefficient
constexpr uint32_t kNoCode = (31u << 10) | (63u << 4);  // one bit, the end of the block
__device__ static inline uint32_t coef_entry(int len, int rs) {
  const int size = rs & 15, run = rs >> 4;
  const int move = size ? run + 1 : (run == 15 ? 16 : 63);
  return (uint32_t)(((32 - len - size) << 10) | (move << 4) | size);
}

// Where the second part of an AC table starts: behind the codes of up to kFastBits bits, or later if
// what follows is too much for it (codes in between have no entry and are looked up in the ranges).
__device__ static inline uint32_t long_from(const HuffAc& h) {
  return min(max(h.range[kFastBits - 1].limit, 65536u - kLongCodes), 65536u);  // (any file's table)
}
// Bit readers hold the next 32 bits as (hi:lo) >> left; 32 - `off` of them used.
template <typename Reader>
__device__ static __forceinline__ uint32_t sym_top(const Reader& r) {
  return __builtin_amdgcn_alignbit(r.hi, r.lo, (uint32_t)r.left);
}
template <typename Reader>
__device__ static __forceinline__ void sym_skip(Reader& r, int off, uint32_t ahead) {
  const int sum = r.left + off;  // below 32: the dword in `hi` is used up
  const bool top_up = sum < 32;
  r.hi = top_up ? r.lo : r.hi;
  r.lo = top_up ? ahead : r.lo;
  r.taken += top_up ? 1 : 0;
  r.left = sum & 31;
}
template <typename Reader>
__device__ static __forceinline__ uint32_t sym_ahead(const Reader& r) {
  return r.ring[(r.taken & (kRingBytes / 4 - 1)) * kJpegThreads];
}
// `size` value bits that end `off` bits above the lowest, as the signed value they stand for (T.81
// F.2.2.1: the lower half of the range is the negative numbers); 0 for none.  With t the bits as a two's
// complement number: t + 2^size where t is negative, else t + 1 - 2^size.
__device__ static __forceinline__ int symbol_value(uint32_t top, int off, int size) {
  const int t = __builtin_amdgcn_sbfe((int)top, (uint32_t)off, (uint32_t)size);
  const int below = (int)(0xFFFFFFFFu << (size & 31));
  return t + ((below ^ (t >> 31)) + 1);
}
// The value of the symbol with entry e, found in the bits `top`, which leaves a block at its coefficient
// k - 1 (at the last one if that is behind it); `block`: 2 bytes in front of it.
__device__ static __forceinline__ void store_symbol(uint8_t* coefs, uint32_t block, int k, uint32_t top,
                                                    uint32_t e) {
  *reinterpret_cast<int16_t*>(coefs + (block + 2u * (uint32_t)min(k, 64))) =
      (int16_t)symbol_value(top, (int)(e >> 10), (int)(e & 15u));
}

// The tables of an image: AC luma, AC chroma, DC luma, DC chroma (kThreads threads).
template <int kThreads>
__device__ static void coef_tables(const JpegImage& im, uint16_t* tables) {
  const int lane = threadIdx.x;
  for (int t = 0; t < 2; ++t) {
    const HuffAc& h = im.ac[t];
    const HuffDc& g = im.dc[t];
    const uint32_t limit = long_from(h);
    uint16_t* table = tables + t * kCoefAc;
    const int direct = (int)(limit >> (16 - kFastBits));
#pragma unroll 4
    for (int j = lane; j < kDirect; j += kThreads) {
      const int e = h.fast[j];
      if (j < direct) table[j] = (uint16_t)(e ? coef_entry(e >> 8, e & 255) : kMiss);
    }
    for (int j = lane; j < kLongCodes; j += kThreads) {
      const uint32_t x = limit + (uint32_t)j;
      uint32_t e = kMiss;
      if (x <= 0xFFFFu) {
        int index;
        const int len = find_code<kFastBits>(h.range, x, index);
        if (len < 16) e = coef_entry(len + 1, h.symbols[index & 255]);
      }
      table[direct + j] = (uint16_t)e;
    }
    table = tables + 2 * kCoefAc + (t << kDcBits);
    for (int j = lane; j < (1 << kDcBits); j += kThreads) {
      int index;
      const int len = find_code<0>(g.range, (uint32_t)j << (16 - kDcBits), index);
      const int sym = len < kDcBits ? g.symbols[index & 15] : 16;
      table[j] = (uint16_t)(sym <= 11 ? coef_entry(len + 1, sym) : kMiss);
    }
  }
}

// ---- files that are one chain of codes: where does each of the crop's rows start? ----------------
// Huffman codes re-synchronise (Ferguson and Rabinowitz, "Self-synchronizing Huffman codes", 1984;
// used to decode JPEG files in parallel by Klein and Wiseman, 2003): a decoder set down anywhere in
// the data soon reads the same blocks as one that came from the start (measured over the synthetic
// files: after 700 bits at the median, 4000 at the 99th percentile; white noise 2000 / 15000).  The
// workgroup, of one wavefront or, for few and long files, of two or four (launch_sync), cuts the data
// into equal parts, 64 or, with kPartBits and more bits in each, up to a lane each.  Every lane walks its part from a
// guessed block boundary and notes the one (bit position and block of the MCU) at which it leaves
// the part, which is where the next lane should have entered.  A lane whose entry turns out to be
// another walks again, but only until it meets its earlier walk at one of the marks in its part.
// The first lane's entry is known, so after i rounds the first i lanes are right, whatever the
// guesses were: when no entry changes any more the result is that of the walk from the start (a round
// per part at most, three or four in practice).  Prefix sums over the parts' block counts and DC
// differences then say in which part each row of MCUs starts, and a lane per row walks there from
// the mark before it.
//
// The bits come from the data without byte stuffing, so topping up is a select.  1024 files of 256
// pixels: 0.58 ms, on one wavefront per SIMD, bound by the steps' issue and latency (with DC and AC
// symbols and the blocks' ends all in one step of 100 instructions 1.05 ms, by one lane per file
// 12.7 ms).
constexpr int kMarks = 3;         // block boundaries remembered inside a part (at each quarter)
constexpr int kPartBits = 2304;   // of a part, where the file makes more than 64 of them

// A block boundary of a walk and what came before it in the part.
struct alignas(16) WalkMark {
  int bit, phase_blocks;  // blocks << 3 | block of the MCU
  uint16_t dc[3];         // sums of DC differences per component, modulo 2^16 like the predictors
  uint16_t pad;
};
// What several wavefronts tell each other.
template <int kWaves>
struct SyncExchange {
  int sums[kWaves][4];   // per wavefront: blocks, DC differences
  int asked[2][kWaves];  // has a lane to walk again? (in turn)
  int tail[4];           // last part: block it is left at; DC differences of an MCU of zero bits
};
template <>
struct SyncExchange<1> {};  // (exchanged in registers)
template <int kWaves>
struct JpegSyncLds : SyncExchange<kWaves> {
  uint16_t table[kCoefTable];
  uint32_t ring[kWaves][kRingBytes / 4][kJpegThreads];  // big-endian dwords of the data
  WalkMark mark[kMarks + 1][kWaves * kJpegThreads];     // [0]: the entry; bit -1 = none
  // per part: what came before it; until that is known where the part is left, bit and block
  int first_block[kWaves * kJpegThreads], dc[3][kWaves * kJpegThreads];
};
// (48 bytes more and it is seven: whole calls with 2000 files of 256 pixels 1.69 ms instead of 1.28, 4096 2.88
// instead of 2.54, 2000 of 500 pixels 4.34 instead of 3.51)
static_assert(sizeof(JpegSyncLds<1>) <= 160 * 1024 / 8, "eight files at a time on a compute unit");
// Reads the data of one image, a bit position at a time.  (hi:lo) >> left are the next 32 bits.
struct CleanReader {
  const uint8_t* clean;
  int bytes;
  uint32_t* ring;  // this lane's column
  uint32_t hi, lo;
  int left;        // 0..31
  int taken;       // dwords of the data that have been in hi / lo
  int have;        // dwords that have been in the ring (multiple of 8)
  bool pending;    // `next` is dwords have .. have + 7
  u32x4_a8 next[2];
};
__device__ static __forceinline__ void clean_request(CleanReader& r) {
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int at = 4 * r.have + 16 * j;
    r.next[j] = u32x4_a8{0u, 0u, 0u, 0u};
    // (the slot goes on for 16 bytes and more behind the data)
    if (at < r.bytes) r.next[j] = *reinterpret_cast<const u32x4_a8*>(r.clean + at);
  }
  r.pending = true;
}
__device__ static __forceinline__ void clean_accept(CleanReader& r) {
  const int i = r.have & (kRingBytes / 4 - 1);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int good = r.bytes - 4 * (r.have + j);  // bytes of the dword that exist: zeros follow
    uint32_t w = __builtin_bswap32(r.next[j >> 2][j & 3]);
    if (good < 4) w = good <= 0 ? 0u : w & ~(0xFFFFFFFFu >> (8 * good));
    r.ring[(i + j) * kJpegThreads] = w;
  }
  r.have += 8;
  r.pending = false;
}
__device__ static __forceinline__ void clean_feed(CleanReader& r) {
  if (r.pending) clean_accept(r);
#pragma unroll 1
  while (r.have - r.taken < kAhead) {
    clean_request(r);
    clean_accept(r);
  }
  // the 8 dwords to come replace those 32 back, which must have been taken
  if (r.have - r.taken <= kRingBytes / 4 - 8) clean_request(r);
}
__device__ static __forceinline__ void clean_open(CleanReader& r, int bit) {
  const int w = bit >> 5;
  r.left = -bit & 31;
  r.have = w & ~7;
#pragma unroll 1
  for (int j = 0; j < 3; ++j) {  // (the first feed comes after one DC symbol)
    clean_request(r);
    clean_accept(r);
  }
  r.hi = r.ring[(w & (kRingBytes / 4 - 1)) * kJpegThreads];
  r.taken = w + (r.left ? 2 : 1);
  r.lo = r.ring[((r.taken - 1) & (kRingBytes / 4 - 1)) * kJpegThreads];
}
__device__ static inline int clean_bit(const CleanReader& r) { return 32 * r.taken - 32 - r.left; }

// What the wavefront does next: every lane walks its part (again), the zero bits behind data that
// ends early are looked at, the rows' starts are walked to, then their pieces'.
enum class SyncStage { kParts, kTail, kRows, kPieces };

template <int kWaves>
__global__ __launch_bounds__(kWaves * kJpegThreads) void jpeg_sync_kernel(JpegArgs a) {
  constexpr int kParts = kWaves * kJpegThreads;
  __shared__ JpegSyncLds<kWaves> s;
  const int lane = threadIdx.x;  // of the workgroup: the part
  const int wave = __builtin_amdgcn_readfirstlane(lane / kJpegThreads);
  const int b = (int)blockIdx.x;
  const JpegImage* im = &reinterpret_cast<const JpegPrepared*>(a.prepared)[b].im;
  const int live = im->live;
  if (!live || im->clean_bytes < 0) return;
  const int nblk = im->hs * im->hs, last_phase = nblk + 1, per_mcu = nblk + 2;
  const int my0 = im->my0, nrows = min(im->nrows, a.max_rows);
  const int row_blocks = im->mcux * per_mcu;
  const int ncols = im->mx1 - im->mx0 + 1, sub = pieces_per_row(nrows, ncols);
  const uint32_t limit_y = long_from(im->ac[0]), limit_c = long_from(im->ac[1]);
  coef_tables<kParts>(*im, s.table);
  for (int i = 0; i <= kMarks; ++i) s.mark[i][lane].bit = -1;
  __syncthreads();

  CleanReader r;
  r.clean = a.regions + im->region_off;
  r.bytes = im->clean_bytes & (kCutShort - 1);
  r.ring = &s.ring[wave][0][lane % kJpegThreads];
  const int bits = 8 * r.bytes;  // below 2^30 (clean_fits)
  // (the lanes behind the last part have nothing to do until the rows)
  const int parts = max(kJpegThreads, min(kParts, bits / kPartBits));
  const int quarter = (int)((((int64_t)bits + parts - 1) / parts + 31) & ~(int64_t)31) / 4;
  constexpr int kPartQuarters = kMarks + 1;
  const int begin = min(bits, lane * kPartQuarters * quarter);
  const int part_end = min(bits, begin + kPartQuarters * quarter);
  constexpr int kNever = 0x7FFFFFFF;

  // the lane's part as its latest walk left it
  int enter = begin, enter_phase = 0;
  int leave = 0, leave_phase = 0, blocks = 0, bad_at = kNever;
  int dc0 = 0, dc1 = 0, dc2 = 0;
  int first_block = 0, total = 0, row = lane, from = 0;
  bool bad = false;
  // (as row_can_start; a file that merely stops has none)
  const int padding = (im->clean_bytes & kCutShort)
                          ? 0
                          : min(__builtin_ctz(~(uint32_t)r.clean[max(r.bytes - 1, 0)]), 7);
  SyncStage stage = SyncStage::kParts;
  int round = 0;
  for (;;) {
    // ---- where does this lane's next walk start, and where does it end? ----
    bool go;
    int bit, phase, limit, end, base0 = 0, base1 = 0, base2 = 0;
    if (stage == SyncStage::kParts) {
      if (round) {
        int e, ph;
        if constexpr (kWaves == 1) {
          e = __shfl_up(leave, 1);
          ph = __shfl_up(leave_phase, 1);
        } else {
          s.first_block[lane] = leave;
          s.dc[0][lane] = leave_phase;
          __syncthreads();
          e = s.first_block[max(lane - 1, 0)];
          ph = s.dc[0][max(lane - 1, 0)];
        }
        if (lane == 0) {
          e = 0;
          ph = 0;
        }
        if (lane >= parts) {
          e = enter;
          ph = enter_phase;
        }
        go = e != enter || ph != enter_phase;
        enter = e;
        enter_phase = ph;
      } else {
        go = lane < parts;
      }
      bool more = __builtin_amdgcn_ballot_w64(go) != 0;
      if constexpr (kWaves > 1) {  // (the barrier also ends the exchange above)
        if (lane % kJpegThreads == 0) s.asked[round & 1][wave] = more ? 1 : 0;
        __syncthreads();
        int any = 0;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) any |= s.asked[round & 1][w];
        more = any != 0;
      }
      if (round > parts || !more) {
        // blocks and DC differences before each part
        first_block = blocks;
        int d0 = dc0, d1 = dc1, d2 = dc2;
        for (int off = 1; off < kWave; off <<= 1) {
          const int t = __shfl_up(first_block, off), t0 = __shfl_up(d0, off),
                    t1 = __shfl_up(d1, off), t2 = __shfl_up(d2, off);
          if (lane % kWave >= off) {
            first_block += t;
            d0 += t0;
            d1 += t1;
            d2 += t2;
          }
        }
        if constexpr (kWaves == 1) {
          total = __shfl(first_block, kWave - 1);
        } else {
          if (lane % kWave == kWave - 1) {
            s.sums[wave][0] = first_block;
            s.sums[wave][1] = d0;
            s.sums[wave][2] = d1;
            s.sums[wave][3] = d2;
          }
          __syncthreads();
          total = 0;
#pragma unroll
          for (int w = 0; w < kWaves; ++w) {
            total += s.sums[w][0];
            if (w >= wave) continue;
            first_block += s.sums[w][0];
            d0 += s.sums[w][1];
            d1 += s.sums[w][2];
            d2 += s.sums[w][3];
          }
        }
        first_block -= blocks;
        s.first_block[lane] = first_block;
        s.dc[0][lane] = d0 - dc0;
        s.dc[1][lane] = d1 - dc1;
        s.dc[2][lane] = d2 - dc2;
        s.mark[0][lane] = WalkMark{enter, enter_phase, {0, 0, 0}, 0};
        __syncthreads();
        // the walk ends with the crop's last row; a bad code up to there flags the sample
        bad = bad_at != kNever && first_block + bad_at < (my0 + nrows) * row_blocks;
        stage = SyncStage::kTail;
        continue;
      }
      bit = enter;
      phase = enter_phase;
      limit = kNever;
      end = part_end;
    } else if (stage == SyncStage::kTail) {
      // where the data ends early zero bits follow, block after block of a component the same: one
      // MCU tells
      go = lane == parts - 1 && total < (my0 + nrows) * row_blocks;
      bit = leave;
      phase = leave_phase;
      limit = per_mcu;
      end = kNever;
    } else {
      if (stage == SyncStage::kRows && row - lane >= nrows) {  // (the same for all lanes)
        // (files whose data ends early are decoded row by row)
        if (live != kLiveCoefs || total < (my0 + nrows) * row_blocks || nrows != im->nrows ||
            !pieces_fit(a, im->size, im->scan_off, nrows))
          break;
        stage = SyncStage::kPieces;
        row = lane / sub;
      }
      int target = (my0 + row) * row_blocks;
      if (stage == SyncStage::kPieces)
        target += (im->mx0 + (lane - row * sub) * ncols / sub) * per_mcu;
      go = row < nrows && (target < total || target == 0);
      from = 0;  // the last part that starts at or before the row's first block
      for (int step = kParts / 2; step > 0; step >>= 1)
        if (s.first_block[from + step] <= target) from += step;
      const int inside = target - s.first_block[from];
      WalkMark m = s.mark[0][from];
      for (int i = 1; i <= kMarks; ++i) {
        const WalkMark t = s.mark[i][from];
        if (t.bit >= 0 && (t.phase_blocks >> 3) <= inside) m = t;
      }
      bit = m.bit;
      phase = m.phase_blocks & 7;
      base0 = s.dc[0][from] + m.dc[0];
      base1 = s.dc[1][from] + m.dc[1];
      base2 = s.dc[2][from] + m.dc[2];
      limit = inside - (m.phase_blocks >> 3);
      end = kNever;
    }

    // ---- the walk: blocks until one ends at or behind bit `end`, or `limit` blocks are done ----
    // walk_bad: the first block with a code that does not exist or a run past its end (such a code
    // counts as one bit and ends the block, which only matters after a wrong guess)
    int done = 0, sum0 = 0, sum1 = 0, sum2 = 0, walk_bad = kNever;
    const bool asked = go;
    int next_mark = stage == SyncStage::kParts ? 1 : kMarks + 1;
    int mark_at = stage == SyncStage::kParts ? begin + quarter : kNever;
    bool met = false;
    go = go && bit < end && limit > 0;
    if (go) {
      clean_open(r, bit);
      int k = 64, ac = 0, round = 0;  // (as behind a block before the first)
      uint32_t e = 0, ac_limit = 0;
      bool is_chroma = false;
      done = -1;
      phase = phase == 0 ? last_phase : phase - 1;
      while (go) {
        if (__builtin_expect(k >= 64 && e == kMiss, 0)) {
          int index;
          const HuffAc& h = im->ac[is_chroma];
          const uint32_t ahead = sym_ahead(r), top = sym_top(r);
          const int len = find_code<0>(h.range, top >> 16, index);
          walk_bad = len < 16 ? walk_bad : min(walk_bad, done);
          e = len < 16 ? coef_entry(len + 1, h.symbols[index & 255]) : kNoCode;
          k += (int)((e >> 4) & 63u) - 63;
          sym_skip(r, (int)(e >> 10), ahead);
        }
        if (k >= 64) {
          if ((e & 15u) != 0u && k > 64) walk_bad = min(walk_bad, done);
          ++done;
          phase = phase == last_phase ? 0 : phase + 1;
          const int now = clean_bit(r);
          go = done == 0 || (now < end && done < limit);
          if (done > 0 && now >= mark_at) {
            // the first block boundary at or behind one or more of the part's quarters
            WalkMark& m = s.mark[next_mark][lane];
            const WalkMark old = m;
            const WalkMark here{now, (done << 3) | phase,
                                {(uint16_t)sum0, (uint16_t)sum1, (uint16_t)sum2}, 0};
            m = here;
            const int old_blocks = old.phase_blocks >> 3;
            if (old.bit == now && (old.phase_blocks & 7) == phase &&
                (bad_at == kNever || bad_at >= old_blocks)) {
              // the earlier walk came by here, and its first bad code, if any, came later: the rest
              // of the part is as it was
              const int more = done - old_blocks;
              const int m0 = sum0 - old.dc[0], m1 = sum1 - old.dc[1], m2 = sum2 - old.dc[2];
              for (int j = next_mark + 1; j <= kMarks; ++j) {
                WalkMark& t = s.mark[j][lane];
                if (t.bit < 0) continue;
                t.phase_blocks += more << 3;
                t.dc[0] = (uint16_t)(t.dc[0] + m0);
                t.dc[1] = (uint16_t)(t.dc[1] + m1);
                t.dc[2] = (uint16_t)(t.dc[2] + m2);
              }
              walk_bad = min(walk_bad, bad_at == kNever ? kNever : bad_at + more);
              done = blocks + more;
              sum0 = dc0 + m0;
              sum1 = dc1 + m1;
              sum2 = dc2 + m2;
              met = true;
              go = false;
            } else {
              ++next_mark;
              mark_at += quarter;
              // (a block longer than a quarter: marks it went past do not exist)
              while (next_mark <= kMarks && now >= mark_at) {
                s.mark[next_mark][lane].bit = -1;
                ++next_mark;
                mark_at += quarter;
              }
              if (next_mark > kMarks) mark_at = kNever;
            }
          }
          if (go) {  // the next block's DC difference
            is_chroma = phase >= nblk;
            ac_limit = is_chroma ? limit_c : limit_y;
            ac = is_chroma ? kCoefAc : 0;
            const uint32_t ahead = sym_ahead(r), top = sym_top(r);
            uint32_t d =
                s.table[2 * kCoefAc + (is_chroma ? 1 << kDcBits : 0) + (int)(top >> (32 - kDcBits))];
            k = 1;
            e = 0;
            if (__builtin_expect(d == kMiss, 0)) {
              int index;
              const HuffDc& h = im->dc[is_chroma];
              const int len = find_code<0>(h.range, top >> 16, index);
              const int sym = len < 16 ? h.symbols[index & 15] : 16;
              d = kNoCode;
              if (sym <= 11) {
                d = coef_entry(len + 1, sym);
              } else {
                walk_bad = min(walk_bad, done);
                k = 64;
              }
            }
            const int size = (int)(d & 15u), off = (int)(d >> 10);
            const int diff = symbol_value(top, off, size);
            sym_skip(r, off, ahead);
            sum0 += is_chroma ? 0 : diff;
            sum1 += phase == nblk ? diff : 0;
            sum2 += phase == last_phase ? diff : 0;
          }
        }
        if (!go) break;
        if (round == 0) clean_feed(r);
        round = round + 1 == kRounds ? 0 : round + 1;
#pragma unroll
        for (int i = 0; i < kSteps; ++i) {
          const bool on = k < 64;
          const uint32_t ahead = sym_ahead(r), top = sym_top(r);
          const uint32_t beyond = __builtin_elementwise_sub_sat(top >> 16, ac_limit);
          const uint32_t found =
              s.table[(uint32_t)ac + min(top >> (32 - kFastBits), ac_limit >> (16 - kFastBits)) + beyond];
          e = on ? found : e;
          const uint32_t step = on ? found : kNoStep;
          k += (int)((step >> 4) & 63u);
          sym_skip(r, (int)(step >> 10), ahead);
        }
      }
      bit = clean_bit(r);
    }

    // ---- what it means ----
    if (stage == SyncStage::kParts) {
      if (asked) {
        if (!met) {
          leave = bit;
          leave_phase = phase;
          // marks of the earlier walk that this one did not reach
          for (int j = next_mark; j <= kMarks; ++j) s.mark[j][lane].bit = -1;
        }
        blocks = done;
        dc0 = sum0;
        dc1 = sum1;
        dc2 = sum2;
        bad_at = walk_bad;
      }
      ++round;
    } else if (stage == SyncStage::kTail) {
      bad = bad || (walk_bad != kNever && total + walk_bad < (my0 + nrows) * row_blocks);
      if (__builtin_expect((im->clean_bytes & kCutShort) != 0, 0)) {
        // Behind a file that merely stops a row is zero bits, and so are the blocks between the last
        // that the data began and the row's first (the rest of an MCU, then whole ones).
        int ph, mcu0, mcu1, mcu2, end0 = 0, end1 = 0, end2 = 0;
        if constexpr (kWaves == 1) {
          ph = __shfl(leave_phase, kWave - 1);
          mcu0 = __shfl(sum0, kWave - 1);
          mcu1 = __shfl(sum1, kWave - 1);
          mcu2 = __shfl(sum2, kWave - 1);
          end0 = s.dc[0][kWave - 1] + __shfl(dc0, kWave - 1);
          end1 = s.dc[1][kWave - 1] + __shfl(dc1, kWave - 1);
          end2 = s.dc[2][kWave - 1] + __shfl(dc2, kWave - 1);
        } else {
          if (lane == parts - 1) {
            s.tail[0] = leave_phase;
            s.tail[1] = sum0;
            s.tail[2] = sum1;
            s.tail[3] = sum2;
          }
          __syncthreads();
          ph = s.tail[0];
          mcu0 = s.tail[1];
          mcu1 = s.tail[2];
          mcu2 = s.tail[3];
          for (int w = 0; w < kWaves; ++w) {
            end0 += s.sums[w][1];
            end1 += s.sums[w][2];
            end2 += s.sums[w][3];
          }
        }
        const int rest = ph ? per_mcu - ph : 0;
        for (int i = lane; i < nrows; i += kParts) {
          const int target = (my0 + i) * row_blocks;
          if (target < total || target == 0) continue;
          const int whole = (target - total - rest) / per_mcu;
          RowState st;
          st.pos = im->size;
          st.nbits = 0;
          st.acc = 0;
          st.pred[0] = (int16_t)(end0 + whole * mcu0 + (ph ? max(nblk - ph, 0) * (mcu0 / nblk) : 0));
          st.pred[1] = (int16_t)(end1 + (whole + (ph && ph <= nblk ? 1 : 0)) * mcu1);
          st.pred[2] = (int16_t)(end2 + (whole + (ph ? 1 : 0)) * mcu2);
          st.rst_left = 0;
          st.pad = 0;
          (reinterpret_cast<RowState*>(a.row_states) + (int64_t)b * a.max_rows)[i] = st;
        }
      }
      stage = SyncStage::kRows;
    } else {
      const bool piece = stage == SyncStage::kPieces;
      const bool first_row = my0 + row == 0 && !piece;
      // (bit < bits: the walk counted this block, or it is the file's first)
      if (asked && (first_row || piece || bits - bit > padding)) {
        const uint8_t* file = a.files + im->origin;
        const int32_t* map =
            reinterpret_cast<const int32_t*>(r.clean + clean_map_offset(im->size, im->scan_off));
        const int at = bit >> 3, used = bit & 7;
        int pos = first_row ? im->scan_off : map[at >> 4];
        for (int i = 0; i < (at & 15); ++i) pos += file[pos] == 0xFF ? 2 : 1;
        RowState st;
        st.nbits = used ? 8 - used : 0;
        st.acc = used ? (uint64_t)(file[pos] & (0xFF >> used)) : 0;
        st.pos = used ? pos + (file[pos] == 0xFF ? 2 : 1) : pos;
        st.pred[0] = (int16_t)(base0 + sum0);
        st.pred[1] = (int16_t)(base1 + sum1);
        st.pred[2] = (int16_t)(base2 + sum2);
        st.rst_left = 0;
        st.pad = 0;
        if (piece) piece_states(a, im->region_off)[lane] = st;
        else (reinterpret_cast<RowState*>(a.row_states) + (int64_t)b * a.max_rows)[row] = st;
      }
      if (piece) {
        if (lane == 0) reinterpret_cast<JpegPrepared*>(a.prepared)[b].im.live = kLivePieces;
        break;
      }
      row += kParts;
    }
  }
  if (bad) {
    reinterpret_cast<CropRec*>(a.workspace + kWorkspaceHeader)[b].valid = 0;
    if (a.crop_out) a.crop_out[(int64_t)b * 6 + 5] = 0;
  }
}

template <int kGroup>
__global__ __launch_bounds__(kJpegThreads) void jpeg_decode_kernel(JpegArgs a) {
  __shared__ JpegLds<kGroup> s;
  const int lane = threadIdx.x;
  const int b0 = (int)blockIdx.x * kGroup;
  const int nimg = min(kGroup, a.B - b0);
  bool need = false;
  if (lane < nimg) {
    const JpegImage& im = reinterpret_cast<const JpegPrepared*>(a.prepared)[b0 + lane].im;
    need = im.live == kLivePlanes;
  }
  if (__builtin_amdgcn_ballot_w64(need) == 0) return;  // the usual case: all decoded already
  {  // the images' tables, as the table kernel left them
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4* src = reinterpret_cast<const u32x4*>(a.prepared + (size_t)b0 * sizeof(JpegPrepared));
    u32x4* dst = reinterpret_cast<u32x4*>(&s.img[0]);
    const int n16 = nimg * (int)(sizeof(JpegPrepared) / 16);
    for (int i = lane; i < n16; i += kJpegThreads) dst[i] = src[i];
  }
  __syncthreads();

  // the rows of MCUs of the group's images, one after the other, are dealt to the lanes
  int first_task[kGroup + 1];
  first_task[0] = 0;
#pragma unroll
  for (int i = 0; i < kGroup; ++i)
    first_task[i + 1] =
        first_task[i] +
        (i < nimg && s.img[i].im.live == kLivePlanes ? min(s.img[i].im.nrows, a.max_rows) : 0);
  const int ntasks = first_task[kGroup];
  int16_t* coef = &s.coef[0][lane];  // element k at coef[k * 64]
#pragma unroll 1
  for (int task = lane; task < ntasks; task += kJpegThreads) {
    int slot = 0, slot_first = 0;
#pragma unroll
    for (int i = 1; i < kGroup; ++i) {
      if (task >= first_task[i]) {
        slot = i;
        slot_first = first_task[i];
      }
    }
    const int row = task - slot_first;  // row of MCUs inside the crop's range
    const JpegImage& im = s.img[slot].im;
    const int b = b0 + slot;
    const RowState st = (reinterpret_cast<const RowState*>(a.row_states) +
                         (int64_t)b * a.max_rows)[row];
    const int hs = im.hs, mcu = 8 * hs;
    const int mx0 = im.mx0, mx1 = im.mx1, region_w = im.region_w;
    // the image's slot of the plane buffer: Y (region_w wide), then Cb and Cr (region_w / hs wide)
    const int chroma_w = region_w / hs;
    uint8_t* plane_y = a.planes + im.region_off;
    uint8_t* plane_cb = plane_y + (int64_t)im.nrows * mcu * region_w;
    uint8_t* plane_cr = plane_cb + (int64_t)im.nrows * 8 * chroma_w;
    const bool found = st.pos >= im.scan_off && st.pos <= im.size;
    BitReader r;
    reader_for(r, a, im, &s.ring[0][lane]);
    r.ended = !found;  // start unknown: zero bits, and the sample is flagged below
    if (found) {
      open_at(r, st);
    } else {
      open_reader(r, im.scan_off);
    }
    int pred_y = st.pred[0], pred_cb = st.pred[1], pred_cr = st.pred[2];
    const int interval = im.restart;
    int rst_left = st.rst_left;
    const int nblk = hs * hs;  // luma blocks per MCU
    bool bad = !found;
    for (int mx = 0; mx <= mx1; ++mx) {
      if (interval) {  // a restart boundary inside the row
        if (mx > 0 && rst_left == 0) {
          bad = bad || !restart_reader(r);
          pred_y = pred_cb = pred_cr = 0;
          rst_left = interval;
        }
        --rst_left;
      }
      const bool want = mx >= mx0;
      const int x0 = (mx - mx0) * mcu, y0 = row * mcu;
      for (int blk = 0; blk < nblk + 2; ++blk) {
        const int c = blk < nblk ? 0 : blk - nblk + 1;  // component
        const int t = c ? 1 : 0;                        // table set
        if (want)
          for (int i = 0; i < 64; ++i) coef[i * kJpegThreads] = 0;
        feed_ring(r);
        int diff;
        bad = bad || !decode_dc(r, im.dc[t], diff);
        pred_y += c == 0 ? diff : 0;
        pred_cb += c == 1 ? diff : 0;
        pred_cr += c == 2 ? diff : 0;
        const int dcv = c == 0 ? pred_y : (c == 1 ? pred_cb : pred_cr);
        const uint16_t* qz = im.qz[t];
        if (want) coef[0] = (int16_t)min(max(dcv * (int)(qz[0] & 255), -32767), 32767);
        bad = bad || !decode_ac<true>(r, im.ac[t], qz, coef, want);
        if (!want) continue;
        idct_columns(coef);
        // the block's rows, eight samples = one 8-byte store each (rows of every plane start on
        // 8-byte boundaries: widths are multiples of 8)
        uint8_t* out;
        int pitch;
        if (c == 0) {
          pitch = region_w;
          out = plane_y + (int64_t)(y0 + (blk / hs) * 8) * region_w + x0 + (blk % hs) * 8;
        } else {
          pitch = chroma_w;
          out = (c == 1 ? plane_cb : plane_cr) + (int64_t)row * 8 * chroma_w + (mx - mx0) * 8;
        }
        for (int y = 0; y < 8; ++y) {
          int v[8];
          idct_row(coef, y, v);
          const uint32_t lo = (uint32_t)v[0] | ((uint32_t)v[1] << 8) | ((uint32_t)v[2] << 16) |
                              ((uint32_t)v[3] << 24);
          const uint32_t hi = (uint32_t)v[4] | ((uint32_t)v[5] << 8) | ((uint32_t)v[6] << 16) |
                              ((uint32_t)v[7] << 24);
          *reinterpret_cast<u32x2*>(out + (int64_t)y * pitch) = u32x2{lo, hi};
        }
      }
    }
    if (bad) {
      reinterpret_cast<CropRec*>(a.workspace + kWorkspaceHeader)[b].valid = 0;
      if (a.crop_out) a.crop_out[(int64_t)b * 6 + 5] = 0;
    }
  }
}


// ---- the crop's coefficients, entropy decoding only ------------------------------------------------
// A lane per row of MCUs, as above, but the lanes do not wait for the longest block among them: a step
// is one AC symbol, one table look-up and no branch in the usual case, and its value goes straight to
// its place (zig-zag order) in the image's coefficients, which the table kernel has cleared.  Every
// kSteps steps come the things that only some lanes need: the next block's DC coefficient and the
// file bytes; a lane that ends its block in between waits for that point, three steps on average.
// There is one wavefront per SIMD at most, so what counts is the number of instructions and LDS
// round trips per symbol; the inverse transform, which needs neither, is left to jpeg_idct_kernel,
// where it fills the chip.  Every step stores: a symbol without a value a zero where one is (the
// last of the coefficients that it skips), and the blocks to the left of the crop go where the
// row's first block will be, which is cleared once they are behind. The file's bytes lose their
// stuffing on the way into the ring (SymbolReader): topping up the bit buffer is then a select.
// 4096 files of 256 pixels with a restart interval per row: 0.72 ms and 0.22 ms for the
// inverse transform and colours (entropy decoding and transform by the same lanes, block after
// block, as in jpeg_decode_kernel: 1.42 ms and 0.20 ms for the colours); 1024 files without
// markers, rows in pieces: 0.18 + 0.06 ms (1.34 + 0.04 ms).
struct SymbolReader {
  const uint8_t* chunks;  // as in BitReader
  int64_t chunks_bytes;
  uint32_t* ring;  // this lane's column: big-endian dwords without byte stuffing
  int skew, start, n;
  int at;          // position (from `chunks`) of the 16 bytes in `next`, or of those to request
  uint32_t part;   // the low nb bytes wait for a whole dword
  int nb;
  bool pend_ff;    // the last byte was 0xFF: its follower says what it is
  bool ended;      // marker or end of the file: zeros from here on
  bool pending;
  u32x4_a8 next;
  uint32_t hi, lo;  // (hi:lo) >> left are the next 32 bits
  int left, taken, have;  // 0..31 / dwords that have been in hi, lo / in the ring
};
__device__ static __forceinline__ void sym_request(SymbolReader& r) {
  if (!r.ended) r.next = load_chunk(r.chunks, r.chunks_bytes, r.at);
  r.pending = true;
}
// Byte stuffing leaves four bytes at a time: of the bytes that are not there to stay (a zero behind a 0xFF;
// a 0xFF in the last place, which waits for its follower and then takes that one's place) there is one at
// most, as a rule, and it is taken out without looking at single bytes.  (A third of a wavefront's dwords has
// a 0xFF in one of its lanes: entropy decoding of 4096 files 805 -> 762 us against single bytes for all
// of them.)  What is more than that goes byte by byte: two such bytes, a marker, the ends of the row's
// data.
__device__ static __forceinline__ void sym_accept(SymbolReader& r) {
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t x = r.ended ? 0u : r.next[j];
    const int p = r.at + 4 * j - r.skew;  // file position
    const uint32_t ff = ((x & 0x7F7F7F7Fu) + 0x01010101u) & x & 0x80808080u;  // bit 7 of bytes 0xFF
    const uint32_t pend = r.pend_ff ? 0xFFu : 0u;
    const uint32_t behind = (ff << 8) | (pend & 0x80u);    // of bytes behind one
    const uint32_t drop = (ff << 8) | (ff & 0x80000000u);  // of bytes that go, or wait
    const bool odd = ((drop & (drop - 1u)) | (x & ((behind << 1) - (behind >> 7)))) != 0u;
    const bool inside = (int)r.ended | ((int)(p >= r.start) & (int)(p + 4 <= r.n));
    if ((int)!odd & (int)inside) {
      const uint32_t low = (drop >> 7) - 1u;  // the bytes in front of it (all of them if there is none)
      const uint32_t y = x | pend;
      const uint32_t be = __builtin_bswap32((y & low) | ((y >> 8) & ~low));
      const int out = drop ? 1 : 0;
      r.ring[(r.have & (kRingBytes / 4 - 1)) * kJpegThreads] =
          __builtin_amdgcn_alignbit(r.part, be, 8u * (uint32_t)r.nb);  // (to be written again if too short)
      r.part = be >> (8 * out);
      const int bytes = r.nb + 4 - out;
      r.have += bytes >> 2;
      r.nb = bytes & 3;
      r.pend_ff = (ff >> 31) != 0u;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint32_t b = (x >> (8 * i)) & 0xFFu;
        const bool here = !r.ended && p + i >= r.start;
        r.ended = r.ended || (here && (p + i >= r.n || (r.pend_ff && b != 0u)));
        const bool data = here && !r.ended && (r.pend_ff || b != 0xFFu);
        const uint32_t v = r.pend_ff ? 0xFFu : b;
        r.pend_ff = here && !r.ended && !r.pend_ff && b == 0xFFu;
        r.part = data ? (r.part << 8) | v : r.part;
        r.nb += data ? 1 : 0;
        if (r.nb == 4) {
          r.ring[(r.have & (kRingBytes / 4 - 1)) * kJpegThreads] = r.part;
          ++r.have;
          r.nb = 0;
        }
      }
    }
  }
  r.at += 16;
  r.pending = false;
}
__device__ static __forceinline__ void sym_feed(SymbolReader& r) {
  if (r.pending) sym_accept(r);
#pragma unroll 1
  while (r.have - r.taken < kAhead) {
    sym_request(r);
    sym_accept(r);
  }
  // room: at most four dwords come out of 16 bytes, which last for a little more than two rounds
  if (r.have - r.taken <= kRingBytes / 4 - 4) sym_request(r);
}
// Opens the reader in a row's state: its unread bits (up to 64) are the first two dwords.
__device__ static __forceinline__ void sym_open(SymbolReader& r, const RowState& st) {
  r.start = st.pos;
  r.at = (st.pos + r.skew) & ~15;
  r.part = 0;
  r.nb = 0;
  r.pend_ff = r.ended = r.pending = false;
  r.ring[0] = (uint32_t)(st.acc >> 32);
  r.ring[kJpegThreads] = (uint32_t)st.acc;
  r.have = 2;
#pragma unroll 1
  while (r.have < 4 + kAhead) {
    sym_request(r);
    sym_accept(r);
  }
  const int bit = 64 - st.nbits;
  const int w = bit >> 5;
  r.left = -bit & 31;
  r.hi = r.ring[w * kJpegThreads];
  r.taken = w + (r.left ? 2 : 1);
  r.lo = r.ring[(r.taken - 1) * kJpegThreads];
}

template <int kGroup>
struct JpegEntropyLds {
  uint16_t table[kGroup * kCoefTable];  // per image AC luma, AC chroma, DC luma, DC chroma
  uint32_t ring[kRingBytes / 4][kJpegThreads];
};

template <int kGroup>
__global__ __launch_bounds__(kJpegThreads) void jpeg_entropy_kernel(JpegArgs a) {
  __shared__ JpegEntropyLds<kGroup> s;
  const int lane = threadIdx.x;
  // the first half of the workgroups stores to the plane buffer, the second the spilled rows
  const uint32_t half = gridDim.x / 2;
  const bool spill = blockIdx.x >= half;
  const int b0 = (int)(blockIdx.x - (spill ? half : 0u)) * kGroup;
  const int nimg = min(kGroup, a.B - b0);
  const JpegPrepared* prepared = reinterpret_cast<const JpegPrepared*>(a.prepared) + b0;
  // (below 2^32: a side of at most 32768, and one image per group where a slot is that large)
  const uint32_t slot_bytes = (uint32_t)a.slot_side * (uint32_t)a.slot_side * 3u;
  uint8_t* coefs = (spill ? a.regions : a.planes) + (int64_t)b0 * slot_bytes;  // (slots follow each other)
  int first_task[kGroup + 1];
  first_task[0] = 0;
#pragma unroll
  for (int i = 0; i < kGroup; ++i) {
    int rows = 0;
    if (i < nimg && prepared[i].im.live >= kLiveCoefs) {
      const JpegImage& im = prepared[i].im;
      const int ncols = im.mx1 - im.mx0 + 1;
      rows = spill ? 0 : min(im.nrows, a.max_rows);
      if (im.live == kLivePieces) rows *= pieces_per_row(im.nrows, ncols);
      if (im.live == kLiveSpill) {
        const uint32_t row_bytes = (uint32_t)ncols * (uint32_t)((im.hs * im.hs + 2) * kBlockBytes);
        const int spilled = spilled_rows(slot_bytes, row_bytes, im.nrows);
        rows = spill ? spilled : rows - spilled;
        if (spill) {  // (not earlier: the walk's copy of the file's data was there)
          typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
          const uint32_t bytes = (uint32_t)spilled * row_bytes;
          u32x4* coef = reinterpret_cast<u32x4*>(coefs + (uint32_t)(i + 1) * slot_bytes - bytes);
          for (uint32_t j = (uint32_t)lane; j < bytes / 16; j += kJpegThreads)
            coef[j] = u32x4{0u, 0u, 0u, 0u};
        }
      }
    }
    first_task[i + 1] = first_task[i] + rows;
    if (rows == 0) continue;
    coef_tables<kJpegThreads>(prepared[i].im, s.table + i * kCoefTable);
  }
  __syncthreads();
  const int ntasks = first_task[kGroup];

#pragma unroll 1
  for (int task = lane; task < ntasks; task += kJpegThreads) {
    int slot = 0, slot_first = 0;
#pragma unroll
    for (int i = 1; i < kGroup; ++i) {
      if (task >= first_task[i]) {
        slot = i;
        slot_first = first_task[i];
      }
    }
    const JpegImage& im = prepared[slot].im;
    const int b = b0 + slot;
    const int nblk = im.hs * im.hs, last_phase = nblk + 1, per_mcu = nblk + 2;
    const int mx0 = im.mx0, mx1 = im.mx1, ncols = mx1 - mx0 + 1;
    int row = task - slot_first;  // row of MCUs inside the crop's range
    uint32_t origin = (uint32_t)slot * slot_bytes;  // where row 0 would be
    if (im.live == kLiveSpill) {
      const uint32_t row_bytes = (uint32_t)(ncols * per_mcu * kBlockBytes);
      const int spilled = spilled_rows(slot_bytes, row_bytes, im.nrows);
      row += spill ? 0 : spilled;
      origin += (spill ? slot_bytes : 0u) - (uint32_t)spilled * row_bytes;
    }
    int first = 0;                // MCU of the crop that the lane's blocks are stored from
    int skip = mx0 * per_mcu, total = (mx1 + 1) * per_mcu;  // blocks
    RowState st = (reinterpret_cast<const RowState*>(a.row_states) + (int64_t)b * a.max_rows)[
        min(row, a.max_rows - 1)];
    bool bad = false;
    if (im.live == kLivePieces) {
      const int sub = pieces_per_row(im.nrows, ncols);
      st = piece_states(a, im.region_off)[row];
      const int piece = row % sub;
      row /= sub;
      first = piece * ncols / sub;
      skip = 0;
      total = ((piece + 1) * ncols / sub - first) * per_mcu;
      // (a row whose start is not known flags the sample, also when its pieces' are)
      bad = (reinterpret_cast<const RowState*>(a.row_states) + (int64_t)b * a.max_rows)[row].pos < 0;
    }
    const uint32_t limit_y = long_from(im.ac[0]), limit_c = long_from(im.ac[1]);
    const int table = slot * kCoefTable;
    // byte offsets of the row's first block, and of the current one less one coefficient
    const uint32_t base = origin +
                          (uint32_t)(row * ncols + first) * (uint32_t)(per_mcu * kBlockBytes);
    uint32_t out = base - 2;
    // (a row's restart boundary, if any, lies behind its last MCU: a state that says otherwise is
    // not one of this file's)
    bad = bad || st.pos < im.scan_off || st.pos > im.size || st.nbits < 0 || st.nbits > 64 ||
          (im.restart != 0 && st.rst_left != 0 && (int)st.rst_left <= mx1);
    bool go = !bad;
    SymbolReader r;
    r.skew = (int)(im.origin & 7);
    r.chunks = a.files + (im.origin - r.skew);
    r.chunks_bytes = a.files_bytes - (im.origin - r.skew);
    r.ring = &s.ring[0][lane];
    r.n = im.size;
    int pred0 = st.pred[0], pred1 = st.pred[1], pred2 = st.pred[2];
    int k = 64, phase = -1, done = -1;  // (as behind a block before the first)
    uint32_t e = 0;                     // the last AC symbol's entry
    uint32_t limit = 0;
    int ac = table;
    bool is_chroma = false;
    if (go) sym_open(r, st);
    int round = 0;  // (the same in all lanes that are still at work)
#pragma unroll 1
    while (go) {
      if (__builtin_expect(k >= 64 && e == kMiss, 0)) {
        int index;
        const HuffAc& h = im.ac[is_chroma];
        const uint32_t ahead = sym_ahead(r), top = sym_top(r);
        const int len = find_code<0>(h.range, top >> 16, index);
        k -= 63;
        if (len < 16) {
          e = coef_entry(len + 1, h.symbols[index & 255]);
          k += (int)((e >> 4) & 63u);
          store_symbol(coefs, out, k, top, e);
          sym_skip(r, (int)(e >> 10), ahead);
        } else {  // no such code
          bad = true;
          break;
        }
      }
      // ---- lanes whose block has ended: the next one's DC coefficient ----
      int dc = 0;
      const bool opens = k >= 64;
      if (opens) {
        bad = bad || ((e & 15u) != 0u && k > 64);  // a run past the end of the block
        ++done;
        out += done > skip ? (uint32_t)kBlockBytes : 0u;
        if (done == skip && skip) {
          // the blocks to the left of the crop have left their values where the first block goes
          typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
          for (int i = 0; i < kBlockBytes / 16; ++i)
            reinterpret_cast<u32x4*>(coefs + base)[i] = u32x4{0u, 0u, 0u, 0u};
        }
        phase = phase == last_phase ? 0 : phase + 1;
        is_chroma = phase >= nblk;
        limit = is_chroma ? limit_c : limit_y;
        ac = table + (is_chroma ? kCoefAc : 0);
        go = done < total && !bad;
        const uint32_t ahead = sym_ahead(r), top = sym_top(r);
        uint32_t d = s.table[table + 2 * kCoefAc + (is_chroma ? 1 << kDcBits : 0) +
                             (int)(top >> (32 - kDcBits))];
        if (__builtin_expect(d == kMiss, 0)) {
          int index;
          const HuffDc& h = im.dc[is_chroma];
          const int len = find_code<0>(h.range, top >> 16, index);
          const int sym = len < 16 ? h.symbols[index & 15] : 16;
          if (sym <= 11) d = coef_entry(len + 1, sym);
          else if (go) bad = true;
        }
        const int size = (int)(d & 15u), off = (int)(d >> 10);
        const int diff = symbol_value(top, off, size);
        sym_skip(r, off, ahead);
        pred0 += is_chroma ? 0 : diff;
        pred1 += phase == nblk ? diff : 0;
        pred2 += phase == last_phase ? diff : 0;
        // (clamped to 16 bits: beyond them the de-quantised value is clamped to the same anyway)
        dc = min(max(is_chroma ? (phase == nblk ? pred1 : pred2) : pred0, -32767), 32767);
        k = 1;
        go = go && !bad;
      }
      if (!go) break;
      if (round == 0) sym_feed(r);
      round = round + 1 == kRounds ? 0 : round + 1;
      if (opens) *reinterpret_cast<int16_t*>(coefs + (out + 2u)) = (int16_t)dc;
      // ---- AC symbols; a lane whose block ends waits for the next round ----
      // No branch: a waiting lane keeps its last symbol and stores that value again.  A symbol's value is
      // made and stored while the next one's entry comes out of LDS.
      uint32_t bits = 0;  // those that `e` was found in
#pragma unroll
      for (int i = 0; i < kSteps; ++i) {
        const bool on = k < 64;
        const uint32_t ahead = sym_ahead(r), top = sym_top(r);
        const uint32_t beyond = __builtin_elementwise_sub_sat(top >> 16, limit);
        const uint32_t found =
            s.table[(uint32_t)ac + min(top >> (32 - kFastBits), limit >> (16 - kFastBits)) + beyond];
        if (i > 0) store_symbol(coefs, out, k, bits, e);
        __builtin_amdgcn_sched_barrier(0);
        e = on ? found : e;
        bits = on ? top : bits;
        const uint32_t step = on ? found : kNoStep;
        k += (int)((step >> 4) & 63u);
        sym_skip(r, (int)(step >> 10), ahead);
      }
      store_symbol(coefs, out, k, bits, e);
    }
    if (bad) {
      reinterpret_cast<CropRec*>(a.workspace + kWorkspaceHeader)[b].valid = 0;
      if (a.crop_out) a.crop_out[(int64_t)b * 6 + 5] = 0;
    }
  }
}

size_t jpeg_prepared_bytes() { return sizeof(JpegPrepared); }
size_t jpeg_row_state_bytes() { return sizeof(RowState); }

hipError_t launch_jpeg_header(const JpegArgs& a, hipStream_t stream) {
  dim3 grid((uint32_t)((a.B + kJpegThreads - 1) / kJpegThreads)), block(kJpegThreads);
  hipLaunchKernelGGL(jpeg_header_kernel, grid, block, 0, stream, a);
  return hipGetLastError();
}

// Four pixels of a row of the region: interleaved RGB, 12 bytes at a 4-byte aligned address.
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef u32x3 u32x3_a4 __attribute__((aligned(4)));
__device__ static inline void store_rgb4(uint8_t* dst, uint32_t yy, uint32_t cb, uint32_t cr) {
  uint32_t px[4];
#pragma unroll
  for (int j = 0; j < 4; ++j)
    px[j] = ycc_to_rgbx((int)((yy >> (8 * j)) & 0xFFu), (int)((cb >> (8 * j)) & 0xFFu),
                        (int)((cr >> (8 * j)) & 0xFFu));
  *reinterpret_cast<u32x3_a4*>(dst) =
      u32x3{px[0] | (px[1] << 24), (px[1] >> 8) | (px[2] << 16), (px[2] >> 16) | (px[3] << 8)};
}
// Two chroma samples, each over two pixels (T.81 A.1.1 leaves upsampling open; repetition is this
// library's definition).
__device__ static inline uint32_t repeat2(uint32_t c) {
  return (c & 0xFFu) * 0x0101u | (c >> 8) * 0x01010000u;
}

// Two 16-bit values saturated to bytes 0 .. 255: bytes 0 and 1 of the result.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
__device__ static inline uint32_t saturate2(uint32_t v) {
  uint32_t r;
  asm("v_sat_pk_u8_i16 %0, %1" : "=v"(r) : "v"(v));
  return r;
}
__device__ static inline uint32_t add2(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_bit_cast(u16x2, a) + __builtin_bit_cast(u16x2, b));
}
// What a chroma sample adds to its pixels (ycc_to_rgbx), each twice as 16-bit values.
struct ChromaTerms {
  uint32_t r, g, b;
};
__device__ static inline ChromaTerms chroma_terms(int cb, int cr) {
  const int b = cb - 128, r = cr - 128;
  const int rt = (91881 * r + 32768) >> 16, bt = (116130 * b + 32768) >> 16;
  const int gt = -((22554 * b + 46802 * r + 32768) >> 16);
  return {(uint32_t)(rt & 0xFFFF) * 0x10001u, (uint32_t)(gt & 0xFFFF) * 0x10001u,
          (uint32_t)(bt & 0xFFFF) * 0x10001u};
}
// Four pixels of which each two share a chroma sample, two values per instruction.
__device__ static inline void store_rgb4_pairs(uint8_t* dst, uint32_t yy, const ChromaTerms& c0,
                                               const ChromaTerms& c1) {
  const uint32_t y01 = __builtin_amdgcn_perm(0u, yy, 0x0c010c00u);
  const uint32_t y23 = __builtin_amdgcn_perm(0u, yy, 0x0c030c02u);
  // bytes R0 R1 G0 G1 / B0 B1, and the same for pixels 2, 3
  const uint32_t rg01 = saturate2(add2(y01, c0.r)) | saturate2(add2(y01, c0.g)) << 16;
  const uint32_t rg23 = saturate2(add2(y23, c1.r)) | saturate2(add2(y23, c1.g)) << 16;
  const uint32_t b01 = saturate2(add2(y01, c0.b)), b23 = saturate2(add2(y23, c1.b));
  const uint32_t g1b1 = __builtin_amdgcn_perm(b01, rg01, 0x0c0c0503u);
  const uint32_t r2g2 = __builtin_amdgcn_perm(0u, rg23, 0x02000c0cu);
  *reinterpret_cast<u32x3_a4*>(dst) = u32x3{__builtin_amdgcn_perm(b01, rg01, 0x01040200u), g1b1 | r2g2,
                                            __builtin_amdgcn_perm(b23, rg23, 0x05030104u)};
}

// Coefficients or planes -> interleaved RGB, the region's rows as the resampling kernel reads them.
// A workgroup takes 192 blocks of an image at a time, one per lane: 32 MCUs with 4:2:0 sampling (two
// wavefronts of luma, one of chroma) or 64 with 4:4:4 (a wavefront per component), so that a
// wavefront has one quantiser table, in scalar registers.  The transform is unrolled over registers
// (zig-zag order is then free); its even and odd halves are summed apart and give two outputs each,
// which halves the products (sums of the same integers: nothing changes in the result).  The samples
// meet in LDS, from where four pixels per lane and step are converted and stored along the rows.
// Bound by vector instructions, half of them the transform; the bytes are taken two per instruction where
// they fit 16 bits (4096 files of 256 pixels: 0.25 ms; 0.34 with an image's parts next to each other in
// the grid, where the parts with nothing to do left some compute units more work than others, and
// 0.45 with a 32-bit clamp and shift per value besides).
// Images that jpeg_decode_kernel has decoded have planes instead of coefficients; images with spilled
// rows are one workgroup's work.
constexpr int kIdctThreads = 3 * kWave;
constexpr int kIdctStride = 72;   // bytes per block of samples: 64 and a pad against bank conflicts
constexpr int kCoefStride = 144;  // the same for its coefficients
constexpr int kColourBand = 32;

constexpr int kZigzagOf[64] = {  // kZigzag for compile-time indices
    0,  1,  8,  16, 9,  2,  3,  10, 17, 24, 32, 25, 18, 11, 4,  5,  12, 19, 26, 33, 40, 48,
    41, 34, 27, 20, 13, 6,  7,  14, 21, 28, 35, 42, 49, 56, 57, 50, 43, 36, 29, 22, 15, 23,
    30, 37, 44, 51, 58, 59, 52, 45, 38, 31, 39, 46, 53, 60, 61, 54, 47, 55, 62, 63};

// Eight outputs of one line of the transform; c = inputs 0|2, 4|6, 1|3, 5|7 as pairs of 16 bits.
__device__ static inline void idct_line(const s16x2 c[4], int rounding, int out[8]) {
  constexpr s16x2 kEven[4][2] = {{{5793, 7568}, {5793, 3135}},
                                 {{5793, 3135}, {-5793, -7568}},
                                 {{5793, -3135}, {-5793, 7568}},
                                 {{5793, -7568}, {5793, -3135}}};
  constexpr s16x2 kOdd[4][2] = {{{8035, 6811}, {4551, 1598}},
                                {{6811, -1598}, {-8035, -4551}},
                                {{4551, -8035}, {1598, 6811}},
                                {{1598, -4551}, {6811, -8035}}};
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    int e = __builtin_amdgcn_sdot2(c[0], kEven[x][0], rounding, false);
    e = __builtin_amdgcn_sdot2(c[1], kEven[x][1], e, false);
    int o = __builtin_amdgcn_sdot2(c[2], kOdd[x][0], 0, false);
    o = __builtin_amdgcn_sdot2(c[3], kOdd[x][1], o, false);
    out[x] = e + o;
    out[7 - x] = e - o;
  }
}

// A block of coefficients -> its samples, eight rows of eight bytes at `samples`.  qz: quantiser step
// of zig-zag position `lane` (the wavefront's blocks share the table).
typedef uint32_t u32x4_c __attribute__((ext_vector_type(4)));
__device__ static inline void idct_block(const u32x4_c raw[8], int qz, uint8_t* samples) {
  int c[64];
#pragma unroll
  for (int k = 0; k < 64; ++k) {
    const int v = (int16_t)(raw[k >> 3][(k >> 1) & 3] >> (16 * (k & 1)));
    c[kZigzagOf[k]] = min(max(__mul24(v, __builtin_amdgcn_readlane(qz, k)), -32767), 32767);
  }
  int t[64];
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    s16x2 in[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int y = (i & 1) * 4 + (i >> 1);  // rows 0|2, 4|6, 1|3, 5|7
      in[i] = s16x2{(short)c[y * 8 + u], (short)c[(y + 2) * 8 + u]};
    }
    int line[8];
    idct_line(in, 1 << 10, line);
#pragma unroll
    for (int y = 0; y < 8; ++y) t[y * 8 + u] = min(max(line[y] >> 11, -32767), 32767);
  }
#pragma unroll
  for (int y = 0; y < 8; ++y) {
    s16x2 in[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int u = (i & 1) * 4 + (i >> 1);
      in[i] = s16x2{(short)t[y * 8 + u], (short)t[y * 8 + u + 2]};
    }
    // (v + 2^16 >> 17) + 128, clamped: the high halves two at a time, one more bit, saturated (the sums
    // stay below 2^31 with the 128 among them)
    int v[8];
    idct_line(in, (1 << 16) + (128 << 17), v);
    uint32_t two[4];
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const uint32_t high =
          __builtin_amdgcn_perm((uint32_t)v[2 * x + 1], (uint32_t)v[2 * x], 0x07060302u);
      two[x] = saturate2(__builtin_bit_cast(uint32_t, __builtin_bit_cast(s16x2, high) >> (short)1));
    }
    *reinterpret_cast<u32x2*>(samples + 8 * y) = u32x2{two[0] | two[1] << 16, two[2] | two[3] << 16};
  }
}

// The planes of one band of rows -> RGB.
__device__ static void colour_band(const JpegArgs& a, const JpegRec& rec, int b, int first) {
  const int region_w = a.region_widths[b], hs = rec.hs;
  const int chroma_w = region_w / hs;
  const int64_t off = a.region_offsets[b];
  const uint8_t* plane_y = a.planes + off;
  const uint8_t* plane_cb = plane_y + (int64_t)rec.region_h * region_w;
  const uint8_t* plane_cr = plane_cb + (int64_t)(rec.region_h / hs) * chroma_w;
  uint8_t* region = a.regions + off;
  const int ng = region_w >> 2;
  const int rows = min(kColourBand, rec.region_h - first);
  for (int i = (int)threadIdx.x; i < rows * ng; i += kIdctThreads) {
    const int y = first + i / ng, g = i % ng;
    const uint32_t yy = *reinterpret_cast<const uint32_t*>(plane_y + (int64_t)y * region_w + 4 * g);
    uint32_t cb, cr;  // one byte per pixel
    if (hs == 2) {
      const int64_t o = (int64_t)(y >> 1) * chroma_w + 2 * g;
      cb = repeat2(*reinterpret_cast<const uint16_t*>(plane_cb + o));
      cr = repeat2(*reinterpret_cast<const uint16_t*>(plane_cr + o));
    } else {
      const int64_t o = (int64_t)y * chroma_w + 4 * g;
      cb = *reinterpret_cast<const uint32_t*>(plane_cb + o);
      cr = *reinterpret_cast<const uint32_t*>(plane_cr + o);
    }
    // rows of the region start on 4-byte boundaries (their width is a multiple of 8 pixels)
    store_rgb4(region + ((int64_t)y * region_w + 4 * g) * 3, yy, cb, cr);
  }
}

__global__ __launch_bounds__(kIdctThreads) void jpeg_idct_kernel(JpegArgs a, int parts) {
  // the step's coefficients, then (all lanes have theirs in registers) its samples
  __shared__ __attribute__((aligned(16))) uint8_t samples[kIdctThreads * kCoefStride];
  __shared__ uint32_t place[kWave];  // of an MCU's first pixel in the region
  // all images' first parts first: the longest work, where an image is one workgroup's
  const int part = (int)(blockIdx.x / (uint32_t)a.B);
  const int b = (int)(blockIdx.x - (uint32_t)part * (uint32_t)a.B);
  const JpegImage& im = reinterpret_cast<const JpegPrepared*>(a.prepared)[b].im;
  if (!im.live) return;
  if (im.live == kLivePlanes) {
    const JpegRec rec = a.recs[b];
    for (int first = part * kColourBand; first < rec.region_h; first += parts * kColourBand)
      colour_band(a, rec, b, first);
    return;
  }
  const int lane = threadIdx.x % kWave;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave);
  const int hs = im.hs, per_mcu = hs * hs + 2, mcu = 8 * hs;
  const int ncols = im.mx1 - im.mx0 + 1, nmcu = ncols * im.nrows;
  const int region_w = im.region_w;
  const uint8_t* coef = a.planes + im.region_off;
  uint8_t* region = a.regions + im.region_off;
  const bool spill = im.live == kLiveSpill;
  if (spill && part != 0) return;  // (its rows in order: spilled_rows)
  const int64_t slot_bytes = (int64_t)a.slot_side * a.slot_side * 3;
  const int64_t row_bytes = (int64_t)ncols * per_mcu * kBlockBytes;
  const int64_t spilled_bytes = spill ? spilled_rows(slot_bytes, row_bytes, im.nrows) * row_bytes : 0;
  const int qz = im.qz[hs == 2 ? wave == 2 : wave != 0][lane] & 255;
  const int group = kWave / hs;  // MCUs per step
  // this lane's block: MCU inside the group, block of the MCU
  const int m = hs == 2 ? (wave == 2 ? lane >> 1 : 16 * wave + (lane >> 2)) : lane;
  const int blk = hs == 2 ? (wave == 2 ? 4 + (lane & 1) : lane & 3) : wave;
  // MCUs of a step: any, or whole rows, or parts of one row that is longer
  const int row_steps = (ncols + group - 1) / group, step_mcus = spill ? max(group / ncols, 1) * ncols : group;
  const int nsteps = spill && row_steps > 1 ? im.nrows * row_steps : (nmcu + step_mcus - 1) / step_mcus;
  for (int step = spill ? 0 : part; step < nsteps; step += spill ? 1 : parts) {
    int m0 = step * step_mcus, end = min(nmcu, m0 + step_mcus);
    if (spill && row_steps > 1) {
      const int row = step / row_steps;
      m0 = row * ncols + (step - row * row_steps) * group;
      end = (row + 1) * ncols;
    }
    if ((int)threadIdx.x < group) {
      const int i = min(m0 + (int)threadIdx.x, end - 1);
      const int my = i / ncols, mx = i - my * ncols;
      place[threadIdx.x] = ((uint32_t)(my * mcu) * (uint32_t)region_w + (uint32_t)(mx * mcu)) * 3u;
    }
    // the step's blocks lie one after the other in memory: 16 bytes per lane and load
    const int64_t first = (int64_t)m0 * per_mcu * kBlockBytes;
    const int pieces = min(group, end - m0) * per_mcu * (kBlockBytes / 16);
    u32x4_c raw[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t at = first + 16 * min((int)threadIdx.x + i * kIdctThreads, pieces - 1);
      const uint8_t* src = (at < spilled_bytes ? region + slot_bytes : coef) - spilled_bytes;
      raw[i] = *reinterpret_cast<const u32x4_c*>(src + at);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int at = (int)threadIdx.x + i * kIdctThreads;
      *reinterpret_cast<u32x4_c*>(samples + (at >> 3) * kCoefStride + (at & 7) * 16) = raw[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i)
      raw[i] = *reinterpret_cast<const u32x4_c*>(samples + (m * per_mcu + blk) * kCoefStride + 16 * i);
    __syncthreads();
    idct_block(raw, qz, samples + threadIdx.x * kIdctStride);
    __syncthreads();
    // 128 pieces of four pixels per row of the group's MCUs; with 4:2:0 a lane takes two rows, which
    // share their chroma samples
    for (int i = (int)threadIdx.x; i < 128 * 8; i += kIdctThreads) {
      const int y = (i >> 7) * hs, r = i & 127;
      const int pm = r >> hs, piece = r & (2 * hs - 1);
      if (m0 + pm >= end) continue;
      uint8_t* dst = region + (place[pm] + (uint32_t)((y * region_w + 4 * piece) * 3));
      if (hs == 2) {
        const int luma = 4 * pm + (y >> 3) * 2 + (piece >> 1), chroma = 128 + 2 * pm;
        const uint32_t* yy = reinterpret_cast<const uint32_t*>(samples + luma * kIdctStride +
                                                               (y & 7) * 8 + 4 * (piece & 1));
        const uint8_t* c = samples + chroma * kIdctStride + (y >> 1) * 8 + 2 * piece;
        const uint32_t cb = *reinterpret_cast<const uint16_t*>(c);
        const uint32_t cr = *reinterpret_cast<const uint16_t*>(c + kIdctStride);
        const ChromaTerms c0 = chroma_terms((int)(cb & 0xFFu), (int)(cr & 0xFFu));
        const ChromaTerms c1 = chroma_terms((int)(cb >> 8), (int)(cr >> 8));
        store_rgb4_pairs(dst, yy[0], c0, c1);
        store_rgb4_pairs(dst + 3 * region_w, yy[2], c0, c1);
      } else {
        const uint8_t* s = samples + pm * kIdctStride + y * 8 + 4 * piece;
        store_rgb4(dst, *reinterpret_cast<const uint32_t*>(s),
                   *reinterpret_cast<const uint32_t*>(s + kWave * kIdctStride),
                   *reinterpret_cast<const uint32_t*>(s + 2 * kWave * kIdctStride));
      }
    }
    __syncthreads();
  }
}

// Wavefronts per file.  Long files fill more than one with parts of kPartBits bits, which shortens the
// walks until the SIMDs have other files to switch to; on files of 256 pixels (2200 to 3200 bits in each of
// 64 parts) shorter parts only take more rounds.  The line is drawn by what the call knows of its files, the
// largest side that they may have.  Whole calls with 1 / 2 / 4 wavefronts in us, files without markers whose
// sides reach the limit: 300 pixels, 16 files 768 / 728 / 725, 512 1068 / 1096 / 1089; 320 pixels, 16 files 862 / 771 / 779, 512
// 1121 / 1068 / 1056, 1024 1299 / 1243 / 1741; 384 pixels, 128 files 1221 / 1039 / 1063, 512 1493 / 1328 / 1312, 1024 1743 / 1522 /
// 2087; 500 pixels, 16 files 1622 / 1214 / 1141, 128 1761 / 1420 / 1311, 512 2045 / 1766 / 1604, 1024 2337 / 2113 / 2532.  Short
// files under a large limit leave wavefronts without a part: 256 pixels and a limit of 500, 16 files 670 / 697 /
// 688, 512 921 / 943 / 944, 1024 1141 / 1144 / 1583; a limit of 320, 16 files 671 / 695 / 707; 160 and 500, 512 files 796 / 789 /
// 778.
static hipError_t launch_sync(const JpegArgs& a, hipStream_t stream) {
  const int waves = a.slot_side < 320 || a.B > 1024 ? 1 : (a.B > 512 ? 2 : 4);
  if (waves == 4)
    hipLaunchKernelGGL(jpeg_sync_kernel<4>, dim3((uint32_t)a.B), dim3(4 * kJpegThreads), 0, stream, a);
  else if (waves == 2)
    hipLaunchKernelGGL(jpeg_sync_kernel<2>, dim3((uint32_t)a.B), dim3(2 * kJpegThreads), 0, stream, a);
  else
    hipLaunchKernelGGL(jpeg_sync_kernel<1>, dim3((uint32_t)a.B), dim3(kJpegThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_jpeg_index(const JpegArgs& a, hipStream_t stream) {
  dim3 block(kJpegThreads);
  hipLaunchKernelGGL(jpeg_tables_kernel, dim3((uint32_t)a.B), block, 0, stream, a);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (!a.row_index) {
    err = launch_sync(a, stream);
    if (err != hipSuccess) return err;
  }
  hipLaunchKernelGGL(jpeg_scan_kernel, dim3((uint32_t)((a.B + kScanImages - 1) / kScanImages)),
                     block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_jpeg_decode(const JpegArgs& a, hipStream_t stream) {
  dim3 block(kJpegThreads);
  hipLaunchKernelGGL(jpeg_tables_kernel, dim3((uint32_t)a.B), block, 0, stream, a);
  hipError_t err = hipGetLastError();
  if (err != hipSuccess) return err;
  if (!a.row_index) {
    err = launch_sync(a, stream);
    if (err != hipSuccess) return err;
  }
  // files whose rows are not independent (its wavefronts leave at once where there are none)
  hipLaunchKernelGGL(jpeg_scan_kernel, dim3((uint32_t)((a.B + kScanImages - 1) / kScanImages)),
                     block, 0, stream, a);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  // as many images per wavefront as fill its lanes with rows of MCUs: an image of the largest
  // side allowed has slot_side / 16 rows of them when its luma is sampled 2x2
  const int rows = a.slot_side / 16;
  const uint32_t B = (uint32_t)a.B;
  const int most = rows <= 16 ? 4 : (rows <= 32 ? 2 : 1);
  // fewer when the batch leaves SIMDs without a wavefront (4 per compute unit): a wavefront with
  // fewer lanes has fewer of them on a rare path at a time
  const int group = B <= 1024 ? 1 : (B <= 2048 ? (most < 2 ? most : 2) : most);
  if (group == 4)
    hipLaunchKernelGGL(jpeg_entropy_kernel<4>, dim3(2 * ((B + 3) / 4)), block, 0, stream, a);
  else if (group == 2)
    hipLaunchKernelGGL(jpeg_entropy_kernel<2>, dim3(2 * ((B + 1) / 2)), block, 0, stream, a);
  else
    hipLaunchKernelGGL(jpeg_entropy_kernel<1>, dim3(2 * B), block, 0, stream, a);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  // files with restart boundaries inside a row of MCUs, and crops whose coefficients do not fit
  if (most == 4)
    hipLaunchKernelGGL(jpeg_decode_kernel<4>, dim3((B + 3) / 4), block, 0, stream, a);
  else if (most == 2)
    hipLaunchKernelGGL(jpeg_decode_kernel<2>, dim3((B + 1) / 2), block, 0, stream, a);
  else
    hipLaunchKernelGGL(jpeg_decode_kernel<1>, dim3(B), block, 0, stream, a);
  err = hipGetLastError();
  if (err != hipSuccess) return err;
  // workgroups per image: a step each for the largest image with 4:2:0 sampling
  const int parts = (rows * rows + 31) / 32;
  hipLaunchKernelGGL(jpeg_idct_kernel, dim3(B * (uint32_t)parts), dim3(kIdctThreads), 0, stream, a,
                     parts);
  return hipGetLastError();
}

}  // namespace mae
