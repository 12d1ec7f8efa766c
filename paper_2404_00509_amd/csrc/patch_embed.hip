// Patch embedding of the visible tokens (Sec. 2: only the visible patches reach the encoder;
// Sec. 5: the ViT's linear patch embedding): tokens = visible x weight^T + bias + pos[ids_keep].
//
// The one dense contraction next to the input pipeline, so it runs on the matrix cores:
// v_mfma_f32_32x32x16_bf16, bf16 operands, fp32 accumulation.  Both operands are K-contiguous
// (visible [M, D], weight [E, D]), which is the layout the instruction wants: a lane supplies 8
// consecutive k of one row.
//
// A workgroup makes a tile of 256 x 256 results (eight wavefronts, 2 x 4, 128 x 64 each), or of 128 x 128
// or 64 x 64 where larger ones would leave compute units idle or take longer (embed_tile).  D is
// walked in slices of 64 values, so that every row contributes one full 128-byte line per slice:
// half-line requests cost the vector memory pipeline as much as whole lines.  The two operand
// slices (of the large tile 512 rows of 128 bytes = 64 KiB) go from global memory straight into LDS
// (global_load_lds_dwordx4, no trip through registers) into one of the stage buffers while
// another one is multiplied.  A staged row is eight 16-byte chunks whose position is XORed with
// bits 1..3 of the row number: 16 consecutive rows of one chunk column then fall into 16
// different 16-byte bank groups, which is what a ds_read_b128 of the 64-bank LDS needs to run at
// full rate (fragment reads: 32 rows of one chunk column per half wave).  Because a direct load
// always writes lane l to slot l of the wave's 1 KiB window, the swizzle is applied on the global
// side: each lane fetches the chunk that belongs in its slot.  In the last, partial slice of a D
// that is no multiple of 64 the lanes behind the row's end fetch zeros, a last half chunk (D no
// multiple of 8) is put in its place from registers, and the sub-steps without values are left out.
//
// The fragment reads are issued through inline assembly: the compiler does not see them as LDS
// accesses, so it does not make each of them wait for every direct load in flight (which would
// undo the pipeline); the code waits on lgkmcnt itself and reads one sub-step ahead.
//
// What bounds the large tile.  200704 rows, 768 -> 768, bf16, by a clock read at the turns of every
// workgroup: a tile takes 31.3 us at the 1.91 GHz that the card holds in this kernel, 3.8 until its
// first slice is there, 20.4 for eleven slices (3540 cycles each), 1.5 for the last one, 5.7 for the epilogue; a
// compute unit makes 9.2 of them one after the other, the tenth round a fifth full.  The matrix
// instructions are 12.8 us of it (2048 cycles of a slice).  In a slice no unit is busy all the time: beside them the
// LDS moves 256 KiB (2048 cycles: 192 KiB of fragments, 64 KiB coming in), and 64 loads of 1 KiB take the
// vector memory pipeline about 35 cycles each (2240); over the kernel the counters show the data return
// of that pipeline at work 75 % of the time and the wavefronts 34 % waiting for data or barriers, 41 % for an
// instruction to be taken.  Hence the large tile, which needs the fewest operand bytes per result, and loads that
// are spread over three of a slice's four sub-steps.  Calls with inputs from memory: 310 us in bf16, 343 in fp32 (324
// and 370 with the turn between slices where nothing is multiplied, a burst of loads behind it and lines of later
// slices requested into L2; with such requests beside the present loads 1 and 2 % slower than without); 32768 rows,
// 588 -> 1024: 60 and 62 us (65 and 75).
//
// Epilogue: each wavefront turns its accumulators into rows through a private strip of LDS, 32
// rows at a time, so that the stores to `tokens` and the loads of the positional rows are
// contiguous along a row (16-byte stores).  The patch indices are fetched at kernel start
// and exchanged between lanes, and the positional rows of the next 32 rows are requested
// before the current ones are transposed.  Bias and pos[ids_keep] are added in fp32 before the
// single rounding to the output type.  Consecutive workgroups of an XCD walk the E direction of
// one row block first: they share the rows of `visible` through that XCD's L2.
#include "mae_device.hpp"
#include "mae_kernels.hpp"

namespace mae {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef u32x2 u32x2_a4 __attribute__((aligned(4)));
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));

constexpr int kBK = 64;            // values of D per pipeline stage: one 128-byte line per row
constexpr int kRowChunks = 8;      // 16-byte chunks per staged row
constexpr int kEpiPad = 8;         // floats of padding per staged output row

// What lanes fetch whose chunk lies behind the end of a row (last slice of a D that is no multiple of
// a slice).
__device__ const u32x4 kZeroChunk = {0u, 0u, 0u, 0u};

// 16-byte LDS read the compiler does not see as an LDS access (see the file comment).  The
// caller waits on lgkmcnt itself before it touches the result.
template <int kOff>
__device__ static inline u32x4 lds_read16(uint32_t addr) {
  u32x4 v;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(kOff) : "memory");
  return v;
}

// s_waitcnt immediate: vmcnt(n) and lgkmcnt(0), expcnt not waited for
constexpr int waitcnt_vm(int n) { return (n & 0xF) | ((n >> 4) << 14) | 0x0070; }

template <int TM, int TN, int WGM, int WGN, int STAGES, bool kOutBf16>
__global__ __launch_bounds__(64 * WGM * WGN) void patch_embed_kernel(EmbedArgs a) {
  constexpr int kThreads = 64 * WGM * WGN;
  constexpr int kWaves = WGM * WGN;
  constexpr int BM = 32 * TM * WGM, BN = 32 * TN * WGN;
  constexpr int kSlots = (BM + BN) * kRowChunks;  // 16-byte slots per stage
  constexpr int NL = kSlots / kThreads;           // direct loads per lane and stage
  static_assert(kSlots % kThreads == 0, "stage must divide into wave-wide loads");
  static_assert(NL <= 8 && NL * (STAGES - 1) <= 63, "half rows of a wave per lane; vmcnt range");
  constexpr int kStageBytes = kSlots * 16;
  constexpr int kEpiStride = 32 * TN + kEpiPad;           // floats
  constexpr int kEpiWave = 32 * kEpiStride;               // floats per wave
  constexpr int kMainBytes = STAGES * kStageBytes;
  constexpr int kEpiBytes = kWaves * kEpiWave * 4;
  constexpr int kLdsBytes = kMainBytes > kEpiBytes ? kMainBytes : kEpiBytes;
  __shared__ __attribute__((aligned(16))) u32x4 lds[kLdsBytes / 16];

  const int tid = threadIdx.x;
  const int lane = tid % kWave;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int wm = wave / WGN, wn = wave % WGN;
  const uint32_t tiles_n = (uint32_t)((a.E + BN - 1) / BN);
  const uint32_t tile = xcd_remap(blockIdx.x, gridDim.x);
  const uint32_t tile_m = tile / tiles_n, tile_n = tile - tile_m * tiles_n;
  const int64_t m0 = (int64_t)tile_m * BM;
  const int n0 = (int)tile_n * BN;
  const int rows_m = (int)min((int64_t)BM, a.M - m0), rows_n = min(BN, a.E - n0);
  const int D = a.D;
  const uint16_t* A = static_cast<const uint16_t*>(a.visible) + m0 * D;
  const uint16_t* W = static_cast<const uint16_t*>(a.weight) + (int64_t)n0 * D;

  // patch index of row (lane % 32) of each of the wave's 32-row bands, for the epilogue
  int idr[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int r = min(wm * 32 * TM + i * 32 + (lane & 31), rows_m - 1);
    idr[i] = a.pos ? a.ids_keep[m0 + r] : 0;  // clamped where it is used: no wait for it here
  }

  // what this lane brings in per stage: slot s = (wave * NL + q) * 64 + lane holds chunk
  // (s % 8) ^ (row / 2 % 8) of row s / 8 (rows of `visible` first, then rows of `weight`; eight rows
  // per load, so a load's operand is the same for all lanes).  Rows past the end: any valid row.
  uint32_t off[NL];  // bytes from the operand's first row of the tile
#pragma unroll
  for (int q = 0; q < NL; ++q) {
    const int s = (wave * NL + q) * kWave + lane;
    const int row = s / kRowChunks;
    const int chunk = (s % kRowChunks) ^ ((row >> 1) % kRowChunks);
    const int r = row < BM ? min(row, rows_m - 1) : min(row - BM, rows_n - 1);
    off[q] = (uint32_t)(r * D + 8 * chunk) * 2u;
  }
  // a D that is no multiple of 8 ends in half a chunk: the last four values of row (wave * 8 NL + lane)
  // of the stage, which this wave brings in
  const int tail = D % kBK;
  u32x2 half = {0u, 0u};
  const int half_row = wave * 8 * NL + lane;
  if ((tail & 4) != 0 && lane < 8 * NL) {
    const uint16_t* row = half_row < BM ? A + (int64_t)min(half_row, rows_m - 1) * D
                                        : W + (int64_t)min(half_row - BM, rows_n - 1) * D;
    half = *reinterpret_cast<const u32x2_a4*>(row + D - 4);
  }

  auto issue = [&](int it, int stage, int q0, int q1) {
    u32x4* dst = lds + stage * kSlots + wave * NL * kWave;
    // (opaque: base plus 32-bit offset is the form that costs no vector instructions)
    const char* a_base = reinterpret_cast<const char*>(A) + it * (kBK * 2);
    const char* w_base = reinterpret_cast<const char*>(W) + it * (kBK * 2);
    asm("" : "+s"(a_base), "+s"(w_base));
    if ((it + 1) * kBK <= D) {
#pragma unroll
      for (int q = q0; q < q1; ++q) {
        const char* base = (wave * NL + q) * (kWave / kRowChunks) < BM ? a_base : w_base;
        __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(base + off[q]),
                                         (void __attribute__((address_space(3)))*)(dst + q * kWave),
                                         16, 0, 0);
      }
    } else {
      // (a load for every lane, whatever it holds: the waits count them)
#pragma unroll
      for (int q = q0; q < q1; ++q) {
        const int first_row = (wave * NL + q) * (kWave / kRowChunks);
        const int row = first_row + lane / kRowChunks;
        const int chunk = (lane % kRowChunks) ^ ((row >> 1) % kRowChunks);
        const char* src = (first_row < BM ? a_base : w_base) + off[q];
        if (8 * chunk + 8 > tail) src = reinterpret_cast<const char*>(&kZeroChunk);
        __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)src,
                                         (void __attribute__((address_space(3)))*)(dst + q * kWave),
                                         16, 0, 0);
      }
    }
  };
  // the half chunks of a partial slice whose loads have landed
  auto patch_halves = [&](int it, int stage) {
    if ((it + 1) * kBK > D && (tail & 4) != 0 && lane < 8 * NL) {
      const int chunk = (tail / 8) ^ ((half_row >> 1) % kRowChunks);
      reinterpret_cast<u32x2*>(lds + stage * kSlots + half_row * kRowChunks + chunk)[0] = half;
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
  };

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

  // fragment addresses inside a stage (bytes): row (lane % 32) of the wave's first 32-row block,
  // chunk (2 ks + lane / 32) ^ (row / 2 % 8); the row blocks and ks = 0..3 differ by constants
  const uint32_t lds_base =
      (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) u32x4*)lds;
  const uint32_t c0 = (uint32_t)((lane >> 5) ^ ((lane >> 1) & 7)) * 16u;
  const uint32_t a_off = lds_base + (uint32_t)(wm * 32 * TM + (lane & 31)) * 128u + c0;
  const uint32_t b_off = lds_base + (uint32_t)(BM + wn * 32 * TN + (lane & 31)) * 128u + c0;

  const int nk = (D + kBK - 1) / kBK;

  u32x4 fa[2][TM], fb[2][TN];
  auto read_frags = [&](int stage, int ks, int set) {
    const uint32_t va = (a_off ^ (32u * ks)) + (uint32_t)stage * kStageBytes;
    const uint32_t vb = (b_off ^ (32u * ks)) + (uint32_t)stage * kStageBytes;
    if constexpr (TM >= 1) fa[set][0] = lds_read16<0>(va);
    if constexpr (TM >= 2) fa[set][1] = lds_read16<4096>(va);
    if constexpr (TM >= 3) fa[set][2] = lds_read16<8192>(va);
    if constexpr (TM >= 4) fa[set][3] = lds_read16<12288>(va);
    if constexpr (TN >= 1) fb[set][0] = lds_read16<0>(vb);
    if constexpr (TN >= 2) fb[set][1] = lds_read16<4096>(vb);
    __builtin_amdgcn_sched_barrier(0);  // the multiplies of the other set come behind the reads,
  };
  // the fragments of `set` have arrived: nothing that uses them is scheduled above this wait
  auto arrive = [&](int set) {
    __builtin_amdgcn_sched_barrier(0);  // and in front of the wait for them
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(fa[set][i]));
#pragma unroll
    for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(fb[set][j]));
  };
  auto multiply = [&](int set, int from, int to) {
#pragma unroll
    for (int i = from; i < to; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, fa[set][i]), __builtin_bit_cast(bf16x8, fb[set][j]),
            acc[i][j], 0, 0, 0);
  };
  // slice `next` has landed (later ones, at most STAGES - 2, may be on their way), for
  // all wavefronts, and all of them have read what they need of the slice before
  auto turn = [&](int next, int stage) {
    if (next + STAGES - 1 <= nk) {  // the loads of STAGES - 2 slices behind it have been issued
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(NL * (STAGES - 2)));
    } else {
      __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
    }
    patch_halves(next, stage);
    __builtin_amdgcn_s_barrier();
  };

#pragma unroll
  for (int s = 0; s < STAGES; ++s)
    if (s < nk) issue(s, s, 0, NL);
  if (nk >= STAGES) __builtin_amdgcn_s_waitcnt(waitcnt_vm(NL * (STAGES - 1)));
  else __builtin_amdgcn_s_waitcnt(waitcnt_vm(0));
  patch_halves(0, 0);
  __builtin_amdgcn_s_barrier();
  read_frags(0, 0, 0);
  arrive(0);

  // A slice is four sub-steps of 16 values; the fragments of a sub-step are read while the one before
  // it is multiplied, across slices too: the turn to the next slice comes between the third and the
  // fourth multiply, when the stage's last fragments are in registers, so that neither the reads of
  // the next slice's first fragments nor the barrier are waited for with idle matrix cores.  The loads
  // that refill the stage come in three parts, the last two in the slice that follows.
  static_assert(kBK == 64, "four sub-steps");
  constexpr int kLoads1 = 3 * NL / 8, kLoads2 = 6 * NL / 8;
  int cur = 0;
  for (int it = 0; it + 1 < nk; ++it) {
    const bool more = it >= 1 && it + STAGES - 1 < nk;
    const int prv = cur == 0 ? STAGES - 1 : cur - 1;
#pragma unroll
    for (int ks = 0; ks < 3; ++ks) {
      read_frags(cur, ks + 1, (ks + 1) & 1);
      multiply(ks & 1, 0, 1);
      __builtin_amdgcn_sched_barrier(0);
      if (more && ks == 0) issue(it + STAGES - 1, prv, kLoads1, kLoads2);
      if (more && ks == 1) issue(it + STAGES - 1, prv, kLoads2, NL);
      __builtin_amdgcn_sched_barrier(0);
      multiply(ks & 1, 1, TM);
      arrive((ks + 1) & 1);
    }
    const int nxt = cur + 1 == STAGES ? 0 : cur + 1;
    turn(it + 1, nxt);
    read_frags(nxt, 0, 0);
    multiply(1, 0, 1);
    __builtin_amdgcn_sched_barrier(0);
    if (it + STAGES < nk) issue(it + STAGES, cur, 0, kLoads1);
    __builtin_amdgcn_sched_barrier(0);
    multiply(1, 1, TM);
    arrive(0);
    cur = nxt;
  }

  // ---- the last slice, and what the epilogue wants from memory ---------------------------------------
  constexpr int kCols = kOutBf16 ? 8 : 4;  // columns per lane: 16-byte stores
  constexpr int kLanesPerRow = 32 * TN / kCols;
  constexpr int kRowsPerRep = kWave / kLanesPerRow;
  constexpr int kReps = 32 / kRowsPerRep;
  const int col = (lane % kLanesPerRow) * kCols;
  const int n = n0 + wn * 32 * TN + col;
  const bool whole_pieces = a.E % kCols == 0;  // the columns of a lane are all there or none
  const bool vec_ok = whole_pieces && n < a.E;
  f32x4 bias[kCols / 4];
#pragma unroll
  for (int c = 0; c < kCols / 4; ++c) {
    bias[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (!a.bias) continue;
    if (vec_ok) bias[c] = *reinterpret_cast<const f32x4_a4*>(a.bias + n + 4 * c);
    else
      for (int q = 0; q < 4; ++q) bias[c][q] = n + 4 * c + q < a.E ? a.bias[n + 4 * c + q] : 0.f;
  }
  f32x4 p[2][kReps][kCols / 4];
  auto band_id = [&](int i, int rep) {  // (all lanes: a lane at rest hands out nothing)
    const int r = rep * kRowsPerRep + lane / kLanesPerRow;
    return min(max(__builtin_amdgcn_ds_bpermute(4 * r, idr[i]), 0), a.L - 1);
  };
  auto load_pos = [&](int i, int buf) {
#pragma unroll
    for (int rep = 0; rep < kReps; ++rep) {
      const int id = band_id(i, rep);
#pragma unroll
      for (int c = 0; c < kCols / 4; ++c) {
        p[buf][rep][c] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (a.pos && vec_ok)
          p[buf][rep][c] =
              *reinterpret_cast<const f32x4*>(a.pos + (int64_t)id * a.E + (n + 4 * c));
      }
    }
  };
  load_pos(0, 0);
  {
    const int left = tail ? (tail + 15) / 16 : 4;  // sub-steps that hold values
    if (left > 1) read_frags(cur, 1, 1);
    multiply(0, 0, TM);
    if (left > 1) {
      arrive(1);
      if (left > 2) read_frags(cur, 2, 0);
      multiply(1, 0, TM);
    }
    if (left > 2) {
      arrive(0);
      if (left > 3) read_frags(cur, 3, 1);
      multiply(0, 0, TM);
    }
    if (left > 3) {
      arrive(1);
      multiply(1, 0, TM);
    }
  }

  // ---- epilogue: each wavefront turns its own accumulators into rows through a private strip
  // of LDS (32 rows at a time), adds bias and the positional row, stores 16 bytes per lane, whole
  // rows of the wavefront's columns after each other.
  // The positional rows of the next band are requested before the current band is transposed.
  __syncthreads();  // every wavefront is done with the staged operands
  float* epi = reinterpret_cast<float*>(lds) + wave * kEpiWave;
  char* tokens = static_cast<char*>(a.tokens) +
                 (m0 * a.E + n0) * (int64_t)(kOutBf16 ? sizeof(uint16_t) : sizeof(float));
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if (i + 1 < TM) load_pos(i + 1, (i + 1) & 1);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int r = (e >> 2) * 8 + (lane >> 5) * 4 + (e & 3);
        epi[r * kEpiStride + j * 32 + (lane & 31)] = acc[i][j][e];
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int rep = 0; rep < kReps; ++rep) {
      const int r = rep * kRowsPerRep + lane / kLanesPerRow;
      const int row = wm * 32 * TM + i * 32 + r;  // of the tile
      const int id = whole_pieces ? 0 : band_id(i, rep);
      if (row >= rows_m || n >= a.E) continue;
      // (a tile's rows span less than 2^23 bytes)
      const uint32_t at = (uint32_t)(row * a.E + (n - n0));
      f32x4 v[kCols / 4];
#pragma unroll
      for (int c = 0; c < kCols / 4; ++c)
        v[c] = *reinterpret_cast<const f32x4*>(epi + r * kEpiStride + col + 4 * c) + bias[c];
      if (vec_ok) {
#pragma unroll
        for (int c = 0; c < kCols / 4; ++c) v[c] += p[i & 1][rep][c];
        if constexpr (kOutBf16)
          *reinterpret_cast<u32x4*>(tokens + 2u * at) =
              u32x4{pack_bf16x2(v[0].x, v[0].y), pack_bf16x2(v[0].z, v[0].w),
                    pack_bf16x2(v[1].x, v[1].y), pack_bf16x2(v[1].z, v[1].w)};
        else
          *reinterpret_cast<f32x4*>(tokens + 4u * at) = v[0];
      } else {
        const float* pos = a.pos ? a.pos + (int64_t)id * a.E + n : nullptr;
        for (int q = 0; q < kCols && n + q < a.E; ++q) {
          const float x = v[q >> 2][q & 3] + (pos ? pos[q] : 0.f);
          if (kOutBf16) reinterpret_cast<uint16_t*>(tokens)[at + q] = (uint16_t)bf16_rne(x);
          else reinterpret_cast<float*>(tokens)[at + q] = x;
        }
      }
    }
  }
}

template <int TM, int TN, int WGM, int WGN, int STAGES>
static hipError_t launch_cfg(const EmbedArgs& a, hipStream_t stream) {
  constexpr int BM = 32 * TM * WGM, BN = 32 * TN * WGN;
  const int64_t tiles_m = (a.M + BM - 1) / BM;
  const int64_t tiles_n = (a.E + BN - 1) / BN;
  dim3 grid((uint32_t)(tiles_m * tiles_n)), block(64 * WGM * WGN);
  if (a.out_bf16) {
    hipLaunchKernelGGL((patch_embed_kernel<TM, TN, WGM, WGN, STAGES, true>), grid, block, 0,
                       stream, a);
  } else {
    hipLaunchKernelGGL((patch_embed_kernel<TM, TN, WGM, WGN, STAGES, false>), grid, block, 0,
                       stream, a);
  }
  return hipGetLastError();
}

// The side of the tiles.  Tiles of 64 x 64, with three stages, where 128 x 128 (eight wavefronts of 64 x 32)
// would leave every second compute unit without one; 256 x 256 beyond two rounds of them, a compute unit
// holding one at a time; in between what takes less time by the numbers of tiles that the busiest unit gets.
// A tile of 256 takes 11 us and 1.3 us per slice, one of 128 (two of which share a unit) 1.5 us and 0.5, a
// seventh more where rows do not begin on a line, and 2 us once.  That is within 5 % of the better one
// of both wherever it was measured up to two rounds.  Times of 256 / 128 in us, inputs in the caches, bf16:
//   large tiles     147          180          216          255          300          384          468          510
//   768 -> 768   27.3 / 27.4  27.4 / 28.0  28.4 / 33.0  30.8 / 35.1  52.1 / 43.8  52.5 / 51.7  56.4 / 64.1  60.0 / 67.3
//   588 -> 1024  24.1 / 26.1  24.4 / 26.7  25.9 / 31.8  28.2 / 33.5  46.8 / 41.1  47.4 / 50.0  51.1 / 62.5  53.4 / 65.4
//   1200 -> 1024 36.7 / 43.2  38.6 / 45.2  40.2 / 51.5  44.0 / 56.4  75.5 / 71.1  76.3 / 82.9  81.8 / 105   86.1 / 110
//   192 -> 384   14.2 / 9.0   14.3 / 12.0  14.5 / 12.6  15.3 / 13.3  25.6 / 16.0  26.2 / 19.7  27.8 / 22.9  29.5 / 23.3
// Beyond: 516 of 768 -> 768 81.7 / 74.9, 600 82.4 / 80.4, 660 83.8 / 90.5, 1023 119 / 137; in fp32, whose outputs
// leave the caches earlier, 660 92.0 / 97.8, 768 104 / 140.  64 / 128: 784 rows, 768 -> 768 (28 tiles of 128) 7.5 /
// 9.7, 3136 (150) 11.7 / 10.3, 4800 rows, 1200 -> 192 (76) 10 / 13.
int embed_tile(int64_t M, int D, int E) {
  const auto tiles = [&](int side) { return ((M + side - 1) / side) * ((E + side - 1) / side); };
  if (tiles(128) < 128) return 64;
  const int64_t large = (tiles(256) + 255) / 256, small = (tiles(128) + 255) / 256;  // per compute unit
  if (large > 2) return 256;
  const int64_t nk = (D + kBK - 1) / kBK;
  const int64_t small_time = 2000 + small * (150 + 50 * nk) * (D % kBK ? 115 : 100) / 10;  // in units of 1 ns
  return small_time < large * (11000 + 1300 * nk) ? 128 : 256;
}

hipError_t launch_patch_embed(const EmbedArgs& a, hipStream_t stream) {
  const int side = embed_tile(a.M, a.D, a.E);
  if (side == 256) return launch_cfg<4, 2, 2, 4, 2>(a, stream);
  if (side == 128) return launch_cfg<2, 1, 2, 4, 2>(a, stream);
  return launch_cfg<1, 1, 2, 2, 3>(a, stream);
}

}  // namespace mae
