// The logit tile loop: 192 (vocabulary) x 256 (token) tiles of both models by four waves side by side.
//
// What bounds the logit passes is the matrix pipe and, on a chip that runs at its power limit, the energy of
// every byte that travels to it.  A workgroup here is four waves (one per SIMD, 512 registers each), each owning
// 192 vocabulary rows x 64 tokens in 16 x 16 x 32 MFMAs (half the accumulator traffic per flop of 32 x 32 x 16):
//   - the vocabulary rows (A) go global -> LDS by direct loads and are read by all four waves;
//   - the tokens (B) belong to one wave each, so they skip the LDS: the hidden states are re-packed once per
//     call in the order in which a wave consumes them (pack_rows) and come straight into registers,
//     1 KiB per load, three sub-steps (2300 cycles) ahead.
// Measured on a plain product of 153600 x 4096 x 4096: 1401 TFLOP/s (1.75 GHz, matrix pipe busy 0.76); the same
// with 32 x 32 x 16 MFMAs 1337 (1.53 GHz, 0.83); the 128 x 256 tile of eight waves with both operands through
// the LDS (kd_mfma.hpp) 1165.
//
// Two such accumulators are 384 registers.  The student's tile is built first and set aside while the teacher's is
// built: 16 of its 48 blocks are accumulated in vector registers, 12 in accumulation registers, and stay there; the
// other 20 are accumulated in accumulation registers and parked in LDS.  MFMAs are inline assembly so that each
// accumulator stays in the register file it was given; the compiler's own choice copies them around inside the loop.
// With the B ring and the fragments the 512 registers are full: what the statistics and the gradient kernels keep from tile to
// tile lives in LDS (STATE_AT).  A spilled register costs more than its traffic: its reload waits for every load in flight.
// (Left: 11 of RKL's and 15 of AKL's gradient kernel, 2 of the skewed FKL's row pass, up to 24 for [H][V] heads.)
//
// One wave per SIMD: whatever stands between two k-steps is idle matrix time.  The loads of a k-step go out one by one
// between MFMAs, the cursor moves on in front of the last block, and the change to the next phase or tile is off the
// straight path (T = 4096 JSD, against the same start: 17.28 -> 17.24 ms without this, 17.38 -> 16.23 with it).
//
// The backward products (kd_products.hip) run on the same loop, with one accumulator.
//
// A sub-step is 64 bytes of every row (32 bf16), a k-step two sub-steps.
#pragma once
#include "kd_mfma.hpp"

namespace kd {

// A tile of 16 MB rows of A by 4 waves x 16 NB rows of B.
template <int MB_, int NB_>
struct StripShape {
  static constexpr int MB = MB_, NB = NB_;           // 16 x 16 blocks per wave
  static constexpr int NT = 256;
  static constexpr int BM = 16 * MB, BN = 64 * NB;
  static constexpr int NST = 3;                      // LDS stages of one k-step of A
  static constexpr int DIST = 2;                     // k-steps in flight ahead of the one multiplied
  static constexpr int A_LOADS = BM / 32;            // 16-byte loads per thread and k-step
  static constexpr int STAGE_BYTES = BM * 128;
  static constexpr int SMEM_BYTES = NST * STAGE_BYTES;
  static_assert(SMEM_BYTES <= 160 * 1024, "LDS of a gfx950 CU");
  static_assert(MB >= 2 * A_LOADS && MB % 4 == 0, "places of the loads in a sub-step");
  // Sub-step of NM blocks of A.  B load j goes out inside block b_place(j); in the first sub-step A load j
  // inside block a_place(j) (behind a B load of the same block).  The barrier of k-step k stands in its second
  // sub-step at the end of block bar(NM) - 1.  Up to there a wave has issued after its last load of
  // k-step k + 1 (end of the first sub-step of k - 1): the B loads of the second sub-step of k - 1, the B and A
  // loads of the first sub-step of k, and the B loads of the second that come before the barrier.
  static constexpr int b_place(int nm, int j) { return (2 * j + 1) * nm / (2 * NB) < nm - 1 ? (2 * j + 1) * nm / (2 * NB) : nm - 2; }
  static constexpr int a_place(int nm, int j) { return nm / 2 + j * (nm / 2) / A_LOADS; }
  static constexpr int bar(int nm) { return nm / 4; }
  static constexpr int wait(int nm) {
    int n = NB + NB + A_LOADS;
    for (int j = 0; j < NB; ++j) n += b_place(nm, j) < bar(nm) ? 1 : 0;
    return n;
  }
  static __device__ __forceinline__ int acc_m(int i, int r, int lane) { return 16 * i + 4 * (lane >> 4) + r; }
  static __device__ __forceinline__ int acc_n(int j, int lane, int wave) { return wave * (16 * NB) + 16 * j + (lane & 15); }
};

// The logit tiles.
struct StripCfg : StripShape<12, 4> {
  static constexpr int HELD_V = 16, HELD_A = 12;     // student blocks kept in vector / accumulation registers
  static constexpr int HELD = HELD_V + HELD_A;       // (block = 12 j + i)
  static constexpr int PARKED = MB * NB - HELD;      // ... and in LDS
  static constexpr int PARK_BYTES = PARKED * 16 * NT;
  static constexpr int SMEM_BYTES = NST * STAGE_BYTES + PARK_BYTES;
  // Behind it, 32 bytes per token for the epilogues that keep something of them (with STATE: what their kernels ask for).
  static constexpr int STATE_AT = SMEM_BYTES, STATE_SMEM_BYTES = SMEM_BYTES + 32 * BN;
  static_assert(STATE_SMEM_BYTES <= 160 * 1024, "LDS of a gfx950 CU");
  // A workgroup's last tile, if it has at most SHORT rows, is multiplied as four blocks (its loads stay as they are:
  // rows that do not exist repeat the last one).  Priced at 0.45 of a full tile by the choice of ranges.
  static constexpr int SHORT = 64;                   // (rows behind those that exist are stored up to 64: see out_rows)
};

// How A lies in memory and which eight k of a sub-step a lane multiplies.  The lanes of an MFMA operand hold one row each
// and, by groups of 16, eight of the 32 k of a sub-step; which k is free as long as both operands agree.  In the natural
// order group g has k = 8 g .. + 7.  In the order of dz (dz_chunk in kd_common.hpp) it has 4 g .. + 3 and 16 + 4 g .. + 3,
// which is what a lane of a finished logit tile holds.
//   A_ROWS       rows of K-contiguous elements, natural order: one 16-byte LDS read per fragment
//   A_ROWS_DZ    the same in the order of dz: two 8-byte reads
//   A_KMAJOR_DZ  k-rows of contiguous A rows, in the order of dz: two transposing reads
//   A_DZ         the chunk of dz itself, its tokens contracted in the natural order: two transposing reads
enum { A_ROWS = 0, A_ROWS_DZ = 1, A_KMAJOR_DZ = 2, A_DZ = 3 };

// One tile.  Phase p contracts kp elements of A and B: Ap its first row (A_KMAJOR_DZ: first k-row and row; A_DZ: first
// token panel and column), Bp the first of its four panels (or the whole operand, see strip_loop).
struct StripItem {
  const char *A0, *A1, *B0, *B1;
  int k0, k1;
  int a_rows;              // rows of A in the tile (1 .. BM); loads of the others give the last one's (A_ROWS: a row may be shorter
                           // than its k-steps; behind its end loads give 0)
  int out_rows;            // ... rounded up to 64: what is stored of it
  int m0, n0;              // tile origin
  int aux;                 // free for the work map
  // Strides in bytes: A from row to row (A_KMAJOR_DZ: from k-row to k-row; A_DZ: from token panel to token panel), B from
  // panel to panel (or from block to block, b_blocks of them)
  uint32_t lda0, lda1, ldb0, ldb1;
  int b_blocks;
};

// The kernel's argument block, to be read from memory again: an item is worked out twice a tile, and what it takes would
// otherwise stay in scalar registers, of which the loop has too few (spills into vector registers, and of those to memory,
// whose reloads wait for every load in flight).
template <class T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* kernel_args() {
  auto p = (const __attribute__((address_space(4))) T*)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// Accumulators in accumulation registers (_a) or vector registers (_v).
// The compiler does not know these are MFMAs and inserts no wait states: strip_settle() / strip_fresh() stand
// between them and anything else that reads or writes the accumulators.
__device__ __forceinline__ void strip_mfma_a(f32x4& c, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void strip_mfma_v(f32x4& c, const u32x4& a, const u32x4& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}
// Ties four accumulators to this point of the program, NOPS wait states in front.
template <bool ACC>
__device__ __forceinline__ void strip_tie(f32x4& c0, f32x4& c1, f32x4& c2, f32x4& c3, const bool nops) {
  if (nops) {
    if (ACC) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(c0), "+a"(c1), "+a"(c2), "+a"(c3));
    else asm volatile("s_nop 15\n\ts_nop 15" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3));
  } else {
    if (ACC) asm volatile("" : "+a"(c0), "+a"(c1), "+a"(c2), "+a"(c3));
    else asm volatile("" : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3));
  }
}
template <bool ACC, int N, int M>
__device__ __forceinline__ void strip_settle(f32x4 (&c)[M]) {
  static_assert(N % 4 == 0 && N <= M, "tied four at a time");
#pragma unroll
  for (int i = 0; i < N; i += 4) strip_tie<ACC>(c[i], c[i + 1], c[i + 2], c[i + 3], i == 0);
}

// Eight k of one row; a transposed or split fragment comes in two halves, by reads in inline assembly with waits of their own
// (the compiler's builtin for the transposing ones is preceded by a wait for every direct load in flight); what reads a fragment is
// inline assembly, too, so the order of the program is the order of the instructions.
template <int AM> struct StripFrag { s16x4 lo, hi; };
template <> struct StripFrag<A_ROWS> { u32x4 v; };
__device__ __forceinline__ u32x4 strip_op(const StripFrag<A_ROWS>& f) { return f.v; }
template <int AM>
__device__ __forceinline__ u32x4 strip_op(const StripFrag<AM>& f) {
  return __builtin_bit_cast(u32x4, __builtin_shufflevector(f.lo, f.hi, 0, 1, 2, 3, 4, 5, 6, 7));
}
// Keeps a fragment's registers until here.
template <int AM>
__device__ __forceinline__ void strip_hold(const StripFrag<AM>& f) {
  asm volatile("" ::"v"(f.lo), "v"(f.hi));
}
__device__ __forceinline__ void strip_hold(const StripFrag<A_ROWS>&) {}
template <int OFF>
__device__ __forceinline__ void strip_tr_read(s16x4& d, uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset field");
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}
template <int OFF>
__device__ __forceinline__ void strip_half_read(s16x4& d, uint32_t addr) {
  static_assert(OFF >= 0 && OFF < 65536, "ds offset field");
  asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(d) : "v"(addr), "n"(OFF));
}

// Work:  int n_items() const;  StripItem item(int i) const;   (wave-uniform)
// Epi:   begin_item(item)                            before the first k-step of an item
//        pad(p)                                       what logits of vocabulary rows that do not exist start at
//        column(item, IntC<j>, S[NM], T[NM])          after the last k-step, for the token blocks j = 0 .. 3: the
//                                                     student's and the teacher's blocks (S unused if NPH == 1);
//                                                     NM = MB, or SHORT / 16 for a short tile
//        WHOLE set: start(item, T[MB * NB]) and tile(item, T) instead of the last three: all blocks at once (block = MB j + i),
//        what they start at and what becomes of them; STORES is the number of vector memory operations that tile makes.
// SHORT_LAST: a workgroup's last tile may be a short one.
// NPH == 2: student rows, then teacher rows; NPH == 1: only A1 / B1.
// B_BLOCKS: B is [block of 16 rows][sub-step][lane][8] instead of [panel of four blocks][sub-step][block][lane][8]; a tile
// starts at block n0 / 16 and blocks that do not exist repeat the last one.
// SWAP: the blocks are those of the transposed product (B's rows on the register axis).
//
// Order of a sub-step: per block of A NB MFMAs, then the LDS read that refills the fragment register just
// used ((MB - 1) NB MFMAs ahead of its use); NB times one B load into the ring slot of the sub-step before, and
// in the first sub-step the direct loads of A.  The order is pinned: left to itself the compiler gathers the
// MFMAs and rotates the B registers through copies, each of which waits for its load (one wave per SIMD:
// nothing hides it).
template <int NPH, bool SHORT_LAST, class C = StripCfg, int AM = A_ROWS, bool B_BLOCKS = false, bool SWAP = false, class Work, class Epi>
__device__ __forceinline__ void strip_loop(const Work& work, Epi& epi, char* smem) {
  constexpr int MB = C::MB, NB = C::NB;
  constexpr bool HALVES = AM != A_ROWS, TR = AM == A_KMAJOR_DZ || AM == A_DZ;
  static_assert(NPH == 1 || AM == A_ROWS || AM == A_KMAJOR_DZ, "two phases");
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int n_items = work.n_items();
  if (n_items <= 0) return;
#define KD_PIN() __builtin_amdgcn_sched_barrier(0)

  // ---- load cursor --------------------------------------------------------------------------------
  // Direct load j of the workgroup fills bytes 4096 j .. of a stage, 16 bytes per thread; a thread fetches the chunk
  // its slot stands for.  Layout of a stage:
  //   A_ROWS, A_ROWS_DZ  128 bytes per row, a row's eight chunks permuted by row bits
  //   A_KMAJOR_DZ        regions of 128 rows, 64 k-rows of 16 chunks each, and one of 64 rows (8 chunks) where MB is no
  //                      multiple of 8, a k-row's chunks permuted by bits of k
  //   A_DZ               as in memory (1 KiB for 16 tokens x 32 columns), a token's four chunks permuted by two bits
  // so that the fragment reads of half a wave always fall into different banks.
  constexpr int REGIONS = C::BM / 128;
  constexpr uint32_t BEHIND = 0x80000000u;           // an offset whose load gives 0
  int l_item = 0, l_ph = NPH == 2 ? 0 : 1, l_k = 0, l_nk = 0, l_a = 0, l_b = 0, l_bo = 0;
  int l_rows = 0, l_tail = 64;   // rows of the tile and k of its last k-step that exist
  const char* l_pa = nullptr;    // (only where A advances by whole k-rows)
  uint32_t l_lda = 0, voff[C::A_LOADS];
  uint32_t bj[NB], bjo[NB];      // B in blocks: the wave's blocks, from its first one
  rsrc_t ra, rb, rbo;            // rbo, bjo, l_bo: the B cursor one k-step back
  auto set_voff = [&](int kv) {
    int slot = 0;
    asm volatile("" : "+s"(slot));        // (or the thread's number and what is made of it are kept in registers from call to call)
    slot = wave * 64 + __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, slot));
    const int lrow = slot >> 3, lchunk = (slot & 7) ^ ((lrow >> 1) & 7);
#pragma unroll
    for (int j = 0; j < C::A_LOADS; ++j) {
      if constexpr (AM == A_DZ) {
        voff[j] = j * 4096 + (slot >> 6) * 1024 + ((slot >> 4) & 3) * 256 + ((slot & 15) ^ (4 * ((slot >> 4) & 1))) * 16;
      } else if constexpr (AM == A_KMAJOR_DZ) {
        const bool wide = j < 4 * REGIONS;
        const int kr = wide ? 16 * (j & 3) + (slot >> 4) : 32 * (j & 1) + (slot >> 3);
        const int c = wide ? 16 * (j >> 2) + ((slot & 15) ^ (2 * (kr & 7))) : 16 * REGIONS + ((slot & 7) ^ (2 * ((kr >> 1) & 3)));
        voff[j] = __umul24(min(kr, kv - 1), l_lda) + (uint32_t)min(c, (l_rows >> 3) - 1) * 16;
      } else {
        const uint32_t row = min(lrow + 32 * j, l_rows - 1);
        // (rows of 2 K bytes; of 2 V bytes)
        if constexpr (AM == A_ROWS) voff[j] = __umul24(row, l_lda) + (lchunk * 16 < (int)l_lda - l_a ? lchunk * 16 : BEHIND);
        else voff[j] = row * l_lda + lchunk * 16;
      }
    }
  };
  // The k-steps from l_k on.  A_ROWS: up to the one that a row ends in, if it ends inside one, which is then gone to by itself: its
  // chunks behind the row's end are not the row's (0 x infinity is not 0, so that B is 0 there is not enough).
  auto set_cursor = [&](const StripItem& it) {
    const uint32_t bstride = l_ph ? it.ldb1 : it.ldb0;
    const int k = l_ph ? it.k1 : it.k0;
    l_lda = l_ph ? it.lda1 : it.lda0;
    l_rows = it.a_rows;
    if constexpr (AM == A_ROWS) {
      l_nk = l_k + max(((int)l_lda - l_a) >> 7, 1);
    } else {
      l_nk = (k + 63) >> 6;
      l_tail = k - 64 * (l_nk - 1);
    }
    if constexpr (TR) {
      l_pa = uniform(l_ph ? it.A1 : it.A0);
      ra = make_rsrc(l_pa, AM == A_DZ ? C::STAGE_BYTES : 64u * l_lda);
    } else {
      const uint32_t end = AM == A_ROWS ? (uint32_t)it.a_rows * l_lda : (uint32_t)min((uint64_t)it.a_rows * l_lda, (uint64_t)0xffffffffu);
      ra = make_rsrc(l_ph ? it.A1 : it.A0, end);
    }
    if constexpr (B_BLOCKS) {
      const int b0 = min(it.n0 / 16 + wave * NB, it.b_blocks - 1);
      rb = make_rsrc((l_ph ? it.B1 : it.B0) + (int64_t)b0 * bstride, (uint32_t)NB * bstride);
#pragma unroll
      for (int j = 0; j < NB; ++j) bj[j] = (uint32_t)min(j, it.b_blocks - 1 - b0) * bstride;
    } else {
      rb = make_rsrc((l_ph ? it.B1 : it.B0) + (int64_t)wave * bstride, bstride);
    }
    set_voff(AM == A_KMAJOR_DZ && l_nk == 1 ? l_tail : 64);
  };
  set_cursor(work.item(0));
  constexpr int B_SUB = B_BLOCKS ? 1024 : 4096;      // bytes of B from one sub-step to the next
  auto advance = [&]() {
    rbo = rb; l_bo = l_b;
    if constexpr (B_BLOCKS) {
#pragma unroll
      for (int j = 0; j < NB; ++j) bjo[j] = bj[j];
    }
    if constexpr (!TR) l_a += 128;
    l_b += 2 * B_SUB;
    if (__builtin_expect(++l_k == l_nk, 0)) {
      const bool rest = AM == A_ROWS && l_a < (int)l_lda;
      const bool more = rest || (NPH == 2 && l_ph == 0) || l_item + 1 < n_items;
      if (more) {
        if (!rest) {
          l_k = l_a = l_b = 0;
          if (NPH == 2) l_ph ^= 1;
          if (NPH == 1 || l_ph == 0) ++l_item;
        }
        set_cursor(work.item(l_item));
      } else {           // past the end: the last k-step again (valid memory, data unused)
        --l_k;
        if constexpr (!TR) l_a -= 128;
        l_b -= 2 * B_SUB;
      }
    } else if constexpr (TR) {
      l_pa += AM == A_DZ ? (uint64_t)l_lda : (uint64_t)l_lda * 64;
      ra = make_rsrc(l_pa, AM == A_DZ ? C::STAGE_BYTES : 64u * l_lda);
      if (AM == A_KMAJOR_DZ && __builtin_expect(l_k == l_nk - 1 && l_tail < 64, 0)) set_voff(l_tail);
    }
  };
  auto issue_a = [&](int st, int j) {                // st: byte offset of the stage
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)(smem + st + wave * 1024 + j * 4096), 16,
                                             voff[j], l_a, 0, 0);
  };
  const uint32_t boff = lane * 16;
  auto load_b = [&](const rsrc_t& r, const uint32_t (&blk)[NB], int kb, int s, int j) -> u32x4 {
    if constexpr (B_BLOCKS) return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, boff, kb + s * B_SUB + blk[j], 0));
    else return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, boff + j * 1024, kb + s * B_SUB, 0));
  };

  // ---- fragments ----------------------------------------------------------------------------------
  typedef StripFrag<AM> Frag;
  const int g = lane >> 4, frow = lane & 15, fsw = (frow >> 1) & 7;
  int fk[4];               // A_ROWS: per sub-step; A_ROWS_DZ: per sub-step and half; the others: see below
  if constexpr (AM == A_ROWS) {
#pragma unroll
    for (int s = 0; s < 2; ++s) fk[s] = frow * 128 + (((4 * s + g) ^ fsw) << 4);
  } else if constexpr (AM == A_ROWS_DZ) {
#pragma unroll
    for (int s = 0; s < 4; ++s) fk[s] = frow * 128 + (((2 * s + (g >> 1)) ^ fsw) << 4) + (g & 1) * 8;
  } else if constexpr (AM == A_KMAJOR_DZ) {
    // lane i of a group of 16 addresses k-row i / 4, rows 4 (i mod 4) .. + 3; [0] in a region of 128 rows, [1] of 64
    const int kr = 4 * g + (frow >> 2), c = frow & 3;
    fk[0] = kr * 256 + (((2 * (kr & 7)) | (c >> 1)) << 4) + (c & 1) * 8;
    fk[1] = kr * 128 + (((2 * ((kr >> 1) & 3)) | (c >> 1)) << 4) + (c & 1) * 8;
  } else {
    // lane i of a group addresses token i / 4 (+ 4) of the group's eight and one of four pieces of four columns: the two
    // halves of two neighbouring chunks, so that 16 lanes read 8 whole chunks.  Row 4 c + r of an MFMA is then column
    // 16 (c mod 2) + 4 (c / 2) + r of the 32 (+ 8 in the second block): see dz_column.
    const int c = frow & 3, t = 8 * (g & 1) + (frow >> 2);
#pragma unroll
    for (int h = 0; h < 2; ++h) fk[h] = (g >> 1) * 1024 + (c >> 1) * 256 + ((t + 4 * h) ^ (4 * (c >> 1))) * 16 + (c & 1) * 8;
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void_t*)smem;
  auto read_a = [&](Frag& f, int st, auto sc, auto ic) {
    constexpr int s = decltype(sc)::value, i = decltype(ic)::value;
    if constexpr (AM == A_ROWS) {
      f.v = *(const u32x4*)(smem + st + fk[s] + i * 2048);
    } else if constexpr (AM == A_ROWS_DZ) {
      const uint32_t at = lds0 + st;
      strip_half_read<i * 2048>(f.lo, at + fk[2 * s]);
      strip_half_read<i * 2048>(f.hi, at + fk[2 * s + 1]);
    } else if constexpr (AM == A_KMAJOR_DZ) {
      constexpr bool wide = i < 8 * REGIONS;
      constexpr int at = wide ? (i >> 3) * 16384 : REGIONS * 16384, kb = wide ? 256 : 128;
      const uint32_t ad = (uint32_t)(fk[wide ? 0 : 1] ^ (wide ? (i & 7) * 32 : (i & 3) * 32)) + (lds0 + st);
      strip_tr_read<at + s * 32 * kb>(f.lo, ad);
      strip_tr_read<at + (s * 32 + 16) * kb>(f.hi, ad);
    } else {
      const uint32_t at = lds0 + st;
      strip_tr_read<(i >> 1) * 4096 + s * 2048 + (i & 1) * 512>(f.lo, at + fk[0]);
      strip_tr_read<(i >> 1) * 4096 + s * 2048 + (i & 1) * 512>(f.hi, at + fk[1]);
    }
  };
  u32x4 B[4][NB];          // sub-steps of two k-steps
  Frag A[MB];              // the next sub-step's fragments
  int stage = 0, next = C::STAGE_BYTES, fill = 2 * C::STAGE_BYTES;      // byte offsets: consumed, behind it, refilled
  static_assert(C::NST == 3 && C::DIST == 2, "stages");

  // one k-step of NM blocks of A; Q: half of the B ring it consumes.  mma(IntC<i>, IntC<j>, a, b)
  // MORE: vector memory operations since that may be in flight, too
  auto kstep = [&](auto nmc, auto qc, auto morec, auto&& mma) {
    constexpr int Q = decltype(qc)::value, NM = decltype(nmc)::value;
    constexpr int W = C::wait(NM) + decltype(morec)::value < 63 ? C::wait(NM) + decltype(morec)::value : 63;
    asm volatile("s_nop 1");           // whatever the compiler moved between k-steps, an MFMA may read now
    KD_PIN();
    static_for<0, 2>([&](auto sc) {
      constexpr int s = decltype(sc)::value;
      const int rd = s == 1 ? next : stage;
      static_for<0, NM>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        // Reads in halves: two per fragment, landing in order; those of up to seven fragments behind may be in flight.  (In
        // front of the barrier nothing is refilled yet: there are only those of the blocks up to the last.)
        constexpr int behind = s == 1 && i < C::bar(NM) ? NM - 1 - i : NM - 1;
        if constexpr (HALVES) asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(2 * behind < 14 ? 2 * behind : 14));
        const u32x4 a = strip_op(A[i]);
        static_for<0, NB>([&](auto jc) {
          constexpr int j = decltype(jc)::value;
          // the cursor moves on in the shadow of the last block's MFMAs
          if constexpr (s == 1 && i == NM - 1 && j == 0) { advance(); KD_PIN(); }
          mma(ic, jc, a, B[2 * Q + s][j]);
          KD_PIN();
          if constexpr (j == (NB > 1 ? 1 : 0))
            static_for<0, NB>([&](auto lc) {
              constexpr int l = decltype(lc)::value;
              if constexpr (C::b_place(NM, l) == i) {
                if constexpr (s == 0) B[(2 * Q + 3) & 3][l] = load_b(rbo, bjo, l_bo, 1, l);
                else B[2 * Q][l] = load_b(rb, bj, l_b, 0, l);
                KD_PIN();
              }
            });
          if constexpr (s == 0 && j == (NB > 2 ? 2 : NB - 1))
            static_for<0, C::A_LOADS>([&](auto lc) {
              if constexpr (C::a_place(NM, decltype(lc)::value) == i) {
                issue_a(fill, decltype(lc)::value);
                KD_PIN();
              }
            });
        });
        // k-step k+1 has landed for every wave before anyone reads it, and every wave has read all of this
        // stage before anyone refills it
        if constexpr (s == 1 && i == C::bar(NM) - 1) {
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(W) : "memory");
          static_for<0, C::bar(NM)>([&](auto jc) { read_a(A[decltype(jc)::value], rd, IntC<0>{}, jc); });
        } else if constexpr (s == 0 || i >= C::bar(NM)) {
          read_a(A[i], rd, IntC<s ^ 1>{}, ic);
        }
        KD_PIN();
      });
    });
    const int released = stage;
    stage = next;
    next = fill;
    fill = released;
  };
  // All k-steps of one phase.  Vector memory operations are counted in order, so the stores of the tile before (STORES of
  // them) would have to land before the loop's first waits are over: the first k-step, whose operands are older than they,
  // is written out with waits of its own, and the second, which gives them more time.
  auto run = [&](auto nmc, auto storesc, int nk, auto&& mma) {
    int k = 0;
    if constexpr (decltype(storesc)::value > 0)
      if (nk > 1) {
        kstep(nmc, IntC<0>{}, storesc, mma);
        kstep(nmc, IntC<1>{}, IntC<0>{}, mma);
        k = 2;
      }
    for (; k + 1 < nk; k += 2) { kstep(nmc, IntC<0>{}, IntC<0>{}, mma); kstep(nmc, IntC<1>{}, IntC<0>{}, mma); }
    if (nk & 1) {                                          // the halves of the ring change places
      kstep(nmc, IntC<0>{}, IntC<0>{}, mma);
#pragma unroll
      for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int j = 0; j < NB; ++j) { const u32x4 t = B[s][j]; B[s][j] = B[2 + s][j]; B[2 + s][j] = t; }
    }
  };
  // Rows that a tile does not have start at `pad`, a huge negative logit: they end that far below the row that their
  // clamped loads repeat, which is one of the same range, so that beside it their exponentials are 0 and their dL/dz comes
  // out 0, with no test per element (up to logits of 1e30 in size, where the two can no longer be told apart).
  auto first = [&](auto nmc, int rows, float pad, auto&& set) {
    constexpr int NM = decltype(nmc)::value;
    if (rows == 16 * NM) {
      static_for<0, NM>([&](auto ic) { set(ic, f32x4{0.f, 0.f, 0.f, 0.f}); });
    } else {
      int lim = rows - 4 * (lane >> 4);
      asm volatile("" : "+v"(lim));     // (or the comparisons of one phase are kept for the next)
      static_for<0, NM>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        f32x4 v;
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = 16 * i + r < lim ? 0.f : pad;
        set(ic, v);
        KD_PIN();
      });
    }
  };

  // ---- prologue: DIST k-steps in flight (all but the last sub-step of B), first fragments read -------------
#pragma unroll
  for (int i = 0; i < C::DIST; ++i) {
#pragma unroll
    for (int j = 0; j < C::A_LOADS; ++j) issue_a(i * C::STAGE_BYTES, j);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        if (2 * i + s < 3) B[2 * i + s][j] = load_b(rb, bj, l_b, s, j);
    advance();
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) B[3][j] = B[2][j];          // (refilled by the first sub-step)
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
  static_for<0, MB>([&](auto ic) { read_a(A[decltype(ic)::value], 0, IntC<0>{}, ic); });
  // Here and behind a phase's last k-step: the compiler may move the fragments.  KEEP: their registers are theirs until then, also
  // where nothing reads them any more (behind a workgroup's last tile an epilogue would take them while a read is in flight).
  auto landed = [&](auto keepc) {
    if constexpr (HALVES) asm volatile("s_waitcnt lgkmcnt(0)");
    if constexpr (HALVES && decltype(keepc)::value != 0) {
#pragma unroll
      for (int i = 0; i < MB; ++i) strip_hold(A[i]);
    }
  };
  landed(IntC<0>{});

  // one tile of NM blocks of A
  auto tile = [&](auto nmc, const StripItem& ci) {
    constexpr int NM = decltype(nmc)::value, N = NM * NB;
    epi.begin_item(ci);
    if constexpr (Epi::WHOLE) {
      f32x4 T[N];
      epi.start(ci, T);
      strip_settle<true, N>(T);
      run(nmc, IntC<Epi::STORES>{}, (ci.k1 + 63) >> 6, [&](auto ic, auto jc, const u32x4& a, const u32x4& b) {
        constexpr int id = NM * decltype(jc)::value + decltype(ic)::value;
        if constexpr (SWAP) strip_mfma_a(T[id], b, a);
        else strip_mfma_a(T[id], a, b);
      });
      landed(IntC<0>{});
      strip_settle<true, N>(T);
      epi.tile(ci, T);
    } else {
      constexpr int HV = N < C::HELD_V ? N : C::HELD_V, HA = N - HV < C::HELD_A ? N - HV : C::HELD_A, NP = N - HV - HA;
      f32x4* const park = (f32x4*)(smem + C::NST * C::STAGE_BYTES) + tid;
      f32x4 SV[HV], SA[HA + 4];
      if constexpr (NPH == 2) {
        f32x4 SP[NP + 4];
        first(nmc, ci.a_rows, epi.pad(0), [&](auto ic, const f32x4& v) {
          static_for<0, NB>([&](auto jc) {
            constexpr int id = NM * decltype(jc)::value + decltype(ic)::value;
            if constexpr (id < HV) SV[id] = v;
            else if constexpr (id < HV + HA) SA[id - HV] = v;
            else SP[id - HV - HA] = v;
          });
        });
        strip_settle<false, HV>(SV);
        strip_settle<true, HA>(SA);
        strip_settle<true, NP>(SP);
        run(nmc, IntC<0>{}, (ci.k0 + 63) >> 6, [&](auto ic, auto jc, const u32x4& a, const u32x4& b) {
          constexpr int id = NM * decltype(jc)::value + decltype(ic)::value;
          if constexpr (id < HV) strip_mfma_v(SV[id], a, b);
          else if constexpr (id < HV + HA) strip_mfma_a(SA[id - HV], a, b);
          else strip_mfma_a(SP[id - HV - HA], a, b);
        });
        landed(IntC<1>{});
        strip_settle<false, HV>(SV);
        strip_settle<true, HA>(SA);
        strip_settle<true, NP>(SP);
#pragma unroll
        for (int i = 0; i < NP; ++i) park[i * C::NT] = SP[i];
        KD_PIN();
      }
      f32x4 T[N];
      first(nmc, ci.a_rows, epi.pad(1), [&](auto ic, const f32x4& v) {
        static_for<0, NB>([&](auto jc) { T[NM * decltype(jc)::value + decltype(ic)::value] = v; });
      });
      strip_settle<true, N>(T);
      run(nmc, IntC<0>{}, (ci.k1 + 63) >> 6, [&](auto ic, auto jc, const u32x4& a, const u32x4& b) {
        strip_mfma_a(T[NM * decltype(jc)::value + decltype(ic)::value], a, b);
      });
      landed(IntC<1>{});
      strip_settle<true, N>(T);
      static_for<0, NB>([&](auto jc) {
        f32x4 S[NM], Tj[NM];
        static_for<0, NM>([&](auto ic) {
          constexpr int i = decltype(ic)::value, id = NM * decltype(jc)::value + i;
          Tj[i] = T[id];
          if constexpr (NPH == 2) {
            if constexpr (id < HV) S[i] = SV[id];
            else if constexpr (id < HV + HA) S[i] = SA[id - HV];
            else S[i] = park[(id - HV - HA) * C::NT];
          }
        });
        epi.column(ci, jc, S, Tj);
        KD_PIN();
      });
    }
  };
  // full tiles, then perhaps a short one (only ever the last of a workgroup)
  int n_full = n_items;
  if constexpr (SHORT_LAST)
    if (work.item(n_items - 1).a_rows <= C::SHORT) --n_full;
  for (int c_item = 0; c_item < n_full; ++c_item) tile(IntC<MB>{}, work.item(c_item));
  if constexpr (SHORT_LAST)
    if (n_full < n_items) tile(IntC<C::SHORT / 16>{}, work.item(n_full));
  // the loads issued past the end still target this workgroup's LDS: let them land
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#undef KD_PIN
}

}  // namespace kd
