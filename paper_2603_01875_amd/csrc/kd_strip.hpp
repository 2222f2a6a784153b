// The logit tile loop: 192 (vocabulary) x 256 (token) tiles of both models by four waves side by side.
//
// What bounds the logit passes is the matrix pipe and, on a chip that runs at its power limit, the energy of
// every byte that travels to it.  A workgroup here is four waves (one per SIMD, 512 registers each), each owning
// 192 vocabulary rows x 64 tokens in 16 x 16 x 32 MFMAs (half the accumulator traffic per flop of 32 x 32 x 16):
//   - the vocabulary rows (A) go global -> LDS by direct loads and are read by all four waves;
//   - the tokens (B) belong to one wave each, so they skip the LDS: the hidden states are re-packed once per
//     call in the order in which a wave consumes them (pack_rows_kernel) and come straight into registers,
//     1 KiB per load, three sub-steps (2300 cycles) ahead.
// Measured on a plain product of 153600 x 4096 x 4096: 1401 TFLOP/s (1.75 GHz, matrix pipe busy 0.76); the same
// with 32 x 32 x 16 MFMAs 1337 (1.53 GHz, 0.83); the 128 x 256 tile of eight waves with both operands through
// the LDS (kd_mfma.hpp) 1165.
//
// Two such accumulators are 384 registers.  The student's tile is built first and set aside while the teacher's is
// built: 16 of its 48 blocks are accumulated in vector registers, 12 in accumulation registers, and stay there; the
// other 20 are accumulated in accumulation registers and parked in LDS.  MFMAs are inline assembly so that each
// accumulator stays in the register file it was given; the compiler's own choice copies them around inside the loop.
// With the B ring and the fragments the 512 registers do not quite hold what an epilogue needs: 1 to 33 of them are
// spilled between tiles and in epilogues (up to 132 bytes of scratch per lane, under a hundred scratch instructions in a
// kernel), none inside a k-loop.
//
// Operands are described in bytes per row: a sub-step is 64 bytes of every row (32 bf16), a k-step two sub-steps.
#pragma once
#include "kd_mfma.hpp"

namespace kd {

struct StripCfg {
  static constexpr int MB = 12, NB = 4;              // 16 x 16 blocks per wave
  static constexpr int NT = 256;
  static constexpr int BM = 16 * MB;
  static constexpr int NST = 3;                      // LDS stages of one k-step of A
  static constexpr int DIST = 2;                     // k-steps in flight ahead of the one multiplied
  static constexpr int A_LOADS = BM / 32;            // 16-byte loads per thread and k-step
  static constexpr int STAGE_BYTES = BM * 128;
  static constexpr int HELD_V = 16, HELD_A = 12;     // student blocks kept in vector / accumulation registers
  static constexpr int HELD = HELD_V + HELD_A;       // (block = 12 j + i)
  static constexpr int PARKED = MB * NB - HELD;      // ... and in LDS
  static constexpr int PARK_BYTES = PARKED * 16 * NT;
  static constexpr int SMEM_BYTES = NST * STAGE_BYTES + PARK_BYTES;
  static_assert(SMEM_BYTES <= 160 * 1024, "LDS of a gfx950 CU");
  // A workgroup's last tile, if it has at most SHORT rows, is multiplied as four blocks (its loads stay as they are:
  // rows that do not exist repeat the last one).  Priced at 0.45 of a full tile by the choice of ranges.
  static constexpr int SHORT = 64;                   // (rows behind those that exist are stored up to 64: see out_rows)
  static_assert(MB >= 2 * A_LOADS && MB % 4 == 0, "places of the loads in a sub-step");
  // Sub-step of NM vocabulary blocks.  B load j goes out after block b_place(j); in the first sub-step A load j
  // after block a_place(j) (behind a B load of the same block).  The barrier of k-step k stands in its second
  // sub-step before the LDS read of block bar(NM) - 1.  Up to there a wave has issued after its last load of
  // k-step k + 1 (end of the first sub-step of k - 1): the B loads of the second sub-step of k - 1, the B and A
  // loads of the first sub-step of k, and the B loads of the second that come before the barrier.
  static constexpr int b_place(int nm, int j) { return (2 * j + 1) * nm / 8; }
  static constexpr int a_place(int nm, int j) { return nm / 2 + j * (nm / 2) / A_LOADS; }
  static constexpr int bar(int nm) { return nm / 4; }
  static constexpr int wait(int nm) {
    int n = NB + NB + A_LOADS;
    for (int j = 0; j < NB; ++j) n += b_place(nm, j) < bar(nm) - 1 ? 1 : 0;
    return n;
  }
  static __device__ __forceinline__ int acc_m(int i, int r, int lane) { return 16 * i + 4 * (lane >> 4) + r; }
  static __device__ __forceinline__ int acc_n(int j, int lane, int wave) { return wave * 64 + 16 * j + (lane & 15); }
};

// One tile: A0 / A1 the first vocabulary row of the student's / teacher's head, B0 / B1 the packed panels of the
// token tile (four 64-token panels, one per wave).
struct StripItem {
  const char *A0, *A1, *B0, *B1;
  int a_rows;              // vocabulary rows of the tile (1 .. BM); loads of the others give the last one's
  int out_rows;            // ... rounded up to 64: what is stored of it
  int m0, n0;              // tile origin
};

typedef __amdgpu_buffer_rsrc_t rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>((const void*)uniform((const char*)p)), 0,
                                           __builtin_amdgcn_readfirstlane(bytes), 0x00020000);
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

// Work:  int n_items() const;  StripItem item(int i) const;   (wave-uniform)
// Epi:   begin_item(item)                            before the first k-step of an item
//        pad(p)                                       what logits of vocabulary rows that do not exist start at
//        column(item, IntC<j>, S[NM], T[NM])          after the last k-step, for the token blocks j = 0 .. 3: the
//                                                     student's and the teacher's blocks (S unused if NPH == 1);
//                                                     NM = MB, or SHORT / 16 for a short tile
// SHORT_LAST: a workgroup's last tile may be a short one.
// NPH == 2: student rows of rb0 bytes, then teacher rows of rb1 bytes; NPH == 1: only A1 / B1 with rb1.
//
// Order of a sub-step: per vocabulary block four MFMAs, then the LDS read that refills the fragment register just
// used (44 MFMAs ahead of its use); every third block one B load into the ring slot of the sub-step before, and
// in the first sub-step the direct loads of A.  The order is pinned: left to itself the compiler gathers the
// MFMAs and rotates the B registers through copies, each of which waits for its load (one wave per SIMD:
// nothing hides it).
template <int NPH, bool SHORT_LAST, class Work, class Epi>
__device__ __forceinline__ void strip_loop(const Work& work, Epi& epi, const int rb0, const int rb1, char* smem) {
  typedef StripCfg C;
  constexpr int MB = C::MB, NB = C::NB;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int n_items = work.n_items();
  if (n_items <= 0) return;
#define KD_PIN() __builtin_amdgcn_sched_barrier(0)

  // ---- load cursor --------------------------------------------------------------------------------
  // Direct load j of the workgroup fills tile rows 32 j .. 32 j + 31 (eight 16-byte chunks each, permuted by
  // row bits so that the fragment reads are conflict-free); a thread fetches the chunk its slot stands for.
  const int lrow = tid >> 3, lchunk = (tid & 7) ^ ((lrow >> 1) & 7);
  int l_item = 0, l_ph = NPH == 2 ? 0 : 1, l_k = 0, l_nk = 0, l_a = 0, l_b = 0, l_bo = 0;
  uint32_t voff[C::A_LOADS];
  rsrc_t ra, rb, rbo;            // rbo, l_bo: the B cursor one k-step back
  auto set_cursor = [&](const StripItem& it) {
    const int rbytes = l_ph ? rb1 : rb0;
    ra = make_rsrc(l_ph ? it.A1 : it.A0, (uint32_t)it.a_rows * (uint32_t)rbytes);
    rb = make_rsrc((l_ph ? it.B1 : it.B0) + (int64_t)wave * 64 * rbytes, 64u * (uint32_t)rbytes);
#pragma unroll
    for (int j = 0; j < C::A_LOADS; ++j) voff[j] = (uint32_t)min(lrow + 32 * j, it.a_rows - 1) * (uint32_t)rbytes + lchunk * 16;
    l_nk = rbytes >> 7;
    l_a = l_b = 0;
  };
  set_cursor(work.item(0));
  auto advance = [&]() {
    rbo = rb; l_bo = l_b;
    l_a += 128; l_b += 8192;
    if (++l_k == l_nk) {
      const bool more = (NPH == 2 && l_ph == 0) || l_item + 1 < n_items;
      if (more) {
        l_k = 0;
        if (NPH == 2) l_ph ^= 1;
        if (NPH == 1 || l_ph == 0) ++l_item;
        set_cursor(work.item(l_item));
      } else {           // past the end: the last k-step again (valid memory, data unused)
        l_a -= 128; l_b -= 8192; --l_k;
      }
    }
  };
  auto issue_a = [&](int st, int j) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)(smem + st * C::STAGE_BYTES + wave * 1024 + j * 4096), 16,
                                             voff[j], l_a, 0, 0);
  };
  const uint32_t boff = lane * 16;
  auto load_b = [&](const rsrc_t& r, int kb, int s, int j) -> u32x4 {
    return __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(r, boff + j * 1024, kb + s * 4096, 0));
  };

  // ---- fragments ----------------------------------------------------------------------------------
  const int frow = lane & 15, fsw = (frow >> 1) & 7;
  int fk[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) fk[s] = frow * 128 + (((4 * s + (lane >> 4)) ^ fsw) << 4);
  u32x4 B[4][NB];          // sub-steps of two k-steps
  u32x4 A[MB];             // the next sub-step's fragments
  int stage = 0, fill = C::DIST;

  // one k-step of NM vocabulary blocks; Q: half of the B ring it consumes.  mma(IntC<i>, IntC<j>, a, b)
  auto kstep = [&](auto nmc, auto qc, auto&& mma) {
    constexpr int Q = decltype(qc)::value, NM = decltype(nmc)::value;
    const int next = stage == C::NST - 1 ? 0 : stage + 1;
    asm volatile("s_nop 1");           // whatever the compiler moved between k-steps, an MFMA may read now
    KD_PIN();
    static_for<0, 2>([&](auto sc) {
      constexpr int s = decltype(sc)::value;
      const char* rd = smem + (s == 1 ? next : stage) * C::STAGE_BYTES + fk[s ^ 1];
      static_for<0, NM>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        static_for<0, NB>([&](auto jc) {
          mma(ic, jc, A[i], B[2 * Q + s][decltype(jc)::value]);
          KD_PIN();
        });
        // k-step k+1 has landed for every wave before anyone reads it, and every wave has read all of this
        // stage before anyone refills it
        if constexpr (s == 1 && i == C::bar(NM) - 1) {
          asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(C::wait(NM)) : "memory");
          static_for<0, C::bar(NM)>([&](auto jc) { A[decltype(jc)::value] = *(const u32x4*)(rd + decltype(jc)::value * 2048); });
        } else if constexpr (s == 0 || i >= C::bar(NM)) {
          A[i] = *(const u32x4*)(rd + i * 2048);
        }
        static_for<0, NB>([&](auto jc) {
          constexpr int j = decltype(jc)::value;
          if constexpr (C::b_place(NM, j) == i) {
            if constexpr (s == 0) B[(2 * Q + 3) & 3][j] = load_b(rbo, l_bo, 1, j);
            else B[2 * Q][j] = load_b(rb, l_b, 0, j);
          }
        });
        if constexpr (s == 0)
          static_for<0, C::A_LOADS>([&](auto jc) {
            if constexpr (C::a_place(NM, decltype(jc)::value) == i) issue_a(fill, decltype(jc)::value);
          });
        KD_PIN();
      });
    });
    advance();
    stage = next;
    fill = fill == C::NST - 1 ? 0 : fill + 1;
  };
  // all k-steps of one phase
  auto run = [&](auto nmc, int nk, auto&& mma) {
    for (int k = 0; k + 1 < nk; k += 2) { kstep(nmc, IntC<0>{}, mma); kstep(nmc, IntC<1>{}, mma); }
    if (nk & 1) {                                          // the halves of the ring change places
      kstep(nmc, IntC<0>{}, mma);
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
    for (int j = 0; j < C::A_LOADS; ++j) issue_a(i, j);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int j = 0; j < NB; ++j)
        if (2 * i + s < 3) B[2 * i + s][j] = load_b(rb, l_b, s, j);
    advance();
  }
#pragma unroll
  for (int j = 0; j < NB; ++j) B[3][j] = B[2][j];          // (refilled by the first sub-step)
  asm volatile("s_waitcnt vmcnt(0)\n\ts_barrier" ::: "memory");
#pragma unroll
  for (int i = 0; i < MB; ++i) A[i] = *(const u32x4*)(smem + fk[0] + i * 2048);
  const int nk0 = rb0 >> 7, nk1 = rb1 >> 7;
  f32x4* const park = (f32x4*)(smem + C::NST * C::STAGE_BYTES) + tid;

  // one tile of NM blocks
  auto tile = [&](auto nmc, const StripItem& ci) {
    constexpr int NM = decltype(nmc)::value, N = NM * NB;
    constexpr int HV = N < C::HELD_V ? N : C::HELD_V, HA = N - HV < C::HELD_A ? N - HV : C::HELD_A, NP = N - HV - HA;
    epi.begin_item(ci);
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
      run(nmc, nk0, [&](auto ic, auto jc, const u32x4& a, const u32x4& b) {
        constexpr int id = NM * decltype(jc)::value + decltype(ic)::value;
        if constexpr (id < HV) strip_mfma_v(SV[id], a, b);
        else if constexpr (id < HV + HA) strip_mfma_a(SA[id - HV], a, b);
        else strip_mfma_a(SP[id - HV - HA], a, b);
      });
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
    run(nmc, nk1, [&](auto ic, auto jc, const u32x4& a, const u32x4& b) {
      strip_mfma_a(T[NM * decltype(jc)::value + decltype(ic)::value], a, b);
    });
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
  };
  // full tiles, then perhaps a short one (only ever the last of a workgroup)
  int n_full = n_items;
  if (SHORT_LAST && work.item(n_items - 1).a_rows <= C::SHORT) --n_full;
  for (int c_item = 0; c_item < n_full; ++c_item) tile(IntC<MB>{}, work.item(c_item));
  if constexpr (SHORT_LAST)
    if (n_full < n_items) tile(IntC<C::SHORT / 16>{}, work.item(n_full));
  // the loads issued past the end still target this workgroup's LDS: let them land
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#undef KD_PIN
}

}  // namespace kd
