// The backward products on a chunk of dL/dz_s (dz), and what prepares and finishes them:
//   grad_W_s[v][h] (+)= sum_t dz[t][v] h_s[t][h]        complete per chunk, stored straight to the output
//   grad_h_s[t][h]  +=  sum_v dz[t][v] W_s[v][h]        fp32 partial sums, split over v where there are few tiles
// Both run on the strip loop (kd_strip.hpp) with one accumulator of up to 256 x 256: one operand goes through the LDS, the
// other straight to registers.  dz lies in the order in which a lane of a logit tile held it (dz_chunk): as the token
// operand of grad_h_s it is loaded as it is; as the column operand of grad_W_s its tokens are the contraction, and the
// transposing LDS reads turn it.  W_s is read over its outer index by the same reads; h_s is packed transposed once a call.
// Bound by the matrix pipe and the chip's power, like the logit passes, and, the shorter the contraction, by the start and
// the stores of a tile, which one wave per SIMD does not hide.  Measured against the eight-wave loop that read both operands
// through the LDS and dz as [T][V_c] (us a chunk; T tokens x columns x H_s): grad_W_s 32768 x 8192 x 4096 1686 -> 1511 (1.45
// PFLOP/s), 3584 x 16384 x 1024 111 -> 98, 256 x 151936 x 1024 224 -> 158; grad_h_s 32768 x 8192 x 4096 1866 -> 1674,
// 7424 x 8192 x 2048 238 -> 211, 3584 x 151936 x 1024, a call in ten chunks, 1.18 ms (1.24 with 256 rows x 4 parts).
#include "kd_common.hpp"

namespace kd {

// Where lane (g, n) holds rows 4 g .. + 3 of each of four 16-row blocks, as two words of two bf16: a 4 x 4 transposition of
// these 8-byte pieces between the four lanes of n gives each of them the 16 rows of one block.
__device__ __forceinline__ void quad_transpose(uint32_t (&x)[4][2]) {
#pragma unroll
  for (int d = 0; d < 2; ++d) {
    // (x0, x2), (x1, x3): the upper 32 lanes of the first against the lower 32 of the second; then
    // (x0, x1), (x2, x3) in the same way by rows of 16 lanes
    auto r0 = __builtin_amdgcn_permlane32_swap(x[0][d], x[2][d], false, false);
    auto r1 = __builtin_amdgcn_permlane32_swap(x[1][d], x[3][d], false, false);
    auto s0 = __builtin_amdgcn_permlane16_swap(r0[0], r1[0], false, false);
    auto s1 = __builtin_amdgcn_permlane16_swap(r0[1], r1[1], false, false);
    x[0][d] = s0[0]; x[1][d] = s0[1]; x[2][d] = s1[0]; x[3][d] = s1[1];
  }
}
__device__ __forceinline__ bf16x4 to_bf16(const f32x4& v) {
  bf16x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) o[i] = (bf16_t)v[i];
  return o;
}
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x2 pack4(const f32x4& v) { return __builtin_bit_cast(u32x2, to_bf16(v)); }

// Results leave, and what they are added to comes, by buffer operations: one whose offset lies past the buffer's end does
// nothing (a load gives 0), so rows and columns that do not exist take no branch.  (Behind one, all of the accumulator would
// be copied from accumulation to vector registers at once.)
constexpr uint32_t NOWHERE = 0xfffffff0u;
// Cache policy of a store that nothing reads soon: it does not push out of the last-level cache what the next kernel reads.
constexpr int STREAM = 2;
// The lane, as something that has to be worked out again: offsets made from it are not kept from tile to tile (spills).
__device__ __forceinline__ int fresh(int lane) {
  asm volatile("" : "+v"(lane));
  return lane;
}
// four neighbouring results of F32 or bf16 elements
template <bool F32>
__device__ __forceinline__ f32x4 load4(const rsrc_t& r, uint32_t at) {
  if constexpr (F32) {
    return __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, at, 0, 0));
  } else {
    const bf16x4 x = __builtin_bit_cast(bf16x4, __builtin_amdgcn_raw_buffer_load_b64(r, at, 0, 0));
    return f32x4{(float)x[0], (float)x[1], (float)x[2], (float)x[3]};
  }
}
template <bool F32>
__device__ __forceinline__ void store4(const rsrc_t& r, uint32_t at, const f32x4& v) {
  if constexpr (F32) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, at, 0, 0);
  else __builtin_amdgcn_raw_buffer_store_b64(pack4(v), r, at, 0, 0);
}

// ------------------------------------------------------------------------------------------
// grad_W_s
// ------------------------------------------------------------------------------------------
struct GradWArgs {
  const char* dz;          // the chunk
  const char* hT;          // h_s transposed and packed (pack_columns in kd_kernels.hip)
  void* out;               // grad_W_s at the chunk's first column
  int64_t ldo;             // elements from vocabulary row to row ([V][H]) or from hidden row to row ([H][V])
  int width, H_s;
  int n_vt, n_ht;          // tiles
  uint32_t lda, ldb;       // as in StripItem
  int b_blocks;
  int stream;              // few tokens, bf16 heads [V][H], written: the output is stored past the last-level cache
  const int* meta;
};

// 256 vocabulary columns (LDS) x 64 NB hidden rows (16 NB per wave)
template <int NB>
struct GradWWork {
  typedef StripShape<16, NB> C;
  const GradWArgs& a;
  int L, G, k;
  __device__ GradWWork(const GradWArgs& a_) : a(a_) {
    G = gridDim.x;
    L = xcd_logical_id(blockIdx.x, G);
    k = meta_get(a.meta, META_T_EFF);
  }
  __device__ int n_items() const { const int n = a.n_vt * a.n_ht; return L < n ? (n - L + G - 1) / G : 0; }
  __device__ StripItem item(int i) const {
    int vt, ht;
    const auto p = kernel_args<GradWArgs>();
    group_decode(i * G + L, p->n_ht, p->n_vt, ht, vt);
    StripItem it;
    it.m0 = vt * C::BM;
    it.n0 = ht * C::BN;
    it.A0 = it.A1 = p->dz + (int64_t)it.m0 * 128;     // (of the first panel)
    it.B0 = it.B1 = p->hT;
    it.lda0 = it.lda1 = p->lda;
    it.ldb0 = it.ldb1 = p->ldb;
    it.b_blocks = p->b_blocks;
    it.k0 = it.k1 = k;
    it.a_rows = it.out_rows = C::BM;                 // (the buffer holds whole tiles: its width is a multiple of 256)
    it.aux = 0;
    return it;
  }
};

// HV: the output is [H][V], the accumulator's rows are vocabulary columns; else [V][H], and its rows are hidden rows.
// ADD: to what is there, with one rounding behind the whole sum.
template <int NB, bool HV, bool F32, bool ADD>
struct GradWEpi {
  static constexpr bool WHOLE = true;
  static constexpr int MB = 16, ES = F32 ? 4 : 2;
  static constexpr bool PAIRS = HV && !F32 && !ADD, QUADS = !HV && !F32 && !ADD && NB == 4;   // 16-byte stores of bf16, by exchanges between lanes
  static constexpr int STORES = PAIRS || QUADS ? MB * NB / 2 : ADD ? 2 * MB * NB : MB * NB;
  const GradWArgs& a;
  int lane, wave;
  __device__ GradWEpi(const GradWArgs& a_) : a(a_), lane(threadIdx.x & 63), wave(uniform(threadIdx.x >> 6)) {}
  __device__ void begin_item(const StripItem&) {}
  // The buffer of blocks j ([H][V]: 16 hidden rows) or of the tile ([V][H]: its columns' rows).
  __device__ __forceinline__ rsrc_t buffer(const StripItem& it, int j) const {
    const int h = it.n0 + 16 * NB * wave + (HV ? 16 * j : 0);
    const int64_t at = HV ? (int64_t)h * a.ldo + it.m0 : (int64_t)it.m0 * a.ldo + h;
    const int rows = HV ? min(16, a.H_s - h) : min(256, a.width - it.m0);
    // (rows - 1 whole ones and the rest of the last: the columns are checked by place())
    const int64_t bytes = ((rows - 1) * a.ldo + (HV ? a.width - it.m0 : a.H_s - h)) * ES;
    return make_rsrc((char*)a.out + at * ES, rows > 0 && bytes > 0 ? (uint32_t)bytes : 0u);
  }
  // offset of four results of block (i, j) in it
  __device__ __forceinline__ uint32_t place(const StripItem& it, int ln, int i, int j) const {
    const int g = ln >> 4, n = ln & 15;
    if (HV) {
      const int v = dz_column(i, 4 * g);
      return it.m0 + v < a.width ? ((uint32_t)n * (uint32_t)a.ldo + v) * ES : NOWHERE;
    }
    const int h = 16 * j + 4 * g;
    return it.n0 + 16 * NB * wave + h < a.H_s ? ((uint32_t)dz_column(i, n) * (uint32_t)a.ldo + h) * ES : NOWHERE;
  }
  // QUADS: blocks (i, 0 .. 3); PAIRS: blocks (i, j), (i + 1, j), whose pieces change places between the halves of the wave (eight
  // neighbouring columns per lane)
  template <int CACHE = 0>
  __device__ __forceinline__ void store_quad(const rsrc_t& r, const StripItem& it, int ln, int i, const f32x4 (&t)[4]) const {
    const int g = ln >> 4, n = ln & 15;
    uint32_t x[4][2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const u32x2 w = pack4(t[j]);
      x[j][0] = w[0]; x[j][1] = w[1];
    }
    quad_transpose(x);
    // A lane now has 32 bytes of one row.  Lanes n and n + 8 trade halves, so that a store writes eight rows' 128 bytes whole (a step of
    // T = 512, H = 1024 / 2048, V = 128256 1315 -> 1303 us, T = 1024, H = 1024 / 4096 4650 -> 4635, T = 4096, H = 4096 / 1024 the same).
    const bool up = n >= 8;
    u32x4 low, high;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint32_t x0 = x[k >> 1][k & 1], x1 = x[2 + (k >> 1)][k & 1];
      const uint32_t got = __builtin_amdgcn_mov_dpp(up ? x0 : x1, 0x128, 0xf, 0xf, false);      // (row_ror:8)
      low[k] = up ? got : x0;
      high[k] = up ? x1 : got;
    }
    const int h = 16 * g + 8 * up;
    const bool ok = it.n0 + 16 * NB * wave + h < a.H_s;
    const uint32_t at = ((uint32_t)dz_column(i, n & 7) * (uint32_t)a.ldo + h) * ES, below = 4 * (uint32_t)a.ldo * ES;
    __builtin_amdgcn_raw_buffer_store_b128(low, r, ok ? at : NOWHERE, 0, CACHE);
    __builtin_amdgcn_raw_buffer_store_b128(high, r, ok ? at + below : NOWHERE, 0, CACHE);
  }
  __device__ __forceinline__ void store_pair(const rsrc_t& r, const StripItem& it, int ln, int i, const f32x4& t0, const f32x4& t1) const {
    const int g = ln >> 4, n = ln & 15;
    const u32x2 x = pack4(t0), y = pack4(t1);
    auto r0 = __builtin_amdgcn_permlane32_swap(x[0], y[0], false, false);
    auto r1 = __builtin_amdgcn_permlane32_swap(x[1], y[1], false, false);
    const int v = 16 * i + 16 * (g & 1) + 8 * (g >> 1);
    const uint32_t at = it.m0 + v < a.width ? ((uint32_t)n * (uint32_t)a.ldo + v) * ES : NOWHERE;
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{r0[0], r1[0], r0[1], r1[1]}, r, at, 0, 0);
  }
  __device__ __forceinline__ void start(const StripItem&, f32x4 (&T)[MB * NB]) const {
#pragma unroll
    for (int i = 0; i < MB * NB; ++i) T[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  __device__ __forceinline__ void tile(const StripItem& it, f32x4 (&T)[MB * NB]) const {
    const int ln = fresh(lane);
    if constexpr (ADD) {
      // four blocks at a time, the loads of the next four in flight
      f32x4 old[2][4];
      auto block = [](int q, int e) { const int i = HV ? 4 * (q % (MB / 4)) + e : 4 * (q / NB) + e; return MB * (HV ? q / (MB / 4) : q % NB) + i; };
      auto load = [&](auto qc) {
        constexpr int q = decltype(qc)::value;
        const rsrc_t r = buffer(it, block(q, 0) / MB);
#pragma unroll
        for (int e = 0; e < 4; ++e) old[q & 1][e] = load4<F32>(r, place(it, ln, block(q, e) % MB, block(q, e) / MB));
      };
      load(IntC<0>{});
      static_for<0, MB * NB / 4>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        if constexpr (q + 1 < MB * NB / 4) load(IntC<q + 1>{});
        const rsrc_t r = buffer(it, block(q, 0) / MB);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          store4<F32>(r, place(it, ln, block(q, e) % MB, block(q, e) / MB), T[block(q, e)] + old[q & 1][e]);
        __builtin_amdgcn_sched_barrier(0);
      });
    } else if constexpr (HV) {
      static_for<0, NB>([&](auto jc) {
        constexpr int j = decltype(jc)::value;
        const rsrc_t r = buffer(it, j);
        if constexpr (PAIRS) {
          static_for<0, MB / 2>([&](auto ic) {
            constexpr int i = 2 * decltype(ic)::value;
            store_pair(r, it, ln, i, T[MB * j + i], T[MB * j + i + 1]);
          });
        } else {
          static_for<0, MB>([&](auto ic) { store4<F32>(r, place(it, ln, decltype(ic)::value, j), T[MB * j + decltype(ic)::value]); });
        }
      });
    } else {
      const rsrc_t r = buffer(it, 0);
      static_for<0, MB>([&](auto ic) {
        constexpr int i = decltype(ic)::value;
        if constexpr (QUADS) {
          const f32x4 t[4] = {T[i], T[MB * (1 % NB) + i], T[MB * (2 % NB) + i], T[MB * (3 % NB) + i]};
          store_quad(r, it, ln, i, t);
        } else {
          static_for<0, NB>([&](auto jc) { store4<F32>(r, place(it, ln, i, decltype(jc)::value), T[MB * decltype(jc)::value + i]); });
        }
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  }
};

template <int NB, bool HV, bool F32, bool ADD>
KD_STRIP_KERNEL void grad_w_kernel(const GradWArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  GradWWork<NB> work(a);
  GradWEpi<NB, HV, F32, ADD> epi(a);
  strip_loop<1, false, StripShape<16, NB>, A_DZ, true, !HV>(work, epi, smem);
}

// Few tokens (one token tile): the contraction is at most 256 long and the output, V x H_s, is what takes the time, so the tile of the
// strip loop, four k-steps and then 128 KiB to store, has nothing in flight for most of it: T = 256, H_s = 1024, V = 151936 160 us.  Here a wave keeps its 64 hidden rows of all the tokens in registers for good (128 of them),
// and 32 columns of dz at a time go through the LDS, three such steps ahead; two workgroups per CU, so that the stores of one are
// in flight under the other's products: 110 us; T = 100, H_s = 256, V = 8000 12 -> 6.  (Reading and writing take 75 at the rate of a large
// copy; the stores alone measure 49, the loads alone 27, loads and products 62: the products' LDS reads, by all four waves, are next.)
// Panels of 64 tokens without a valid one are left out.  A large output in bf16, [V][H], is stored past the last-level cache: grad_h_s
// behind it 108 -> 92 us.  (The other forms are not: one that is added to has just been read, fp32 and [H][V] have not been tried.)
struct GradWFew {
  static constexpr int AHEAD = 3, NST = AHEAD + 1, PANELS = 4;
  static constexpr int STAGE_BYTES = PANELS * 4096, SMEM_BYTES = NST * STAGE_BYTES;
  static constexpr int SLOTS = 2 * kNumCU;           // workgroups that run at a time
};
// The fragments of 64 tokens (two sub-steps) x 32 columns: two transposing reads each, landed when this returns.
template <int AT>
__device__ __forceinline__ void few_read(s16x4 (&f)[2][2][2], uint32_t at0, uint32_t at1) {
  asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%10\n\tds_read_b64_tr_b16 %1, %9 offset:%10\n\t"
               "ds_read_b64_tr_b16 %2, %8 offset:%11\n\tds_read_b64_tr_b16 %3, %9 offset:%11\n\t"
               "ds_read_b64_tr_b16 %4, %8 offset:%12\n\tds_read_b64_tr_b16 %5, %9 offset:%12\n\t"
               "ds_read_b64_tr_b16 %6, %8 offset:%13\n\tds_read_b64_tr_b16 %7, %9 offset:%13\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(f[0][0][0]), "=&v"(f[0][0][1]), "=&v"(f[0][1][0]), "=&v"(f[0][1][1]), "=&v"(f[1][0][0]), "=&v"(f[1][0][1]),
                 "=&v"(f[1][1][0]), "=&v"(f[1][1][1])
               : "v"(at0), "v"(at1), "n"(AT), "n"(AT + 512), "n"(AT + 2048), "n"(AT + 2560));
}
template <bool HV, bool F32, bool ADD>
__global__ __launch_bounds__(256, 2) void grad_w_few_kernel(const GradWArgs a) {
  typedef GradWFew F;
  typedef GradWEpi<4, HV, F32, ADD> Epi;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
  // workgroup: 256 hidden rows x a range of the chunk's 32-column steps; those of one range side by side on an XCD
  const int L = xcd_logical_id(blockIdx.x, gridDim.x), range = L / a.n_ht, n_steps = (a.width + 31) / 32;
  const int first = (int)((int64_t)range * n_steps / a.n_vt), cnt = (int)((int64_t)(range + 1) * n_steps / a.n_vt) - first;
  const int panels = min(max((meta_get(a.meta, META_N_VALID) + 63) / 64, 1), F::PANELS);
  StripItem it{};
  it.n0 = (L - range * a.n_ht) * 256;
  const Epi epi(a);

  // vector memory operations a step: the loads of a step, and what its results take
  constexpr int STORES = ADD ? 16 : Epi::PAIRS || Epi::QUADS ? 4 : 8;
  const rsrc_t ra = make_rsrc(a.dz, F::PANELS * a.lda);
  uint32_t voff[F::PANELS];
#pragma unroll
  for (int p = 0; p < F::PANELS; ++p)          // (a token's chunks change places on the way, as in A_DZ of strip_loop)
    voff[p] = p < panels ? p * a.lda + wave * 1024 + (lane >> 4) * 256 + ((lane & 15) ^ (4 * ((lane >> 4) & 1))) * 16 : NOWHERE;
  auto issue = [&](int step) {                 // (past the end: the last step again, into a stage that nobody reads)
    const int from = (first + min(step, cnt - 1)) * 4096;
    char* const to = smem + (step % F::NST) * F::STAGE_BYTES + wave * 1024;
#pragma unroll
    for (int p = 0; p < F::PANELS; ++p) __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_void_t*)(to + p * 4096), 16, voff[p], from, 0, 0);
  };
  // h_s of the wave's rows: [block of 16][sub-step of 32 tokens]; blocks that do not exist are 0
  const rsrc_t rb = make_rsrc(a.hT, (uint32_t)a.b_blocks * a.ldb);
  bf16x8 B[4][2 * F::PANELS];
#pragma unroll
  for (int j = 0; j < 4; ++j)
#pragma unroll
    for (int s = 0; s < 2 * F::PANELS; ++s)
      B[j][s] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rb, (uint32_t)(it.n0 / 16 + 4 * wave + j) * a.ldb + s * 1024 + lane * 16, 0, 0));
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int s = 0; s < F::AHEAD; ++s) issue(s);

  const int g = lane >> 4, c = lane & 3, t = 8 * (g & 1) + ((lane & 15) >> 2);
  uint32_t fk[2];
#pragma unroll
  for (int h = 0; h < 2; ++h)
    fk[h] = (uint32_t)(uintptr_t)(lds_void_t*)smem + (g >> 1) * 1024 + (c >> 1) * 256 + ((t + 4 * h) ^ (4 * (c >> 1))) * 16 + (c & 1) * 8;
  for (int step = 0; step < cnt; ++step) {
    // The step has landed for every wave, and every wave has read the one before, whose stage is refilled.  Since its loads were issued
    // AHEAD steps ago there have been those of AHEAD - 1 more and, past the first steps, AHEAD times the results.
    if (step < F::AHEAD) asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(F::PANELS * (F::AHEAD - 1)) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(F::PANELS * (F::AHEAD - 1) + F::AHEAD * STORES) : "memory");
    issue(step + F::AHEAD);
    f32x4 T[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) T[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const uint32_t stage = (uint32_t)(step % F::NST) * F::STAGE_BYTES;
    static_for<0, F::PANELS>([&](auto pc) {
      constexpr int p = decltype(pc)::value;
      if (p < panels) {
        s16x4 f[2][2][2];                      // [sub-step][block of 16 columns][half]
        few_read<4096 * p>(f, fk[0] + stage, fk[1] + stage);
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const bf16x8 x = __builtin_bit_cast(bf16x8, __builtin_shufflevector(f[s][i][0], f[s][i][1], 0, 1, 2, 3, 4, 5, 6, 7));
#pragma unroll
            for (int j = 0; j < 4; ++j)
              T[i][j] = HV ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(x, B[j][2 * p + s], T[i][j], 0, 0, 0)
                           : __builtin_amdgcn_mfma_f32_16x16x32_bf16(B[j][2 * p + s], x, T[i][j], 0, 0, 0);
          }
      }
    });
    it.m0 = (first + step) * 32;
    if constexpr (ADD) {
      f32x4 old[2][4];
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) old[i][j] = load4<F32>(epi.buffer(it, j), epi.place(it, lane, i, j));
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) store4<F32>(epi.buffer(it, j), epi.place(it, lane, i, j), T[i][j] + old[i][j]);
    } else if constexpr (Epi::QUADS) {
      const rsrc_t r = epi.buffer(it, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if (a.stream) epi.template store_quad<STREAM>(r, it, lane, i, T[i]);
        else epi.store_quad(r, it, lane, i, T[i]);
      }
    } else if constexpr (Epi::PAIRS) {
#pragma unroll
      for (int j = 0; j < 4; ++j) epi.store_pair(epi.buffer(it, j), it, lane, 0, T[0][j], T[1][j]);
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) store4<F32>(epi.buffer(it, j), epi.place(it, lane, i, j), T[i][j]);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the loads issued past the end still target this workgroup's LDS
}

// ------------------------------------------------------------------------------------------
// grad_h_s
// ------------------------------------------------------------------------------------------
struct GradHArgs {
  const char* dz;
  const char* W;           // the student's head at the chunk's first column
  float* out;              // part s at out + s * part_stride
  int64_t part_stride;
  int width, H_s;
  int n_ht, n_split, ksteps;   // hidden tiles; parts of ksteps k-steps of 64 columns
  int accumulate;
  uint32_t lda, ldb;
  const int* meta;
};

// 16 MB hidden rows (LDS) x 256 tokens; HV: the head is [H][V]
template <int MB, bool HV>
struct GradHWork {
  typedef StripShape<MB, 4> C;
  const GradHArgs& a;
  int L, G, n_tt;
  __device__ GradHWork(const GradHArgs& a_) : a(a_) {
    G = gridDim.x;
    L = xcd_logical_id(blockIdx.x, G);
    n_tt = meta_get(a.meta, META_N_TT);
  }
  __device__ int n_items() const { const int n = a.n_ht * n_tt * a.n_split; return L < n ? (n - L + G - 1) / G : 0; }
  __device__ StripItem item(int i) const {
    const auto p = kernel_args<GradHArgs>();
    const int q = i * G + L, per = p->n_ht * n_tt, part = q / per;
    int ht, tt;
    group_decode(q - part * per, p->n_ht, n_tt, ht, tt);
    const int k0 = part * p->ksteps * 64;
    StripItem it;
    it.m0 = ht * C::BM;
    it.n0 = tt * 256;
    it.lda0 = it.lda1 = p->lda;
    it.ldb0 = it.ldb1 = p->ldb;
    it.A0 = it.A1 = HV ? p->W + (int64_t)it.m0 * it.lda1 + k0 * 2 : p->W + (int64_t)k0 * it.lda1 + it.m0 * 2;
    it.B0 = it.B1 = p->dz + (int64_t)(it.n0 >> 6) * it.ldb1 + (int64_t)k0 * 128;
    it.k0 = it.k1 = min(p->ksteps * 64, p->width - k0);
    it.a_rows = it.out_rows = min(C::BM, p->H_s - it.m0);
    it.b_blocks = 0;
    it.aux = part;
    return it;
  }
};

template <int MB>
struct GradHEpi {
  static constexpr bool WHOLE = true;
  static constexpr int STORES = 4 * MB;
  const GradHArgs& a;
  int lane, wave, n_valid;
  __device__ GradHEpi(const GradHArgs& a_) : a(a_), lane(threadIdx.x & 63), wave(threadIdx.x >> 6), n_valid(meta_get(a_.meta, META_N_VALID)) {}
  __device__ void begin_item(const StripItem&) {}
  // the tile's valid tokens of its part
  __device__ __forceinline__ rsrc_t buffer(const StripItem& it, bool exists) const {
    const int rows = exists ? max(min(n_valid - it.n0, 256), 0) : 0;
    return make_rsrc(a.out + (int64_t)it.aux * a.part_stride + (int64_t)it.n0 * a.H_s, (uint32_t)rows * (uint32_t)a.H_s * 4u);
  }
  __device__ __forceinline__ uint32_t place(const StripItem& it, int ln, int i, int j) const {
    const int h = 16 * i + 4 * (ln >> 4);
    return h < it.a_rows ? ((uint32_t)(64 * wave + 16 * j + (ln & 15)) * (uint32_t)a.H_s + it.m0 + h) * 4u : NOWHERE;
  }
  __device__ __forceinline__ void start(const StripItem& it, f32x4 (&T)[MB * 4]) const {
    const rsrc_t r = buffer(it, a.accumulate);
    const int ln = fresh(lane);
    static_for<0, 4 * MB>([&](auto nc) {
      constexpr int n = decltype(nc)::value;
      T[n] = load4<true>(r, place(it, ln, n % MB, n / MB));
      if constexpr (n % 16 == 15) __builtin_amdgcn_sched_barrier(0);
    });
  }
  __device__ __forceinline__ void tile(const StripItem& it, f32x4 (&T)[MB * 4]) const {
    const rsrc_t r = buffer(it, true);
    const int ln = fresh(lane);
    static_for<0, 4 * MB>([&](auto nc) {
      constexpr int n = decltype(nc)::value;
      store4<true>(r, place(it, ln, n % MB, n / MB), T[n]);
      if constexpr (n % 16 == 15) __builtin_amdgcn_sched_barrier(0);
    });
  }
};

template <int MB, bool HV>
KD_STRIP_KERNEL void grad_h_kernel(const GradHArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  GradHWork<MB, HV> work(a);
  GradHEpi<MB> epi(a);
  strip_loop<1, false, StripShape<MB, 4>, HV ? A_ROWS_DZ : A_KMAJOR_DZ>(work, epi, smem);
}

// ------------------------------------------------------------------------------------------
// before and behind them
// ------------------------------------------------------------------------------------------

// grad_h_s row t = sum over split-K parts of the fp32 partial sums of its compacted row (zero for a
// masked token), converted to the output dtype.
__global__ void gradh_finish_kernel(const float* parts, int n_parts, int T, int H, const int* inv,
                                    int out_f32, void* out) {
  const int64_t i = (flat_group() * blockDim.x + threadIdx.x) * 4;
  const int64_t n = (int64_t)T * H;
  if (i >= n) return;
  const int t = (int)(i / H), h = (int)(i % H);
  const int j = inv[t];
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (j >= 0) {
    const float* src = parts + (int64_t)j * H + h;
    v = *(const f32x4*)src;
#pragma unroll 8
    for (int p = 1; p < n_parts; ++p) v += *(const f32x4*)(src + (int64_t)p * n);
  }
  if (out_f32) {
    *(f32x4*)((float*)out + i) = v;
  } else {
    *(bf16x4*)((bf16_t*)out + i) = to_bf16(v);
  }
}

// ------------------------------------------------------------------------------------------
// launchers
// ------------------------------------------------------------------------------------------
hipError_t launch_grad_W(const Problem& p, int v0, int width, hipStream_t st) {
  const int nb = grad_W_tile(p.H_s, width, p.n_cu) / 64;
  GradWArgs a{};
  a.dz = (const char*)p.dz; a.hT = (const char*)p.h_sT;
  a.width = width; a.H_s = p.H_s;
  a.n_vt = (width + 255) / 256; a.n_ht = (p.H_s + 64 * nb - 1) / (64 * nb);
  a.ldo = p.w_hv ? p.V : p.H_s;
  a.out = (char*)p.grad_W_s + (size_t)v0 * (p.w_hv ? 1 : p.H_s) * (p.grad_f32 ? 4 : 2);
  a.lda = (uint32_t)p.V_c * 128; a.ldb = (uint32_t)p.T_pad * 32;
  a.b_blocks = (p.H_s + 15) / 16;
  a.meta = p.meta;
  if (p.n_tt == 1) {
    const int steps = (width + 31) / 32;
    a.n_ht = (p.H_s + 255) / 256;
    a.n_vt = GradWFew::SLOTS / a.n_ht < 1 ? 1 : GradWFew::SLOTS / a.n_ht;
    if (a.n_vt > steps) a.n_vt = steps;
    // (more than 128 MiB: half of the cache, which keeps dz and W_s for grad_h_s instead)
    a.stream = !p.w_hv && !p.grad_f32 && !p.accumulate_grad_W && (int64_t)width * p.H_s * 2 > (128 << 20);
#define KD_GF(HV, F32, ADD) launch_big<grad_w_few_kernel<HV, F32, ADD>>(a.n_vt * a.n_ht, 256, GradWFew::SMEM_BYTES, st, &a)
    if (p.accumulate_grad_W)
      return p.w_hv ? (p.grad_f32 ? KD_GF(true, true, true) : KD_GF(true, false, true))
                    : (p.grad_f32 ? KD_GF(false, true, true) : KD_GF(false, false, true));
    return p.w_hv ? (p.grad_f32 ? KD_GF(true, true, false) : KD_GF(true, false, false))
                  : (p.grad_f32 ? KD_GF(false, true, false) : KD_GF(false, false, false));
#undef KD_GF
  }
  const int tiles = a.n_vt * a.n_ht, grid = tiles < p.n_cu ? tiles : p.n_cu;
#define KD_GW3(N, HV, F32) (p.accumulate_grad_W ? launch_big<grad_w_kernel<N, HV, F32, true>>(grid, 256, StripShape<16, N>::SMEM_BYTES, st, &a) \
                                               : launch_big<grad_w_kernel<N, HV, F32, false>>(grid, 256, StripShape<16, N>::SMEM_BYTES, st, &a))
#define KD_GW(N) (p.w_hv ? (p.grad_f32 ? KD_GW3(N, true, true) : KD_GW3(N, true, false)) \
                         : (p.grad_f32 ? KD_GW3(N, false, true) : KD_GW3(N, false, false)))
  switch (nb) {
    case 2: return KD_GW(2);
    case 3: return KD_GW(3);
    default: return KD_GW(4);
  }
#undef KD_GW3
#undef KD_GW
}

hipError_t launch_grad_h(const Problem& p, int v0, int width, bool first, hipStream_t st) {
  const int mb = p.gh_rows / 16;
  GradHArgs a{};
  a.dz = (const char*)p.dz;
  const int64_t ld = p.w_hv_inplace ? p.V : p.prep_Ws ? p.K_s : p.H_s;
  a.W = (const char*)p.W_s + (size_t)v0 * 2 * (p.w_hv_inplace ? 1 : ld);
  a.out = p.gh32; a.part_stride = (int64_t)p.T * p.H_s;
  a.width = width; a.H_s = p.H_s;
  a.n_ht = (p.H_s + 16 * mb - 1) / (16 * mb);
  a.ksteps = p.ksteps_h;
  a.n_split = ((width + 63) / 64 + a.ksteps - 1) / a.ksteps;       // every part has at least one k-step
  a.accumulate = first ? 0 : 1;
  a.lda = 2u * (uint32_t)ld;
  a.ldb = (uint32_t)p.V_c * 128;
  a.meta = p.meta;
  const int tiles = a.n_ht * p.n_tt * a.n_split, grid = tiles < p.n_cu ? tiles : p.n_cu;   // worst case: no token masked
#define KD_GH(N) (p.w_hv_inplace ? launch_big<grad_h_kernel<N, true>>(grid, 256, StripShape<N, 4>::SMEM_BYTES, st, &a) \
                                 : launch_big<grad_h_kernel<N, false>>(grid, 256, StripShape<N, 4>::SMEM_BYTES, st, &a))
  switch (mb) {
    case 4: return KD_GH(4);
    case 8: return KD_GH(8);
    case 12: return KD_GH(12);
    default: return KD_GH(16);
  }
#undef KD_GH
}

hipError_t launch_gradh_finish(const Problem& p, hipStream_t st) {
  const int64_t n = (int64_t)p.T * p.H_s;
  const FlatGrid g = flat_grid(((n + 3) / 4 + 255) / 256);
  hipLaunchKernelGGL(gradh_finish_kernel, dim3(g.x, g.y), dim3(256), 0, st, p.gh32,
                     p.n_ksplit_h, p.T, p.H_s, p.inv, p.grad_f32, p.grad_h_s);
  return hipGetLastError();
}

}  // namespace kd
