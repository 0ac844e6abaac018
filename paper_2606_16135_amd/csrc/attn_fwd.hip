// Causal GQA prefill attention over prefix + new tokens (§2.2: causal
// attention over every earlier position and the token itself; a new turn's tokens attend to the
// cached history plus the new tokens; GQA as used by the models of §5).
//
// Output row (query i of a sequence with P cached tokens, query head h):
//   o = sum_{j <= P + i} softmax_j(scale * q . k_j) v_j,  KV head g = h / group.
//
// Work decomposition (built on the host, see plan_attention): a workgroup
// of 8 waves owns 256 (query, head) rows = rows_q consecutive queries times
// the `group` query heads that share one KV head, and a range of keys.
// Packing the heads of a group into the rows makes every K/V tile staged
// through LDS serve all of them.  Long key ranges are split over several
// workgroups (split-key): each writes a normalised partial output (in the
// element type; it is a convex combination of V rows) and
// its log-sum-exp, and attn_merge_kernel combines them exactly
// (o = sum_s exp(lse_s - lse) o_s).  The merge is not done by the
// last-arriving split's workgroup: that would need device-scope fences,
// whose L2 write-back / invalidate stalls the other workgroups streaming
// K/V.  A single call launches the merge kernel after the forward kernel;
// in a layer stack the forward kernel of the next layer does it, each
// workgroup claiming chunks of rows once its own item is done (the launch
// boundary orders the partials' writes before those reads).
//
// q, K, V and out are bf16 or IEEE fp16 (Elem<DT> below); everything else
// is the same for both types.
//
// Per key tile of 32 and per wave (32 rows):
//   S^T (32 keys x 32 rows) = K_tile . Q^T         MFMA 32x32x16 bf16, fp32 out
//   P = exp2(c S^T - m),  c = scale * log2(e)      online softmax, log2 domain
//   O^T (D x 32 rows) += V^T . P^T                 MFMA 32x32x16 bf16
// The scale stays in fp32: folding it into a bf16 copy of q moves scores by
// about 1% of q's rounding, enough to exceed the tolerance when two keys
// compete for a row.  Every lane holds 16 keys of ONE row (the other 16 are
// in the other half of the wave).  The probabilities never leave registers:
// the S^T accumulator layout is the B-operand layout of the PV product once
// rounded to bf16, for a fixed permutation of the 16 keys of each MFMA step.
// V^T operands come from the row-major V tile through LDS transpose reads
// (ds_read_b64_tr_b16: in each 16-lane group, lanes 4r..4r+3 read 4 dims
// each of key r and lane j gets dim j of the 4 keys).  The row sum adds the
// fp32 probabilities before rounding, in two chains (two v_add_f32 per pair
// measured 1-2% faster at head_dim 128 and 2-4% at 64 than one
// v_dot2c_f32_bf16 on the packed pair); it differs from the sum of the
// rounded weights the PV product uses by the rounding of P, far below the
// tolerance.
//
// Software pipeline.  A single wave issues MFMAs at half the SIMD's matrix
// rate and VALU ops at half its vector rate, so each wave interleaves both:
// iteration j issues QK(j+1) and PV(j-1) (16 MFMAs) in the same basic block
// as the softmax of tile j, and both waves of a SIMD do so.  The MFMAs do
// not hide the vector work completely (measured: each vector instruction
// per score costs 2-3% of the loop), so the softmax is cut to its minimum:
// p = exp2(c s - m), the bf16 packing and the row sum.  The reference max m
// is the exact max of the first tile and moves only when a lane's tile sum
// exceeds kSumLimit: softmax is invariant to the reference, and fp32/bf16
// keep their relative precision at any scale, so a stale reference changes
// nothing but the exponent range, which the limit bounds.  No per-tile row
// max is computed on the common path.
//
// K and V tiles (8 KiB: 32 keys at head_dim 128, 64 at 64) each live in a
// 4-entry LDS ring (slot = tile mod 4), and iteration j reads K(j+1) and
// V(j-1).  The tiles go from memory straight into LDS (buffer loads with the
// LDS flag, swizzled rows instead of padded ones, 64 KiB of LDS): the even
// iteration of each pair issues the loads of K(j+3), K(j+4), V(j+1) and
// V(j+2), and the pair ends with one barrier after they have landed.  A tile
// is in place at least a barrier before it is read and only every second
// iteration ends with a workgroup barrier (one that lets global loads meant
// for later iterations stay in flight), which halves the barrier waits and
// lets the waves drift apart by up to an iteration.  The loop is unrolled so
// that the ring slots, the barrier placement and the score registers are
// fixed at compile time.
//
// At head_dim 64 a score carries half the MFMA work and the same vector
// work, so the loop is bound by the latter: per 64-key tile and SIMD about
// 1660 cycles of vector issue (FMA, exponential, add, half a pack per score)
// against 1024 of MFMAs.  The 64-key tile halves the barriers, loads and
// address arithmetic per score; against 32-key tiles staged through
// registers a 32/8-head call of P=8192, N=512 takes 45.2 us instead of 48.0.
#include "sc_internal.h"
#include "sc_lds_load.h"

#include <cmath>
#include <mutex>
#include <type_traits>

namespace sc {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;

// A record of 32-bit fields read through the constant address space: the
// host writes work items and sequence records before the launch and nothing
// writes them during it, so a uniform index gives scalar loads.
template <class T>
__device__ __forceinline__ T load_const(const T *p) {
  static_assert(sizeof(T) % 4 == 0, "32-bit fields");
  const __attribute__((address_space(4))) int32_t *q = (const __attribute__((address_space(4))) int32_t *)p;
  int32_t v[sizeof(T) / 4];
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) v[i] = q[i];
  T r;
  __builtin_memcpy(&r, v, sizeof(T));
  return r;
}

constexpr int kThreads = 512;            // 8 waves, 2 per SIMD
constexpr int KT = kAttnKeyTile;
static_assert(kAttnRows == 8 * 32, "eight waves of 32 rows");
static_assert(KT == 32, "key ranges are cut at MFMA block boundaries");

// 32x32 MFMA accumulator layout: element r of lane l holds C[m][n] with
// n = l % 32 and m = 8 * (r / 4) + 4 * (l / 32) + r % 4.
__device__ __forceinline__ int acc_m(int r, int half) { return 8 * (r >> 2) + 4 * half + (r & 3); }

// One K or V tile: 8 KiB of key rows of one KV head, i.e. 32 keys at
// head_dim 128 and 64 at head_dim 64, so that an iteration of the loop has
// 16 MFMAs and one load into LDS per wave and operand at either head_dim.
template <int D>
struct Tile {
  static constexpr int kRowBytes = D * 2;
  static constexpr int kSlotBytes = 8192;
  static constexpr int kKeys = kSlotBytes / kRowBytes;
  static constexpr int kBlocks = kKeys / 32;               // 32-key MFMA blocks of the S^T product
  static constexpr int kChunksPerRow = kRowBytes / 16;
  static constexpr int kRowsPerLoad = 1024 / kRowBytes;    // key rows of one wave's load (64 lanes x 16 B)
  static_assert(8 * kRowsPerLoad == kKeys, "eight waves load a tile");
  // LDS rows are unpadded; chunk c (16 B) of row r sits at position
  // c ^ swz_k(r) (K) or c ^ swz_v(r) (V).  K fragment reads take one chunk
  // of 16 consecutive rows, V transpose reads 64 bytes of 4 consecutive
  // rows: with these, each covers all 64 banks once (256 bytes = one row at
  // head_dim 128, two at 64).
  static __device__ __forceinline__ int swz_k(int r) { return D == 128 ? (r & 15) : ((r >> 1) & 7); }
  static __device__ __forceinline__ int swz_v(int r) { return D == 128 ? 4 * (r & 3) : 4 * ((r >> 1) & 1); }
};

// Element type of q, K, V, the probabilities of the PV product and the
// output: bf16 or IEEE fp16 (the paper's serving precision, §5).  Operands
// travel as raw 16-bit patterns; only the MFMA, the packing of fp32 values
// (round to nearest even) and the unpacking depend on the type.
template <int DT>
struct Elem;

template <>
struct Elem<SC_DTYPE_BF16> {
  // A lane's tile sum above this sends the wave through settle_max.  Every
  // probability is then below 2^20, so O and l stay far from fp32 overflow
  // for any sequence length; rows never pay for a max they do not need.
  static constexpr float kSumLimit = 1048576.0f;
  static __device__ __forceinline__ f32x16 mfma(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
  }
  // Two floats to packed bf16, one v_cvt_pk_bf16_f32.
  static __device__ __forceinline__ uint32_t pack(float a, float b) {
    const bf16x2 p = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, p);
  }
  // Packed pair back to floats (exact).
  static __device__ __forceinline__ f32x2 unpack(uint32_t p) {
    f32x2 r;
    r[0] = __builtin_bit_cast(float, p << 16);
    r[1] = __builtin_bit_cast(float, p & 0xFFFF0000u);
    return r;
  }
};

template <>
struct Elem<SC_DTYPE_F16> {
  // As for bf16, but fp16 probabilities must also stay below its largest
  // finite value (65504): with a tile sum of at most 2^15 every one does.
  // A probability that overflowed to inf fails the same test.
  static constexpr float kSumLimit = 32768.0f;
  static __device__ __forceinline__ f32x16 mfma(u32x4 a, u32x4 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0,
                                                  0, 0);
  }
  static __device__ __forceinline__ uint32_t pack(float a, float b) {
    const f16x2 p = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, p);
  }
  static __device__ __forceinline__ f32x2 unpack(uint32_t p) {
    const f16x2 h = __builtin_bit_cast(f16x2, p);
    f32x2 r;
    r[0] = (float)h[0];
    r[1] = (float)h[1];
    return r;
  }
};

// Max with the same lane of the other 32-lane half of the wave.
__device__ __forceinline__ float max_with_other_half(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, x),
                                                  __builtin_bit_cast(uint32_t, x), false, false);
  return fmaxf(__builtin_bit_cast(float, (uint32_t)r[0]), __builtin_bit_cast(float, (uint32_t)r[1]));
}

// K/V slots of 8 KiB, loaded straight into LDS (see attn_item).  Kernels
// with narrow items keep them in one array, `ring`.  Ordinary items: slot s of the four K slots at 8 s KiB, of
// the four V slots 32 KiB further.  Narrow items: two stages of four key groups' slots, K at
// 32 stage + 8 group KiB, V 64 KiB further.  A tile's load has one pair of
// iterations to land in (one iteration for narrow items); two or three pairs
// (rings of 6 or 8 slots) measured 1.5-3% slower on the 8B, 14B and
// long-prefix shapes and 3-15% slower on short turns that stream K/V from
// HBM once.
constexpr int kRing = 4;
constexpr int kNarrowGroups = 4;
constexpr int kSlot = Tile<128>::kSlotBytes;
// The slots of kernels without narrow items: one array per slot and operand,
// so the compiler can tell that a load in flight into one does not alias
// reads of another (see load_to_lds).
#define SC_SLOT(n)                                                              \
  __shared__ __attribute__((aligned(1024))) unsigned char slot_k##n[kSlot];     \
  __shared__ __attribute__((aligned(1024))) unsigned char slot_v##n[kSlot];
SC_SLOT(0)
SC_SLOT(1)
SC_SLOT(2)
SC_SLOT(3)
#undef SC_SLOT
// Narrow items: each wave's reference max and row sums (32 rows), for the
// waves that combine them.
__shared__ f32x2 narrow_ml[8][32];

// f(integral_constant<int, i>) for i = B .. E-1, unrolled.
template <int B, int E, class Fn>
__device__ __forceinline__ void static_for(Fn &&f) {
  if constexpr (B < E) {
    f(std::integral_constant<int, B>());
    static_for<B + 1, E>(f);
  }
}

// Wait until at most VM vector-memory operations of this wave (loads into
// LDS included) are in flight and its LDS and scalar loads are done, then a
// workgroup barrier.  No memory-model fence: the fence of __syncthreads
// would wait for every load into LDS, including those meant to stay in
// flight.
template <int VM>
__device__ __forceinline__ void dma_barrier() {
  static_assert(VM >= 0 && VM < 64, "vmcnt field");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((VM & 15) | ((VM >> 4) << 14) | (7 << 4) | (0 << 8));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// The loads into LDS are written out (load_to_lds) in the kernels with narrow
// items, whose slots are one array (narrow items pick theirs at run time):
// around the builtin the compiler would wait for every load in flight before
// any LDS read.  The waits are dma_barrier's.  Kernels without them keep the
// builtin and an array per slot: run by the kernel with narrow items, the same
// plans take 0.5-1.5% longer (32/8 heads, P=131072, N=2048: 3488 us against
// 3541; 40/8, P=32768, N=1020: 572 against 579; 32/8, P=8192, N=512: 68.8
// against 69.4; head_dim 64, P=32768, N=1024: 274.7 against 276.2).
__device__ __forceinline__ uint32_t lds_address(const void *p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void *)p;
}

// Wait for every vector-memory operation of this wave.
__device__ __forceinline__ void dma_wait_all() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0 | (7 << 4) | (15 << 8));
  asm volatile("" ::: "memory");
}

// Masks keys past a row's last visible key: element r of block b holds key
// offset 32 b + acc_m(r, half) within the tile, and lim is the row's last
// visible offset minus 4 half.
template <int NB>
__device__ __forceinline__ void apply_mask(f32x16 (&s)[NB], int lim) {
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r)
      if (32 * b + acc_m(r, 0) > lim) s[b][r] = -INFINITY;
}

// Row max of sl2 * s over the tile's keys (both wave halves); -inf when
// every key of the row is masked.
template <int NB>
__device__ __forceinline__ float tile_max(const f32x16 (&s)[NB], float sl2) {
  float m4[4 * NB];
#pragma unroll
  for (int i = 0; i < 4 * NB; ++i) {
    const f32x16 &x = s[i >> 2];
    const int r = 4 * (i & 3);
    m4[i] = fmaxf(fmaxf(x[r], x[r + 1]), fmaxf(x[r + 2], x[r + 3]));
  }
  float m = m4[0];
#pragma unroll
  for (int i = 1; i < 4 * NB; ++i) m = fmaxf(m, m4[i]);
  return max_with_other_half(m) * sl2;
}

// p = exp2(sl2 * s - m) for this lane's keys, packed to the element type,
// and their fp32 sum (two chains).
template <int DT, int NB>
__device__ __forceinline__ float softmax_tile(const f32x16 (&s)[NB], u32x4 (&pf)[2 * NB], float sl2, float m) {
  float r2[2] = {0.f, 0.f};
#pragma unroll
  for (int t = 0; t < 2 * NB; ++t)
#pragma unroll
    for (int e = 0; e < 8; e += 2) {
      const float x0 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t >> 1][8 * (t & 1) + e], sl2, -m));
      const float x1 = __builtin_amdgcn_exp2f(__builtin_fmaf(s[t >> 1][8 * (t & 1) + e + 1], sl2, -m));
      pf[t][e >> 1] = Elem<DT>::pack(x0, x1);
      r2[0] += x0;
      r2[1] += x1;
    }
  return r2[0] + r2[1];
}

template <int D>
struct WaveState {
  u32x4 qf[D / 16];   // raw 16-bit patterns
  f32x16 oacc[D / 32];
  f32x16 s[2][Tile<D>::kBlocks];       // raw scores of the even / odd tiles
  u32x4 pfb[2][2 * Tile<D>::kBlocks];  // P of the even / odd tiles (no copy per tile)
  float m_run;        // reference max of sl2 * s, log2 units (0 until a key is visible)
  float l_run;        // this lane's share of the denominator
};

// Rare path, taken by a whole wave when some lane's tile sum left the safe
// range: move every row's reference max to the true running max, rescale l
// and O (O already holds PV(j-1), computed against the old reference), and
// redo the tile's exponentials.  Returns the new tile sum.
template <int D, int DT>
__device__ __forceinline__ float settle_max(WaveState<D> &w, const f32x16 (&s)[Tile<D>::kBlocks],
                                            u32x4 (&pf)[2 * Tile<D>::kBlocks], float sl2) {
  const float m_new = fmaxf(w.m_run, tile_max(s, sl2));
  const float corr = __builtin_amdgcn_exp2f(w.m_run - m_new);
  w.m_run = m_new;
  w.l_run *= corr;
#pragma unroll
  for (int c = 0; c < D / 32; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) w.oacc[c][r] *= corr;
  return softmax_tile<DT>(s, pf, sl2, m_new);
}

// Writes this lane's row of O (times inv, rounded to the element type) to
// `dst`.  A lane holds 4 consecutive dims of each 8-dim block, the other 4
// are in the same lane of the other half of the wave; one lane swap per
// dword gives half 0 the even and half 1 the odd 8-dim blocks of each 16,
// so every lane writes whole 16-byte chunks (the two halves of a row fill
// 32 contiguous bytes per store).  v_permlane32_swap exchanges lanes 32-63
// of its first operand with lanes 0-31 of its second.
template <int DT>
__device__ __forceinline__ void store_chunk(const float (&x)[8], float inv, uint16_t *dst) {
  // A: dims 4 half + [0, 4) of 16; B: the same + 8.
  uint32_t A[2], B[2];
  A[0] = Elem<DT>::pack(x[0] * inv, x[1] * inv);
  A[1] = Elem<DT>::pack(x[2] * inv, x[3] * inv);
  B[0] = Elem<DT>::pack(x[4] * inv, x[5] * inv);
  B[1] = Elem<DT>::pack(x[6] * inv, x[7] * inv);
  u32x4 st;
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    // Half 0 receives the other half's A, half 1 the other half's B.
    const auto r = __builtin_amdgcn_permlane32_swap(A[e], B[e], false, false);
    st[e] = (uint32_t)r[0];
    st[2 + e] = (uint32_t)r[1];
  }
  *reinterpret_cast<u32x4 *>(dst) = st;
}

template <int D, int DT>
__device__ __forceinline__ void store_row(const WaveState<D> &w, float inv, int half, uint16_t *dst) {
#pragma unroll
  for (int c = 0; c < D / 32; ++c)
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = w.oacc[c][8 * m + e];
      store_chunk<DT>(x, inv, dst + 32 * c + 16 * m + 8 * half);
    }
}

// One work item.  kPaged: its keys are read in place from the regular
// cache.  KG = 1: the eight waves hold 256 rows.  KG = 4, a narrow item of
// at most 64 rows: two blocks of 32 rows times four key groups.  Wave w
// holds rows 32 (w / 4) .. + 31 and takes the tiles kg + 4 j, kg = w mod 4,
// so that every wave has work, and the groups are combined through LDS at
// the end.  An iteration stages four K and four V tiles and ends with a
// barrier once they have landed: 64 KiB in flight per CU.  An ordinary item
// runs its 256 rows' worth of MFMAs whatever it holds; a narrow one takes a
// third to a quarter of the time per key, plus 1.7 us (3.4 with two row
// blocks) for its start and the combination.  Calls of 32/8 heads, ordinary
// against narrow: P=8192, N=1 16.0 -> 12.3 us, P=32768, N=8 33.5 -> 28.0,
// P=2048, N=8 11.5 -> 9.8, P=256, N=4 9.6 -> 6.6 (one split, no merge);
// layer stack of 40/8 heads in chunks of 256 tokens, whose last query tile
// has 5 rows: 1633 -> 1590 us.  The kinds are separate copies of the whole
// body so that each is register-allocated on its own.
template <int D, int DT, bool kPaged, int KG, bool kNamed>
__device__ __forceinline__ void attn_item(const AttnArgs &a, unsigned char *ring, const WorkItem &wi, const SeqDesc &sd) {
  static_assert(KG == 1 || (KG == kNarrowGroups && !kPaged && !kNamed), "kinds of item");
  using G_ = Tile<D>;
  constexpr int NB = G_::kBlocks;
  constexpr int TK = G_::kKeys;      // keys per tile
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5;
  const int col = lane & 31;
  const int group = a.group;
  const int kg = KG == 1 ? 0 : wave % KG;          // key group
  const int rb = KG == 1 ? wave : wave / KG;       // block of 32 rows
  const int row = rb * 32 + col;
  const int qi = row / group;
  const int hg = row - qi * group;
  const bool valid = qi < wi.nq;
  const int qpos = wi.q0 + (valid ? qi : wi.nq - 1);
  const int h = wi.kvh * group + hg;
  // qrow: the row in the plan's packed numbering (split partials, lse);
  // io_row: the row of q and out (they differ for a chunk of a new turn).
  const int64_t qrow = (int64_t)(sd.cu_q + qpos) * a.n_q_heads + h;
  const int64_t io_row = (int64_t)(sd.q_off + qpos) * a.n_q_heads + h;

  WaveState<D> w;
  const float sl2 = a.scale_log2;   // scale * log2(e)
#pragma unroll
  for (int c = 0; c < D / 32; ++c)
#pragma unroll
    for (int r = 0; r < 16; ++r) w.oacc[c][r] = 0.f;
  w.m_run = 0.f;
  w.l_run = 0.f;

  // This item's keys [k_begin, k_end) of KV head kvh: rows of kv_stride
  // elements, D of them used.  Tile t is read through a buffer resource that
  // starts at its first row and ends after the item's last row, so rows past
  // the range (the ragged last tile, tiles past the end) read as zero
  // without touching memory outside it; those keys are masked.
  const int64_t kv_stride = (int64_t)a.n_kv_heads * D;
  const int k_begin = wi.k_begin;
  const int k_end = wi.k_end;
  const int n = (k_end - k_begin + TK - 1) / TK;
  const int64_t first_row = ((int64_t)sd.cu_k + k_begin) * kv_stride + (int64_t)wi.kvh * D;
  const uint16_t *const kb = a.k + first_row;
  const uint16_t *const vb = a.v + first_row;
  // Byte counts, also of the tiles loaded past the end, fit in 31 bits
  // (checked on the host).
  const uint32_t range_bytes = (uint32_t)((((int64_t)(k_end - k_begin) - 1) * kv_stride + D) * 2);
  const uint32_t tile_bytes = (uint32_t)(TK * kv_stride * 2);
  // First tile that needs the mask, the same for the whole workgroup: it
  // reaches past the key range or past the diagonal of the first query.
  const int diag0 = sd.prefix + wi.q0;
  const int j_mask = max(0, min(n, (min(k_end, diag0 + 1) - k_begin) / TK)) / KG;
  const int n_it = (n + KG - 1) / KG;   // iterations
  const int my_last = min(k_end - 1, sd.prefix + qpos);
  auto lim_of = [&](int j) { return my_last - (k_begin + (j * KG + kg) * TK) - 4 * half; };

  // Device-side dependency on the copy stream (see AttnArgs::ready_flag).
  // The poll is a relaxed device-scope load (no cache invalidation per
  // workgroup: an acquire here would invalidate the XCD's L2 under the
  // other workgroups' K/V).  No stale K/V lines can be cached: this kernel's
  // dispatch invalidated the caches after the last reader of the slot (two
  // layers back, same stream) had finished, the only kernel that touches the
  // slot after that is the copy kernel, whose completion wrote its data back
  // before the flag was written, and nothing reads the slot until the flag
  // is set.  A stack that also writes the slot from another kernel after
  // this dispatch (debug poisoning) asks for the acquire (ready_acquire).
  bool timed_out = false;
  if (a.ready_flag != nullptr) {
    __shared__ int s_timeout;
    if (tid == 0) {
      int spins = 0, late = 0;
      while (__hip_atomic_load(a.ready_flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < a.ready_value) {
        if (++spins > a.ready_spin_limit) {
          late = 1;
          __hip_atomic_store(a.ready_timeout, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(8);
      }
      if (a.ready_acquire && !late) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      s_timeout = late;
    }
    __syncthreads();
    timed_out = s_timeout != 0;
  }

  // K and V tiles go from memory straight into LDS (buffer loads with the
  // LDS flag; no staging registers).  Wave w loads kRowsPerLoad consecutive
  // rows of every K and V tile (narrow: half of its own group's tile, in
  // four loads): one 16-byte load per lane, lane i filling bytes 16 i ..
  // 16 i + 15 of the wave's rows.  Rows are unpadded
  // and swizzled (see Tile), which keeps the K fragment reads and the V
  // transpose reads free of bank conflicts: each lane loads the chunk that
  // belongs at its position.
  const int row_bytes = (int)(kv_stride * 2);
  const int my_row = KG == 1 ? G_::kRowsPerLoad * wave : rb * (TK / 2);
  int voff_k[KG], voff_v;   // KG loads per tile; V's swizzle repeats with them
#pragma unroll
  for (int i = 0; i < KG; ++i) {
    const int r = i * G_::kRowsPerLoad + lane / G_::kChunksPerRow;
    const int c = lane % G_::kChunksPerRow;
    voff_k[i] = r * row_bytes + ((c ^ G_::swz_k(my_row + r)) << 4);
    if (i == 0) voff_v = r * row_bytes + ((c ^ G_::swz_v(my_row + r)) << 4);
  }
  // This lane's LDS read offsets within a slot (of its key group): K
  // fragment k of block 0 (row col, chunk 2 k + half) and the transpose read
  // of dim block c (key row tr_row); the slots, blocks and key rows of the
  // product are immediates, as the swizzles repeat every 16 rows.
  constexpr int kV0 = (KG == 1 ? kRing : 2 * KG) * kSlot;   // first V slot
  int k_rd[D / 16], v_rd[D / 32];
#pragma unroll
  for (int k = 0; k < D / 16; ++k) k_rd[k] = kg * kSlot + col * G_::kRowBytes + (((2 * k + half) ^ G_::swz_k(col)) << 4);
  {
    const int tr_row = 4 * half + ((lane & 15) >> 2);
    const int lo = 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
#pragma unroll
    for (int c = 0; c < D / 32; ++c)
      v_rd[c] = (kNamed ? 0 : kV0) + kg * kSlot + tr_row * G_::kRowBytes +
                (((4 * c + lo) ^ G_::swz_v(tr_row)) << 4) + 8 * (lane & 1);
  }
  // Regular-cache item: key k of the sequence is row k mod B of local
  // block rc_ids[rc_off + k / B], read in place.  A wave's rows start on a
  // multiple of their count (4 or 8) and B >= 16 is a power of two, so they
  // share one block; its index is a scalar load (the table is read through the
  // constant address space: the host writes it before the launch), made a
  // pair of iterations before the tile's data load.
  const __attribute__((address_space(4))) int32_t *rc_ids_c =
      kPaged ? (const __attribute__((address_space(4))) int32_t *)(a.rc_ids + sd.rc_off) : nullptr;
  // This KV head's K and V rows in block 0 of the layer; block b is
  // b * rc_block_bytes further (under 4 GiB, checked on the host), so the
  // per-tile address is a 32 x 32 -> 64-bit product and two adds.
  const char *rc_kbase =
      kPaged ? reinterpret_cast<const char *>(a.rc_base + a.rc_layer_elems + (int64_t)wi.kvh * D) : nullptr;
  const char *rc_vbase = kPaged ? rc_kbase + a.rc_half_elems * 2 : nullptr;
  const uint32_t rc_block_bytes = kPaged ? (uint32_t)(a.rc_block_elems * 2) : 0u;
  const int rc_mask = (1 << a.block_shift) - 1;
  auto blk_of = [&](int t) -> int {
    if constexpr (!kPaged) {
      return 0;
    } else {
      return rc_ids_c[min(k_begin + t * TK + my_row, k_end - 1) >> a.block_shift];
    }
  };
  // K and V slot S (a stage, for narrow items).
  auto k_slot = [&](auto S) -> unsigned char * {
    constexpr int s = decltype(S)::value;
    if constexpr (kNamed)
      return s % kRing == 0 ? slot_k0 : s % kRing == 1 ? slot_k1 : s % kRing == 2 ? slot_k2 : slot_k3;
    else
      return ring + (KG == 1 ? s % kRing : s % 2 * KG) * kSlot;
  };
  auto v_slot = [&](auto S) -> unsigned char * {
    constexpr int s = decltype(S)::value;
    if constexpr (kNamed)
      return s % kRing == 0 ? slot_v0 : s % kRing == 1 ? slot_v1 : s % kRing == 2 ? slot_v2 : slot_v3;
    else
      return ring + (KG == 1 ? s % kRing : s % 2 * KG) * kSlot;   // kV0 further, in v_rd and dma
  };
  const uint32_t my_lds =
      (uint32_t)__builtin_amdgcn_readfirstlane((int)(kg * kSlot + my_row * G_::kRowBytes));   // within a slot
  // This wave's rows of tile t, K (kV false) or V, into `slot`.  The buffer
  // resource ends after the last row of the item's range (of the block, for
  // a regular-cache item), so rows past it, and whole tiles past the last
  // one, load zeros without touching memory.
  auto dma = [&](unsigned char *slot, int t, auto v_tag, int blk) {
    constexpr bool kV = decltype(v_tag)::value;
    const int key = k_begin + t * TK + my_row;
    const char *base;
    int range;
    if constexpr (kPaged) {
      const int rib = min(key, k_end - 1) & rc_mask;   // first row within the block
      const int rows = min(rc_mask + 1 - rib, k_end - key);
      base = (kV ? rc_vbase : rc_kbase) + (uint64_t)(uint32_t)blk * rc_block_bytes + (uint32_t)(rib * row_bytes);
      range = rows > 0 ? ((rows - 1) * row_bytes + 2 * D) : 0;
    } else {
      // Signed 32-bit offsets (the host keeps a sequence's keys, plus the
      // tiles loaded past its end, under 2^31 bytes): a subtract and a max
      // on the scalar unit.  A 64-bit compare would be a vector
      // instruction whose result the scalar select then waits for (~2%
      // of the loop), as would a saturating unsigned subtract.
      // At head_dim 64 and for narrow items the tiles past the end would
      // reach further than that margin: they all load from the first one,
      // past the range as well.
      const int off = (NB == 1 && KG == 1 ? t : min(t, n)) * (int)tile_bytes + my_row * row_bytes;
      base = reinterpret_cast<const char *>(kV ? vb : kb) + off;
      range = max((int)range_bytes - off, 0);
    }
    if constexpr (kNamed) {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<char *>(base), (short)0, __builtin_amdgcn_readfirstlane(range), 0x00020000);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(slot + my_lds), 16,
                                               kV ? voff_v : voff_k[0], 0, 0, 0);
    } else {
      const uint64_t ad = reinterpret_cast<uint64_t>(base);
      const uint64_t from = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(ad >> 32)) << 32 |
                            (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)ad);
      const uint32_t to = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds_address(slot) + my_lds + (kV ? kV0 : 0)));
      int voff[KG];
#pragma unroll
      for (int i = 0; i < KG; ++i) voff[i] = kV ? voff_v + i * G_::kRowsPerLoad * row_bytes : voff_k[i];
      load_to_lds(to, voff, from, (uint32_t)__builtin_amdgcn_readfirstlane(range));
    }
  };
  auto qk = [&](const unsigned char *slot, f32x16 (&s)[NB]) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int k = 0; k < D / 16; ++k)
        s[b] = Elem<DT>::mfma(*reinterpret_cast<const u32x4 *>(slot + k_rd[k] + 32 * b * G_::kRowBytes), w.qf[k],
                              k == 0 ? f32x16{} : s[b]);
  };
  // V^T operand of PV step (t, c): dims 32 c .. 32 c + 31 of keys
  // 16 t + [0, 16); k-slot e of a lane in half `half` holds key
  // 16 t + 4 half + (e < 4 ? e : e + 4), which is accumulator element
  // 8 (t mod 2) + e of S^T block t / 2, i.e. pf[t] element e.
  auto v_operand = [&](const unsigned char *slot, int t, int c) -> u32x4 {
    const unsigned char *p = slot + v_rd[c] + 16 * t * G_::kRowBytes;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)p);
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 8 * G_::kRowBytes));
    u32x4 vw;
    vw[0] = __builtin_bit_cast(u32x2, lo)[0];
    vw[1] = __builtin_bit_cast(u32x2, lo)[1];
    vw[2] = __builtin_bit_cast(u32x2, hi)[0];
    vw[3] = __builtin_bit_cast(u32x2, hi)[1];
    return vw;
  };
  // O^T += V^T . P^T over the tile's first 16 steps keys.
  auto pv = [&](const unsigned char *slot, const u32x4 (&pfp)[2 * NB], auto steps) {
#pragma unroll
    for (int t = 0; t < decltype(steps)::value; ++t)
#pragma unroll
      for (int c = 0; c < D / 32; ++c) w.oacc[c] = Elem<DT>::mfma(v_operand(slot, t, c), pfp[t], w.oacc[c]);
  };

  using T = std::true_type;
  using F = std::false_type;
  if (KG > 1 && rb * 32 >= wi.nq * group && n > 0 && !timed_out) {
    // A narrow item of at most 32 rows leaves the second row block's waves
    // without rows: they load their halves of the tiles and leave the
    // matrix pipe to the others (same barriers as below).
    dma(ring, kg, F(), 0);
    dma(ring + KG * kSlot, KG + kg, F(), 0);
    dma(ring, kg, T(), 0);
    dma(ring + KG * kSlot, KG + kg, T(), 0);
    dma_barrier<3 * KG>();
    dma_barrier<2 * KG>();
    for (int j = 0; j < n_it; ++j) {
      dma(ring + (j & 1) * KG * kSlot, (j + 2) * KG + kg, F(), 0);
      if (j >= 2) dma(ring + (j & 1) * KG * kSlot, j * KG + kg, T(), 0);
      dma_barrier<0>();
    }
  } else if (n > 0 && !timed_out) {
    constexpr int R = KG == 1 ? kRing : 2;
#define SC_IC(x) std::integral_constant<int, (x)>()
    // Regular-cache block indices of the tiles the current pair loads into
    // K (bk0, bk1) and V (bv0, bv1), and of the next pair's K tiles.  The
    // V tiles of a pair are the K tiles of the pair before.
    int bv0 = blk_of(1), bv1 = blk_of(2), bk0 = blk_of(3), bk1 = blk_of(4);
    int bn0 = 0, bn1 = 0;
    // Prologue: K(0), K(1), K(2) and V(0), the operands of the first pair
    // (narrow: K(0), K(1), V(0) and V(1), all that a short range has, so that
    // its loads share one memory latency), and this wave's Q; then QK(0) once
    // K(0) and Q have landed.  The first loads of the loop go into the slot
    // QK(0) reads: a second barrier.  K(0) is the first load
    // issued, before anything that waits for memory, so that its latency and
    // Q's pass together.
    dma(k_slot(SC_IC(0)), kg, F(), blk_of(0));
    __builtin_amdgcn_sched_barrier(0);
    // Q^T fragments (B operand): lane holds Q[row][16 k + 8 half .. + 7].
    // The buffer resource covers the item's query rows; rows of the
    // workgroup past them get an offset outside it and read zeros without a
    // branch (a masked load made every later load wait for Q).
    {
      const __amdgpu_buffer_rsrc_t qr = __builtin_amdgcn_make_buffer_rsrc(
          const_cast<uint16_t *>(a.q + (int64_t)(sd.q_off + wi.q0) * a.n_q_heads * D), (short)0,
          wi.nq * a.n_q_heads * (2 * D), 0x00020000);
      const int qo = valid ? ((qi * a.n_q_heads + h) * D + 8 * half) * 2 : (int)0x80000000u;
#pragma unroll
      for (int k = 0; k < D / 16; ++k)
        w.qf[k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(qr, qo + 32 * k, 0, 0));
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (KG == 1) {
      dma(k_slot(SC_IC(1)), 1, F(), blk_of(1));
      dma(k_slot(SC_IC(2)), 2, F(), blk_of(2));
      dma(v_slot(SC_IC(0)), 0, T(), blk_of(0));
      dma_barrier<3>();
    } else {
      dma(k_slot(SC_IC(1)), KG + kg, F(), 0);
      dma(v_slot(SC_IC(0)), kg, T(), 0);
      dma(v_slot(SC_IC(1)), KG + kg, T(), 0);
      dma_barrier<3 * KG>();
    }
    qk(k_slot(SC_IC(0)), w.s[0]);
    dma_barrier<KG == 1 ? 0 : 2 * KG>();

    // Iteration j (J = j mod R is the ring slot of tile j; tile j's scores
    // live in s[j mod 2]).  Pair p = iterations 2p, 2p+1 reads K(2p+1),
    // K(2p+2), V(2p-1), V(2p).  Its even iteration loads the operands of
    // pair p+1: K(j+3), K(j+4), V(j+1), V(j+2), into the slots last read in
    // pair p-1; its odd iteration ends with a barrier once they have landed,
    // so only every second iteration waits at a barrier.  A narrow item's
    // iteration j (its j-th tile) loads K(j+2) and, from j = 2 on, V(j) into
    // the stage last read in iteration j-1 and ends with that barrier itself.  Loads of
    // tiles past the last one load zeros.  QK(j+1) runs in every iteration,
    // also the last, whose product of a stale slot is never used: one body
    // throughout keeps the MFMA accumulators in place.
    auto iterate = [&](auto j_tag, auto mask_tag, auto first_tag, int j) {
      constexpr int J = decltype(j_tag)::value;
      constexpr bool kMask = decltype(mask_tag)::value;
      constexpr bool kFirst = decltype(first_tag)::value;
      constexpr int PAR = J & 1;
      const bool late_v = KG > 1 && !kFirst && j >= 2;   // narrow: the prologue loaded V(0) and V(1)
      f32x16 (&sc)[NB] = w.s[PAR];
      f32x16 (&sn)[NB] = w.s[PAR ^ 1];
      if constexpr (kMask) apply_mask(sc, lim_of(j));
      if constexpr (kFirst) {
        const float tm = tile_max(sc, sl2);
        w.m_run = tm > -INFINITY ? tm : 0.f;
      }
      const float mneg = -w.m_run;
      const unsigned char *ks = k_slot(SC_IC(J + 1));
      const unsigned char *vs = v_slot(SC_IC(J + R - 1));
      // The 16 MFMAs of the iteration alternate between QK(j+1) (even
      // steps; block b varies fastest, so no two successive ones depend on
      // each other at head_dim 64) and PV(j-1) (odd steps, V^T block c of
      // 16-key group t), and each step also computes a sixteenth of tile j's
      // softmax (one probability at head_dim 128, two at 64), in this order
      // (scheduling barriers keep the compiler from regrouping them).
      // Operands are read from LDS three steps ahead (two measured ~0.5%
      // slower, four no better).
      constexpr int NC = D / 32;
      auto operand = [&](int i) -> u32x4 {
        const int h = i >> 1;
        if ((i & 1) == 0)
          return *reinterpret_cast<const u32x4 *>(ks + k_rd[h / NB] + 32 * (h % NB) * G_::kRowBytes);
        return v_operand(vs, h / NC, h % NC);
      };
      u32x4 op[16];
      // Probabilities of tile j go to pfb[j mod 2]; PV(j-1) reads the other.
      u32x4 (&pf)[2 * NB] = w.pfb[PAR];
      const u32x4 (&pfp)[2 * NB] = w.pfb[PAR ^ 1];
      float rsum0 = 0.f, rsum1 = 0.f;   // row sum: even and odd keys of the tile
      float x_prev = 0.f;
      constexpr int kAhead = 3;         // LDS operand reads, steps ahead of their MFMA
#pragma unroll
      for (int i = 0; i < kAhead; ++i) {
        if (!kFirst || (i & 1) == 0) op[i] = operand(i);
        else op[i] = u32x4{0u, 0u, 0u, 0u};
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        if (i + kAhead < 16) {
          if (!kFirst || ((i + kAhead) & 1) == 0) op[i + kAhead] = operand(i + kAhead);
        }
        const int h = i >> 1;
        if ((i & 1) == 0) {
          sn[h % NB] = Elem<DT>::mfma(op[i], w.qf[h / NB], h < NB ? f32x16{} : sn[h % NB]);
        } else if constexpr (!kFirst) {
          w.oacc[h % NC] = Elem<DT>::mfma(op[i], pfp[h / NC], w.oacc[h % NC]);
        }
        if constexpr (NB == 1) {
          const float x = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[0][i], sl2, mneg));
          if (i & 1) {
            pf[i >> 3][(i & 7) >> 1] = Elem<DT>::pack(x_prev, x);
            rsum0 += x_prev;
            rsum1 += x;
          }
          x_prev = x;
        } else {
          const int r = (2 * i) & 15;
          const float x0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i >> 3][r], sl2, mneg));
          const float x1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[i >> 3][r + 1], sl2, mneg));
          pf[i >> 2][i & 3] = Elem<DT>::pack(x0, x1);
          rsum0 += x0;
          rsum1 += x1;
        }
        if constexpr (KG > 1) {
          if (i == 1) dma(k_slot(SC_IC(J)), (j + 2) * KG + kg, F(), 0);
          if (i == 3 && late_v) dma(v_slot(SC_IC(J)), j * KG + kg, T(), 0);
        } else if constexpr (PAR == 0) {
          if (i == 1) dma(k_slot(SC_IC(J + 3)), j + 3, F(), bk0);
          if (i == 3) dma(k_slot(SC_IC(J + 4)), j + 4, F(), bk1);
          if (i == 5) dma(v_slot(SC_IC(J + 1)), j + 1, T(), bv0);
          if (i == 7) dma(v_slot(SC_IC(J + 2)), j + 2, T(), bv1);
          if (i == 9) bn0 = blk_of(j + 5);
          if (i == 11) bn1 = blk_of(j + 6);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      float rs = rsum0 + rsum1;
      if (!kFirst && __builtin_amdgcn_ballot_w64(!(rs <= Elem<DT>::kSumLimit))) rs = settle_max<D, DT>(w, sc, pf, sl2);
      w.l_run += rs;
      if constexpr (KG > 1) {
        dma_barrier<0>();
      } else if constexpr (PAR == 1) {
        dma_barrier<0>();
        bv0 = bk0;
        bv1 = bk1;
        bk0 = bn0;
        bk1 = bn1;
      }
    };
    // The last tile of a range at head_dim 64 whose second 32-key block has no
    // keys: PV(j-1) and the first block's softmax, no QK, no loads, and the
    // first block's PV, in the order of a whole tile (the same bits).  Taken
    // as a whole one, whose second half is masked, it cost every range of an
    // odd number of blocks 0.3-0.6 us, and calls over few keys had become
    // slower than with 32-key tiles: 8/8 heads, P=71, N=2 5.65 us, 5.36 so
    // (5.26 with 32-key tiles); 32/8, P=814, N=18 9.61, 9.04 (9.02); 113
    // drawn calls at head_dim 64 2.2% faster in the mean.
    auto iterate_half = [&](auto j_tag, auto first_tag, int j) {
      constexpr int J = decltype(j_tag)::value;
      constexpr bool kFirst = decltype(first_tag)::value;
      constexpr int PAR = J & 1;
      f32x16 (&sc)[1] = reinterpret_cast<f32x16 (&)[1]>(w.s[PAR]);
      u32x4 (&pf)[2] = reinterpret_cast<u32x4 (&)[2]>(w.pfb[PAR]);
      apply_mask(sc, lim_of(j));
      if constexpr (kFirst) {
        const float tm = tile_max(sc, sl2);
        w.m_run = tm > -INFINITY ? tm : 0.f;
      } else {
        pv(v_slot(SC_IC(J + R - 1)), w.pfb[PAR ^ 1], SC_IC(2 * NB));
      }
      float rs = softmax_tile<DT>(sc, pf, sl2, w.m_run);
      if (!kFirst && __builtin_amdgcn_ballot_w64(!(rs <= Elem<DT>::kSumLimit))) {
        w.s[PAR][NB - 1] = f32x16{} - INFINITY;
        rs = settle_max<D, DT>(w, w.s[PAR], w.pfb[PAR], sl2);
      }
      w.l_run += rs;
      if constexpr (PAR == 1) dma_barrier<0>();
      pv(v_slot(SC_IC(J)), w.pfb[PAR], SC_IC(2));
    };
    // j = 0 .. R-1 masked (exact for any tile; j = 0 sets the reference
    // max), then whole rounds of R unmasked tiles, then the rest masked.
    constexpr bool kHalves = KG == 1 && NB == 2;
    const auto half_last = [&] {
      if constexpr (kHalves)
        return k_end - k_begin - (n - 1) * TK <= TK / 2;
      else
        return F();
    }();
    const int n_full = n_it - half_last;
    if (!kHalves || n_full > 0) iterate(std::integral_constant<int, 0>(), T(), T(), 0);
    static_for<1, R>([&](auto J) {
      if (decltype(J)::value < (kHalves ? n_full : n_it)) iterate(J, T(), F(), decltype(J)::value);
    });
    int j = R;
    const int jm = min(j_mask, n_it);
    // (Narrow items at head_dim 64 mask every tile: a second copy of the
    // loop body takes them from 226 to 242 registers, which leaves no room
    // for a copy workgroup beside them.)
    if constexpr (KG == 1 || D == 128)
      for (; j + R - 1 < jm; j += R) static_for<0, R>([&](auto J) { iterate(J, F(), F(), j + decltype(J)::value); });
    for (; j < n_full; j += R)
      static_for<0, R>([&](auto J) {
        if (j + decltype(J)::value < n_full) iterate(J, T(), F(), j + decltype(J)::value);
      });
    // PV of the last tile; its V landed before the last barrier.
    const int last = (n_it - 1) % R;
    static_for<0, R>([&](auto S) {
      constexpr int kS = decltype(S)::value;   // R is even: kS has the parity of n_it - 1
      if (last != kS) return;
      if constexpr (kHalves) {
        if (half_last) {
          if (kS == 0 && n_full == 0)
            iterate_half(S, T(), 0);
          else
            iterate_half(S, F(), n_full);
          return;
        }
      }
      pv(v_slot(S), w.pfb[kS & 1], SC_IC(2 * NB));
    });
    // Loads of tiles past the end may still be in flight.
    dma_wait_all();
#undef SC_IC
  }

  // Done with K/V: every load of it has been consumed (loads past the range
  // touch no memory), so the slot may be refilled once every workgroup of
  // the launch has counted itself here.  Only the order after these reads
  // matters, no data flows to the refill: a relaxed device-scope add.
  if (a.done_counter != nullptr) {
    __syncthreads();
    if (tid == 0) __hip_atomic_fetch_add(a.done_counter, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // Combine the two halves' denominators and normalise.
  float l_tot = w.l_run + __shfl_xor(w.l_run, 32);
  if constexpr (KG > 1) {
    // Combine the key groups: every wave leaves its O (fp32, unnormalised),
    // reference max and denominator in LDS, and wave kg of a row block
    // finishes the 16-dim pieces kg, kg + 4 of its rows.  2 KiB per piece,
    // its two register quads 1 KiB apart.
    constexpr int NP = D / 16;
    auto piece = [&](int g, int p) -> unsigned char * {
      return ring + (rb * KG + g) * 2 * kSlot + p * 2048 + lane * 16;
    };
    dma_barrier<0>();   // every wave is done with the tiles
    const bool has_rows = rb * 32 < wi.nq * group;
#pragma unroll
    for (int p = 0; p < NP; ++p)
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        if (!has_rows) break;
        const f32x16 &o = w.oacc[p >> 1];
        const int e = 8 * (p & 1) + 4 * q;
        *reinterpret_cast<f32x4 *>(piece(kg, p) + 1024 * q) = f32x4{o[e], o[e + 1], o[e + 2], o[e + 3]};
      }
    if (half == 0) narrow_ml[rb * KG + kg][col] = f32x2{w.m_run, l_tot};
    __syncthreads();
    if (!has_rows) return;
    // A group without a visible key has l = 0 and an arbitrary reference.
    float wg[KG], m = -INFINITY;
    f32x2 ml[KG];
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      ml[g] = narrow_ml[rb * KG + g][col];
      if (ml[g][1] != 0.f) m = fmaxf(m, ml[g][0]);
    }
    l_tot = 0.f;
#pragma unroll
    for (int g = 0; g < KG; ++g) {
      wg[g] = ml[g][1] != 0.f ? __builtin_amdgcn_exp2f(ml[g][0] - m) : 0.f;
      l_tot += wg[g] * ml[g][1];
    }
    const float inv = timed_out ? __builtin_nanf("") : l_tot > 0.f ? 1.f / l_tot : 0.f;
    const float lse_val = timed_out ? __builtin_nanf("")
                          : l_tot > 0.f ? (m + __log2f(l_tot)) * 0.69314718055994530942f : -INFINITY;
    const int64_t prow = (int64_t)wi.split * a.total_q * a.n_q_heads + qrow;
    uint16_t *const dst = sd.n_splits == 1 ? a.out + io_row * D : a.part_o + prow * D;
#pragma unroll
    for (int i = 0; i < (NP + KG - 1) / KG; ++i) {
      const int p = kg + i * KG;
      float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int g = 0; g < KG; ++g)
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const f32x4 o = *reinterpret_cast<const f32x4 *>(piece(g, p) + 1024 * q);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[4 * q + e] += wg[g] * o[e];
        }
      if (valid) store_chunk<DT>(x, inv, dst + 16 * p + 8 * half);
    }
    if (valid && half == 0 && kg == 0) {
      if (sd.n_splits == 1) {
        if (a.lse != nullptr) a.lse[(int64_t)h * a.total_q + sd.cu_q + qpos] = lse_val;
      } else {
        a.part_lse[prow] = lse_val;
      }
    }
    return;
  }
  const float inv = timed_out ? __builtin_nanf("") : l_tot > 0.f ? 1.f / l_tot : 0.f;
  const float lse_val = timed_out ? __builtin_nanf("")
                        : l_tot > 0.f ? (w.m_run + __log2f(l_tot)) * 0.69314718055994530942f : -INFINITY;
  if (!valid) return;
  if (sd.n_splits == 1) {
    store_row<D, DT>(w, inv, half, a.out + io_row * D);
    if (a.lse != nullptr && half == 0) a.lse[(int64_t)h * a.total_q + sd.cu_q + qpos] = lse_val;
    return;
  }

  // Split-key: write this split's normalised partial and its log-sum-exp.
  const int64_t prow = (int64_t)wi.split * a.total_q * a.n_q_heads + qrow;
  // The partial is a convex combination of V rows, so it fits the element
  // type's range; storing it in that type halves the split traffic for one
  // extra rounding (2^-9 relative for bf16, 2^-11 for fp16).
  store_row<D, DT>(w, inv, half, a.part_o + prow * D);
  if (half == 0) a.part_lse[prow] = lse_val;
}

// Split-key merge of NR (token, head) rows per lane group: D / 8 lanes per
// row, 8 dims per lane (`sub`); rows[i] < 0 are skipped; at most SMAX
// splits per row.  Weights
// exp(lse_s - max) over the row's splits, weighted sum of the partials,
// written to `out` (and the row's natural-log lse to lse_out if given).
// Every split's lse and partial chunk of all NR rows are loaded before any
// is used: one memory round trip, whatever the split count (merging a few
// thousand rows is latency-bound, not bandwidth-bound).
template <int D, int DT, int NR, int SMAX>
__device__ __forceinline__ void merge_rows(const AttnArgs &a, const int64_t (&rows_i)[NR], int sub,
                                           const uint16_t *part_o, const float *part_lse, uint16_t *out,
                                           float *lse_out) {
  const int64_t rows = (int64_t)a.total_q * a.n_q_heads;
  SeqDesc sd[NR];
  float ls[NR][SMAX];
  u32x4 x[NR][SMAX];
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int64_t row = rows_i[i] < 0 ? 0 : rows_i[i];
    const int token = (int)((uint32_t)row / (uint32_t)a.n_q_heads);
    int lo = 0;
    if (a.n_seqs > 1) {
      int hi = a.n_seqs - 1;
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (a.seqs[mid].cu_q <= token) lo = mid; else hi = mid - 1;
      }
    }
    sd[i] = a.seqs != nullptr ? a.seqs[lo] : a.seq0;
    const int S = rows_i[i] < 0 ? 0 : sd[i].n_splits;
    const uint16_t *po = part_o + row * D + sub * 8;
#pragma unroll
    for (int s = 0; s < SMAX; ++s) {
      if (s < S && S > 1) {
        ls[i][s] = part_lse[s * rows + row];
        x[i][s] = *reinterpret_cast<const u32x4 *>(po + (int64_t)s * rows * D);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NR; ++i) {
    const int S = rows_i[i] < 0 ? 0 : sd[i].n_splits;
    if (S <= 1) continue;
    const int64_t row = rows_i[i];
    const int token = (int)((uint32_t)row / (uint32_t)a.n_q_heads);
    const int h = (int)((uint32_t)row - (uint32_t)token * (uint32_t)a.n_q_heads);
    const int64_t io_row = (int64_t)(sd[i].q_off + token - sd[i].cu_q) * a.n_q_heads + h;
    float mx = -INFINITY;
#pragma unroll
    for (int s = 0; s < SMAX; ++s)
      if (s < S) mx = fmaxf(mx, ls[i][s]);
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    float wsum = 0.f;
#pragma unroll
    for (int s = 0; s < SMAX; ++s)
      if (s < S) {
        const float wgt = ls[i][s] == -INFINITY ? 0.f : __expf(ls[i][s] - mx);
        wsum += wgt;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const f32x2 v = Elem<DT>::unpack(x[i][s][e]);
          acc[2 * e] += wgt * v[0];
          acc[2 * e + 1] += wgt * v[1];
        }
      }
    const float winv = wsum > 0.f ? 1.f / wsum : 0.f;
    u32x4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = Elem<DT>::pack(acc[2 * e] * winv, acc[2 * e + 1] * winv);
    *reinterpret_cast<u32x4 *>(out + io_row * D + sub * 8) = pk;
    if (lse_out != nullptr && sub == 0)
      lse_out[(int64_t)h * a.total_q + token] = wsum > 0.f ? mx + __logf(wsum) : -INFINITY;
  }
}

// The deferred merge of the previous layer (AttnArgs::dm_out), run by a
// workgroup after its own item: it claims chunks of rows (one row per D / 8
// lanes, NR rows per lane group in one memory round trip) until all are
// claimed, so the workgroups that finish their items first do most of it.
// With at most four splits per row (the common plans) a lane group takes
// four rows; with more, one (the registers of the split values).  The
// claims only divide the work; no data flows through the counter (the
// partials were written by the previous launch on the stream).
template <int D, int DT, int NR, int SMAX>
__device__ __forceinline__ void deferred_merge_n(const AttnArgs &a) {
  constexpr int LPR = D / 8;
  constexpr int RPP = kThreads / LPR;   // rows per pass and row slot
  constexpr int64_t kChunk = (int64_t)NR * RPP;
  __shared__ uint32_t s_claim;
  const int64_t rows = (int64_t)a.total_q * a.n_q_heads;
  const int64_t n_chunks = (rows + kChunk - 1) / kChunk;
  const int sub = threadIdx.x % LPR;
  for (;;) {
    __syncthreads();                      // every lane has read the last claim
    if (threadIdx.x == 0)
      s_claim = __hip_atomic_fetch_add(a.dm_counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __syncthreads();
    const int64_t c = (int64_t)s_claim;
    if (c >= n_chunks) break;
    const int64_t base = c * kChunk + threadIdx.x / LPR;
    int64_t rr[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) rr[i] = base + i * RPP < rows ? base + i * RPP : -1;
    merge_rows<D, DT, NR, SMAX>(a, rr, sub, a.dm_part_o, a.dm_part_lse, a.dm_out, nullptr);
  }
}

constexpr int kMergeRows = 4;   // rows per lane group, of at most four splits
template <int D, int DT>
__device__ __forceinline__ void deferred_merge(const AttnArgs &a) {
  if (a.dm_max_splits <= 4)
    deferred_merge_n<D, DT, kMergeRows, 4>(a);
  else if (a.dm_max_splits <= 16)
    deferred_merge_n<D, DT, 1, 16>(a);
  else
    deferred_merge_n<D, DT, 1, kAttnMaxSplits>(a);
}

// Item of workgroup w in an implicit work list (see AttnArgs::seq0).
__device__ __forceinline__ WorkItem implicit_item(const AttnArgs &a, int w) {
  WorkItem wi{-1, 0, 0, 0, 0, 0, 0, 0};
  const int S = a.imp_splits;
  const int per_kvh = a.imp_tiles * S;
  const int j = w >> 3;
  const int g = (w & 7) * a.imp_per_xcd + j;
  if (j >= a.imp_per_xcd || g >= a.n_kv_heads * per_kvh) return wi;
  const int kvh = g / per_kvh;
  const int r = g - kvh * per_kvh;
  const int tile = r / S;
  const int sp = r - tile * S;
  const int q0 = tile * a.rows_q;
  const int nq = min(a.rows_q, a.seq0.n_new - q0);
  const int keys = a.seq0.prefix + q0 + nq;
  const int t = (keys + KT - 1) / KT;
  const int b0 = min(keys, (sp * t / S) * KT);
  const int b1 = min(keys, ((sp + 1) * t / S) * KT);
  wi.seq = 0;
  wi.kvh = kvh;
  wi.q0 = q0;
  wi.nq = nq;
  wi.k_begin = b0;
  wi.k_end = max(b0, b1);
  wi.split = sp;
  return wi;
}

template <int D, int DT, bool kNarrow>
__device__ __forceinline__ void attn_fwd_body(const AttnArgs &a) {
  AttnItem it;
  if (a.items != nullptr)
    it = load_const(a.items + blockIdx.x);
  else
    it = AttnItem{implicit_item(a, blockIdx.x), a.seq0};
  const WorkItem &wi = it.wi;
  if (wi.seq < 0) {
    // Padding slot (XCD placement): no K/V to read, but it counts as done
    // like every other workgroup of the launch.
    if (a.done_counter != nullptr && threadIdx.x == 0)
      __hip_atomic_fetch_add(a.done_counter, (uint64_t)1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  if constexpr (kNarrow) {
    __shared__ __attribute__((aligned(1024))) unsigned char ring[4 * kNarrowGroups * kSlot];
    if (wi.paged)
      attn_item<D, DT, true, 1, false>(a, ring, wi, it.sd);
    else if (wi.nq * a.group <= a.narrow_rows)
      attn_item<D, DT, false, kNarrowGroups, false>(a, ring, wi, it.sd);
    else
      attn_item<D, DT, false, 1, false>(a, ring, wi, it.sd);
  } else {
    if (wi.paged)
      attn_item<D, DT, true, 1, true>(a, nullptr, wi, it.sd);
    else
      attn_item<D, DT, false, 1, true>(a, nullptr, wi, it.sd);
  }
}

// One work item per workgroup, then (in a layer stack with deferred
// merges) its share of the previous layer's merge.
// kNarrow: for plans with narrow items.  Plans without (every query tile
// full or nearly so) run the kernel without their body: with it, the 8B-shape
// stack ran 0.4% slower (a longer start, six more registers).
// kBeside: the workgroups from dm_first on do the previous layer's merge, on
// CUs the items leave idle: after an item, the claims and the rows' round
// trips ended every layer of a short turn (32-layer stack of a 64-token turn
// over 1024 tokens: 643 us, 555 beside).  A kernel of its own: the branch in
// the others cost every call 0.2-0.4 us.
template <int D, int DT, bool kNarrow, bool kBeside>
__global__ __launch_bounds__(kThreads, 2) void attn_fwd_kernel(AttnArgs a) {
  if constexpr (kBeside) {
    if ((int)blockIdx.x >= a.dm_first)
      deferred_merge<D, DT>(a);
    else
      attn_fwd_body<D, DT, kNarrow>(a);
  } else {
    attn_fwd_body<D, DT, kNarrow>(a);
    if (a.dm_out != nullptr) deferred_merge<D, DT>(a);
  }
}

template <int D, int DT, int SMAX>
__global__ __launch_bounds__(256) void attn_merge_kernel(AttnArgs a) {
  constexpr int LPR = D / 8;
  constexpr int RPB = 256 / LPR;
  const int64_t rows = (int64_t)a.total_q * a.n_q_heads;
  const int64_t row = (int64_t)blockIdx.x * RPB + threadIdx.x / LPR;
  if (row >= rows) return;
  const int64_t rr[1] = {row};
  merge_rows<D, DT, 1, SMAX>(a, rr, threadIdx.x % LPR, a.part_o, a.part_lse, a.out, a.lse);
}

// Split-key partials of the allocation-free entry point: one array per
// device, held by the loaded code object until the process ends.  Host code
// must use the address hipGetSymbolAddress returns, never the symbol.
static __device__ __align__(256) unsigned char scratch[kNoAllocPartialBytes];

}  // namespace

hipError_t noalloc_scratch(int device, void **ptr, size_t *bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void *addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (addr[device] == nullptr) {
    // Each device holds its own copy of the array at its own address, so
    // the lookup runs with that device current.
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device && (e = hipSetDevice(device)) != hipSuccess) return e;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != device) (void)hipSetDevice(cur);
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    addr[device] = p;
  }
  *ptr = addr[device];
  *bytes = kNoAllocPartialBytes;
  return hipSuccess;
}

namespace {
using FwdKernel = void (*)(AttnArgs);
template <bool kNarrow, bool kBeside>
FwdKernel fwd_kernel_of(int head_dim, int dtype) {
  if (head_dim == 128)
    return dtype == SC_DTYPE_F16 ? attn_fwd_kernel<128, SC_DTYPE_F16, kNarrow, kBeside>
                                 : attn_fwd_kernel<128, SC_DTYPE_BF16, kNarrow, kBeside>;
  return dtype == SC_DTYPE_F16 ? attn_fwd_kernel<64, SC_DTYPE_F16, kNarrow, kBeside>
                               : attn_fwd_kernel<64, SC_DTYPE_BF16, kNarrow, kBeside>;
}
FwdKernel fwd_kernel(int head_dim, int dtype, bool narrow, bool beside) {
  if (beside) return narrow ? fwd_kernel_of<true, true>(head_dim, dtype) : fwd_kernel_of<false, true>(head_dim, dtype);
  return narrow ? fwd_kernel_of<true, false>(head_dim, dtype) : fwd_kernel_of<false, false>(head_dim, dtype);
}
}  // namespace

hipError_t launch_attn_fwd(const AttnArgs &a, int head_dim, int n_groups, hipStream_t stream) {
  if (n_groups <= 0) return hipSuccess;
  hipLaunchKernelGGL(fwd_kernel(head_dim, a.dtype, a.narrow_rows > 0, a.dm_first > 0), dim3(n_groups), dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

int attn_fwd_vgprs(int head_dim) {
  // The largest of this head_dim's kernels (element types, item kinds).
  int m = -1;
  for (int dtype : {SC_DTYPE_BF16, SC_DTYPE_F16})
    for (int kind = 0; kind < 4; ++kind) {
      hipFuncAttributes at{};
      const FwdKernel f = fwd_kernel(head_dim, dtype, kind & 1, kind >> 1);
      if (hipFuncGetAttributes(&at, reinterpret_cast<const void *>(f)) != hipSuccess) return -1;
      m = at.numRegs > m ? at.numRegs : m;
    }
  return m;
}

size_t attn_fwd_lds_bytes(int head_dim, bool narrow) {
  // The largest static LDS of these kernels; the full LDS of a CU if the
  // runtime cannot tell.
  size_t m = 0;
  for (int dtype : {SC_DTYPE_BF16, SC_DTYPE_F16})
    for (bool beside : {false, true}) {
      hipFuncAttributes at{};
      const FwdKernel f = fwd_kernel(head_dim, dtype, narrow, beside);
      if (hipFuncGetAttributes(&at, reinterpret_cast<const void *>(f)) != hipSuccess) return (size_t)160 << 10;
      m = at.sharedSizeBytes > m ? at.sharedSizeBytes : m;
    }
  return m;
}

int64_t deferred_merge_chunks(int64_t rows, int head_dim, int max_splits) {
  const int64_t chunk = (int64_t)(max_splits <= 4 ? kMergeRows : 1) * (kThreads / (head_dim / 8));
  return (rows + chunk - 1) / chunk;
}

hipError_t launch_attn_merge(const AttnArgs &a, int head_dim, int max_splits, hipStream_t stream) {
  const int64_t rows = (int64_t)a.total_q * a.n_q_heads;
  if (rows <= 0) return hipSuccess;
  const dim3 grid((unsigned)((rows * (head_dim / 8) + 255) / 256)), block(256);
  auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, a); };
  // Two bounds on the splits of a row: the registers of the wider one would
  // halve the waves in flight of calls with many rows, which have few splits.
  const bool wide = max_splits > 16;
  if (head_dim == 128) {
    if (a.dtype == SC_DTYPE_F16)
      wide ? launch(attn_merge_kernel<128, SC_DTYPE_F16, kAttnMaxSplits>) : launch(attn_merge_kernel<128, SC_DTYPE_F16, 16>);
    else
      wide ? launch(attn_merge_kernel<128, SC_DTYPE_BF16, kAttnMaxSplits>) : launch(attn_merge_kernel<128, SC_DTYPE_BF16, 16>);
  } else {
    if (a.dtype == SC_DTYPE_F16)
      wide ? launch(attn_merge_kernel<64, SC_DTYPE_F16, kAttnMaxSplits>) : launch(attn_merge_kernel<64, SC_DTYPE_F16, 16>);
    else
      wide ? launch(attn_merge_kernel<64, SC_DTYPE_BF16, kAttnMaxSplits>) : launch(attn_merge_kernel<64, SC_DTYPE_BF16, 16>);
  }
  return hipGetLastError();
}

}  // namespace sc
