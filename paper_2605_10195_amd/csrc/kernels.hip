// HIP kernels for tree decode attention on gfx950 (CDNA4, 64-lane wavefronts).
//
//   spex_tree_walk_kernel  (the default path)
//       One workgroup per (row block, kv head) carries up to 16 * NTW * NW query rows from the root
//       to their requested nodes in one launch: blocks whose rows span several wavefronts are
//       fetched once per workgroup and staged in LDS as MFMA operand images, blocks of one
//       wavefront stream straight into its operand registers, and the online-softmax state stays
//       in registers until the finished rows are written -- no partial results, no merge.
//   spex_split_attn_kernel
//       The split path: one workgroup per work item = (task, kv head, row tiles), all items of a
//       request in one launch.  A task is a run of KV pages (a chunk of a shared-prefix group or of a
//       private suffix) and a set of query rows.  Items of many rows stage operand images in LDS as
//       the tree-walk kernel does; items of few rows split their pages between four wavefronts that
//       stream them from memory to registers (S^T = K Q^T and O^T = V^T P^T with MFMA 16x16x32,
//       fp32 accumulation).  Small launches, and fp8 ones of middle size whose items are long, take the row tiles of
//       the first kind the second way, a workgroup each.  Every item keeps an online softmax per row and emits the partial state
//       (m, l, o); a shared page is read from memory once for all rows below it.
//   spex_wave_attn_kernel / spex_coop_attn_kernel
//       The same items in launches of their own, few rows (a wavefront an item) and many, where there
//       are items enough; private items come last and finish the rows of suffixes in one piece.
//   spex_rowmajor_attn_kernel
//       Same contract for row-major pools (fp32 KV, other page sizes and head dims): fp32 pools on the fp32
//       MFMA, 16-bit and fp8 ones on the bf16 MFMA with weights in three pieces.
//   spex_generic_attn_kernel
//       Same contract without matrix cores, for rows that its loads do not fit and as a cross-check.
//   spex_lse_merge_kernel
//       Combines the partial states of every query row (log-sum-exp rule) and normalises.
//   spex_write_tiles_kernel / spex_write_rows_kernel / spex_read_pages_kernel
//       Write a run of one node's tokens into the paged pool (quantised to e4m3 on the way where asked
//       for) / read tokens out of it, a page and kv head per workgroup, 16 bytes at a time.
//   spex_scatter_kv_kernel / spex_scatter_quant_kernel / spex_gather_kv_kernel
//       The same element by element, for rows or buffers that are not 16-byte aligned.
//   spex_append_tokens_kernel
//       One token for each of many nodes.
//   spex_patch_plan_kernel
//       Applies {index, value} patches to the device copy of the cached launch lists.
#include "kernels.hpp"

#include <climits>

namespace spex {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

constexpr float kNegInf = -__builtin_huge_valf();
// Largest V page scale the fp16 operand images can hold: 448 * 146 = 65408 <= 65504.  A larger
// scale is read as this one (the page's values shrink together instead of turning into infinities).
constexpr float kMaxVScaleF16 = 146.0f;
// Start value of the tree-walk kernel's softmax reference: finite, so that (-inf) - m stays -inf,
// and so far below any score that the first visible score replaces it.
constexpr float kWalkMInit = -1.0e30f;
// The same for row-major pools, which hold fp32: no finite score lies below it.
constexpr float kRowMajorMInit = -__FLT_MAX__;

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// Wave-uniform read of plan data through the scalar (constant) path.  The plan arrays are
// written by the host before the launch and never by a kernel.  Going through scalar loads keeps
// these small reads out of the vector-memory queue, whose in-order completion counter would
// otherwise make every page-record lookup wait for all K/V loads in flight.
typedef const int32_t __attribute__((address_space(4))) const_i32;
__device__ __forceinline__ int sload(const int32_t *base, int64_t idx) {
  return ((const_i32 *)(uintptr_t)base)[idx];
}

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Maximum over lanes l, l^16, l^32, l^48 (the four lane groups that hold one query row), by the
// gfx950 row-swap instructions: v_permlane16_swap exchanges the odd 16-lane rows of its first
// operand with the even rows of its second, v_permlane32_swap the upper half of the first with
// the lower half of the second; with both operands equal, the pair afterwards holds the value of
// the lane and of its partner.  Two wait states separate a vector write from a swap that reads it.
// The compiler does not track hazards of instructions inside inline assembly, so the argument must
// be the result of an ordinary vector ALU instruction (here: the v_max that folds in the running
// maximum) -- never directly of an MFMA, whose results need many more wait states before they can
// be read.
__device__ __forceinline__ float row_group_max(float v) {
  float a = v, b = v;
  asm("s_nop 1\n\t"
      "v_permlane16_swap_b32 %0, %1\n\t"
      "v_max_f32 %0, %0, %1\n\t"
      "v_mov_b32 %1, %0\n\t"
      "s_nop 1\n\t"
      "v_permlane32_swap_b32 %0, %1\n\t"
      "v_max_f32 %0, %0, %1"
      : "+v"(a), "+v"(b));
  return a;
}

// 128-bit K/V load.  Every K/V byte is used once per launch, so the loads carry the non-temporal
// hint: measured on MI355X, a streaming read of the pool reaches 7.0 TB/s with it against
// 6.2 TB/s without (the lines do not displace each other in the last-level caches).
__device__ __forceinline__ u32x4 load_kv(const char *p) {
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(p));
}

// ---- element offsets inside a (page, kv head) tile ------------------------------------------
template <int KV, int LAYOUT>
__device__ __forceinline__ int k_offset(int t, int d, int D) {
  if (LAYOUT == kRowMajor) return t * D + d;
  const int tt = 4 * (t >> 3) + (t & 3);
  if (KV == kFP8)
    return ((t >> 2) & 1) * 8 * D + (d >> 6) * 512 + ((d & 31) >> 3) * 128 + tt * 16 +
           ((d >> 5) & 1) * 8 + (d & 7);
  return ((t >> 2) & 1) * 8 * D + (d >> 5) * 256 + ((d & 31) >> 3) * 64 + tt * 8 + (d & 7);
}

template <int KV, int LAYOUT>
__device__ __forceinline__ int v_offset(int t, int d, int D) {
  if (LAYOUT == kRowMajor) return t * D + d;
  if (KV == kFP8)
    return (d >> 5) * 512 + (t >> 3) * 256 + (d & 15) * 16 + ((d >> 4) & 1) * 8 + (t & 7);
  return (d >> 4) * 256 + (t >> 3) * 128 + (d & 15) * 8 + (t & 7);
}

__device__ __forceinline__ float bf16_bits_to_float(uint16_t b) {
  return __builtin_bit_cast(float, static_cast<uint32_t>(b) << 16);
}

// OCP e4m3fn code -> fp32 (exact).
__device__ __forceinline__ float e4m3_to_float(uint8_t c) {
  const f32x2 r = __builtin_amdgcn_cvt_pk_f32_fp8(static_cast<int>(c), false);
  return r[0];
}

template <int KV>
__device__ __forceinline__ float load_elem(const void *base, int64_t idx) {
  if (KV == kF32) return static_cast<const float *>(base)[idx];
  if (KV == kBF16) return bf16_bits_to_float(static_cast<const uint16_t *>(base)[idx]);
  return e4m3_to_float(static_cast<const uint8_t *>(base)[idx]);
}

// V of a bf16 pool in the MFMA-tiled layout is stored as IEEE half precision, so that a tile is an
// fp16 operand image of the PV product as it lies in memory.  The append kernels convert once,
// rounding toward zero: exact for magnitudes in [2^-17, 65504] (a bf16 has 8 significant bits, an
// fp16 11, and subnormal fp16 still resolve 2^-24); a finite magnitude above 65504 becomes +-65504
// instead of infinity (0 * inf in the PV product would poison a whole row), one below 2^-17 keeps
// the multiples of 2^-24 it contains.  K stays bf16.
template <int KV, int LAYOUT>
__device__ __forceinline__ constexpr bool v_is_f16() {
  return KV == kBF16 && LAYOUT == kMfmaTiled;
}
__device__ __forceinline__ uint16_t bf16_bits_to_f16_bits(uint16_t b) {
  const uint32_t w = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(bf16_bits_to_float(b), 0.f));
  return static_cast<uint16_t>(w & 0xffffu);
}
// Back to bf16 by truncation: exact for everything bf16_bits_to_f16_bits produced.
__device__ __forceinline__ uint16_t f16_bits_to_bf16_bits(uint16_t h) {
  const float f = static_cast<float>(__builtin_bit_cast(_Float16, h));
  return static_cast<uint16_t>(__builtin_bit_cast(uint32_t, f) >> 16);
}
template <int KV, int LAYOUT>
__device__ __forceinline__ float load_v_elem(const void *base, int64_t idx) {
  if (v_is_f16<KV, LAYOUT>())
    return static_cast<float>(__builtin_bit_cast(_Float16, static_cast<const uint16_t *>(base)[idx]));
  return load_elem<KV>(base, idx);
}

template <int KV>
__device__ __forceinline__ constexpr int elem_size() {
  return KV == kF32 ? 4 : (KV == kBF16 ? 2 : 1);
}

// ---- MFMA attention ------------------------------------------------------------------------
// Two fp32 -> one dword of two bf16 (truncation): low half from a, high half from b.
__device__ __forceinline__ uint32_t pack_hi16(float a, float b) {
  return __builtin_amdgcn_perm(__builtin_bit_cast(uint32_t, b), __builtin_bit_cast(uint32_t, a),
                               0x07060302u);
}

// Eight e4m3 codes (two dwords) -> eight bf16 (exact: 3 mantissa bits fit in 7).  The scaled
// conversion of gfx950 turns two codes into two packed 16-bit values in one instruction; it uses
// only the exponent of its scale operand (checked on the device for all codes), here 2^0.
__device__ __forceinline__ bf16x8 fp8x8_to_bf16x8(uint32_t w0, uint32_t w1) {
  u32x4 r;
  r[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(static_cast<int>(w0), 1.0f, false));
  r[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(static_cast<int>(w0), 1.0f, true));
  r[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(static_cast<int>(w1), 1.0f, false));
  r[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(static_cast<int>(w1), 1.0f, true));
  return __builtin_bit_cast(bf16x8, r);
}

// Wave-uniform description of one work item.
struct Item {
  int pg_begin, pg_count, qt_begin, qt_count, pbase, flags, g, row0;
};

__device__ __forceinline__ Item load_item(const int32_t *items, int idx) {
  const int64_t r = static_cast<int64_t>(uniform(idx)) * 8;
  Item it;
  it.pg_begin = sload(items, r + 0);
  it.pg_count = sload(items, r + 1);
  it.qt_begin = sload(items, r + 2);
  it.qt_count = sload(items, r + 3);
  it.pbase = sload(items, r + 4);
  it.flags = sload(items, r + 5);
  it.g = sload(items, r + 6);
  it.row0 = sload(items, r + 7);
  return it;
}

// Page ids / valid counts / positions of one 32-token block, wave-uniform.
struct BlockMeta {
  int pid_a, pid_b, vp_a, vp_b;  // vp = position << 7 | valid; vp_b = 0 when the block has one page
};

__device__ __forceinline__ BlockMeta load_block_meta(const int32_t *pg_rec, const Item &it, int b) {
  const int ia = it.pg_begin + 2 * b;
  const bool has_b = 2 * b + 1 < it.pg_count;
  const int ib = has_b ? ia + 1 : ia;
  BlockMeta bm;
  bm.pid_a = sload(pg_rec, 2 * ia);
  bm.vp_a = sload(pg_rec, 2 * ia + 1);
  bm.pid_b = sload(pg_rec, 2 * ib);
  bm.vp_b = has_b ? sload(pg_rec, 2 * ib + 1) : 0;
  return bm;
}

// Per-wavefront state of NT tiles of 16 query rows.  Lane (n = lane % 16, jj = lane / 16) works
// on row n of every tile; its accumulators hold dims dt*16 + 4*jj .. +3.
template <int D, int NT>
struct RowState {
  bf16x8 qf[NT][D / 32];  // query operand: dims s*32 + 8*jj .. +7
  int limit[NT], qtok[NT];
  int qidx[NT];           // draft token trees: index of the row's query in its request
  uint32_t dmask[NT];     //   and its visibility mask among the request's drafts
  f32x4 o[NT][D / 16];
  float m[NT], l[NT];     // l is this lane's share; summed over the four jj at the end
};

// Scores of the lane's 8 tokens that the row does not see become -inf.  Chain: the first
// limit - pos positions of the page are visible.  Draft token tree: positions below
// base = limit - 1 - qidx are visible, position base + k iff bit k of the row's mask is set; shifting
// {mask, 32 ones} right by (first position of the lane's tokens - base + 32) puts the visibility of
// the lane's 8 tokens into the low 8 bits.
template <bool TREE>
__device__ __forceinline__ void mask_scores(float (&x)[8], int limit, int qidx, uint32_t dmask, int valid_l,
                                            int pos_l, bool row_in) {
  const int jj = (threadIdx.x & 63) >> 4;
  const int first = 8 * (jj & 1);
  if (TREE) {
    const int base = limit - 1 - qidx;
    const int sh = pos_l + first - base + 32;
    const uint64_t bits = (static_cast<uint64_t>(dmask) << 32) | 0xffffffffull;
    uint32_t vm = sh <= 0 ? 0xffu : (sh >= 64 ? 0u : static_cast<uint32_t>(bits >> sh) & 0xffu);
    const int have = valid_l - first;  // tokens of the lane's 8 that exist
    vm = row_in ? vm : 0u;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = (i < have && ((vm >> i) & 1u)) ? x[i] : kNegInf;
  } else {
    int vis = limit - pos_l;
    vis = vis < valid_l ? vis : valid_l;
    vis -= first;
    vis = row_in ? vis : 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = i < vis ? x[i] : kNegInf;
  }
}

template <int D, int NT>
__device__ __forceinline__ void load_rows(const AttnArgs &p, const Shape &sh, const Item &cur,
                                          int row_base, RowState<D, NT> &st) {
  const int lane = threadIdx.x & 63, m16 = lane & 15, jj = lane >> 4;
  const int G = sh.G, rows = cur.qt_count * G;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int r = row_base + nt * 16 + m16;
    st.limit[nt] = INT_MAX;
    st.qtok[nt] = 0;
    st.qidx[nt] = 0;
    st.dmask[nt] = 0;
    st.m[nt] = kNegInf;
    st.l[nt] = 0.f;
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) st.o[nt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (r < rows) {
      const int2 qr = *reinterpret_cast<const int2 *>(p.qt_rec + 2 * (cur.qt_begin + r / G));
      st.limit[nt] = qr.y;
      st.qtok[nt] = qr.x;
      if (p.qt_mask) {
        const int2 dm = *reinterpret_cast<const int2 *>(p.qt_mask + 2 * qr.x);
        st.qidx[nt] = dm.x;
        st.dmask[nt] = static_cast<uint32_t>(dm.y);
      }
      const uint16_t *qp = static_cast<const uint16_t *>(p.q) +
                           (static_cast<int64_t>(qr.x) * sh.Hq + cur.g * G + r % G) * D + jj * 8;
#pragma unroll
      for (int s = 0; s < D / 32; ++s)
        st.qf[nt][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(qp + s * 32));
    } else {
#pragma unroll
      for (int s = 0; s < D / 32; ++s) st.qf[nt][s] = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});
    }
  }
}

// One 32-token block (pages A and B of one kv head) against the wavefront's rows.
// kf[t][s]: K half-tile t (tokens {0-3, 8-11} + 4t of each page), dims s*32..; rows 0-7 of the MFMA
// tile come from page A, rows 8-15 from page B.  vf[dt]: V^T, dims dt*16.., tokens 8*(jj&1)..+7 of
// page jj/2.  After the two score tiles this lane holds the scores of exactly those 8 tokens, i.e.
// the operand layout of the PV product, so P never leaves the registers.
// VF16: vf holds fp16 (V of a bf16 pool as stored), else bf16 (widened fp8 codes).
template <bool TREE, bool VF16, int D, int NT, class Refill>
__device__ __forceinline__ void block_math(RowState<D, NT> &st, const bf16x8 (&kf)[2][D / 32],
                                           const bf16x8 (&vf)[D / 16], bool masked, int valid_l,
                                           int pos_l, float c, float vs, Refill refill_k) {
  f32x4 sa[NT], sb[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    sa[nt] = sb[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
      sa[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][s], st.qf[nt][s], sa[nt], 0, 0, 0);
      sb[nt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[1][s], st.qf[nt][s], sb[nt], 0, 0, 0);
    }
  }
  refill_k();
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float x[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = sa[nt][i] * c;
      x[4 + i] = sb[nt][i] * c;
    }
    if (masked) mask_scores<TREE>(x, st.limit[nt], st.qidx[nt], st.dmask[nt], valid_l, pos_l, true);
    float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                     fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(st.m[nt], mx);
    const float m_safe = m_new == kNegInf ? 0.f : m_new;
    const float alpha = fast_exp2(st.m[nt] - m_safe);
    float pr[8];
    float lsum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      pr[i] = fast_exp2(x[i] - m_safe);
      lsum += pr[i];
    }
    st.l[nt] = st.l[nt] * alpha + lsum;
    st.m[nt] = m_new;
    if (!__all(alpha == 1.0f)) {
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) st.o[nt][dt] *= alpha;
    }
    // P as two pieces (hi + lo, each rounded toward zero, lo from the exact fp32 remainder) so that
    // the product keeps ~16 (bf16 pieces) or ~22 (fp16 pieces) bits of each weight.
    u32x4 phi, plo;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float a0 = pr[2 * i] * vs, a1 = pr[2 * i + 1] * vs;
      if (VF16) {  // weights are at most 1 here: no overflow
        const auto h = __builtin_amdgcn_cvt_pkrtz(a0, a1);
        phi[i] = __builtin_bit_cast(uint32_t, h);
        plo[i] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(a0 - static_cast<float>(h[0]),
                                                                         a1 - static_cast<float>(h[1])));
      } else {
        const float h0 = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a0) & 0xffff0000u);
        const float h1 = __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a1) & 0xffff0000u);
        phi[i] = pack_hi16(h0, h1);
        plo[i] = pack_hi16(a0 - h0, a1 - h1);
      }
    }
    if (VF16) {
      const f16x8 ph = __builtin_bit_cast(f16x8, phi);
      const f16x8 pl = __builtin_bit_cast(f16x8, plo);
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) {
        const f16x8 vh = __builtin_bit_cast(f16x8, vf[dt]);
        st.o[nt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, ph, st.o[nt][dt], 0, 0, 0);
        st.o[nt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh, pl, st.o[nt][dt], 0, 0, 0);
      }
    } else {
      const bf16x8 ph = __builtin_bit_cast(bf16x8, phi);
      const bf16x8 pl = __builtin_bit_cast(bf16x8, plo);
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) {
        st.o[nt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], ph, st.o[nt][dt], 0, 0, 0);
        st.o[nt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[dt], pl, st.o[nt][dt], 0, 0, 0);
      }
    }
  }
}

// Floats of LDS one wavefront needs to transpose a 16-row tile.
template <int D>
constexpr int stage_floats() { return 16 * (D + 4); }

// Emit the rows of a wavefront: partial state (m, l, o) for the merge step, or the finished output rows:
// when every row of the launch has a single piece, or (ALLOW_FINAL, in a launch behind the one that wrote the
// rows' other pieces) for a task flagged final, after folding those in.  The
// accumulators hold 4 consecutive dims of one row per lane (64 B runs at a 512 B stride); they are
// transposed through the wave-private LDS tile `my` so that every store instruction writes whole
// rows (1 KiB contiguous) instead of half-filled cache lines.
template <int D, int NT, bool ALLOW_FINAL>
__device__ __forceinline__ void finish_rows(const AttnArgs &p, const Shape &sh, const Item &cur,
                                            int row_base, f32x4 (&o)[NT][D / 16],
                                            const float (&m_in)[NT], const float (&l_in)[NT],
                                            const int (&qtok)[NT], float *my) {
  constexpr int kRowPad = D + 4;  // the pad spreads rows over LDS banks
  const int lane = threadIdx.x & 63, m16 = lane & 15, jj = lane >> 4;
  const int G = sh.G, rows = cur.qt_count * G, g = cur.g;
  const bool fold_task = ALLOW_FINAL && (cur.flags & 2) != 0 && !p.finish;
  const bool finish = p.finish || fold_task;
  constexpr int kLanesPerRow = D / 4;  // 16-byte pieces per row
  constexpr int kRowsPerInst = 64 / kLanesPerRow;
  const int sub = lane / kLanesPerRow, piece = lane % kLanesPerRow;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    float l = l_in[nt];
    float m = m_in[nt];
    const int r0w = row_base + nt * 16;  // first row of this tile
    if (r0w >= rows) break;              // wave-uniform
    const bool row_ok = r0w + m16 < rows;
    const int hh = (r0w + m16) % G;
    int64_t dst_row;  // row index in part_o or in out
    if (fold_task) {
      // Fold in the other pieces of this row (written by the shared-prefix kernels, which ran
      // before on the same stream) and normalise.  All rows of a suffix belong to one requested
      // node, so they have the same number of pieces.
      int e0 = 0, n_other = 0;
      if (row_ok) {
        e0 = p.part_indptr[qtok[nt]];
        n_other = p.part_indptr[qtok[nt] + 1] - 1 - e0;
      }
      const int n_max = uniform(n_other);
      auto fold = [&](const f32x2 ml, const f32x4 (&oj)[D / 16], bool use) {
        const float mj = use ? ml[0] : kNegInf;
        const float m_new = fmaxf(m, mj);
        const float m_safe = m_new == kNegInf ? 0.f : m_new;
        const float fa = fast_exp2(m - m_safe), fb = fast_exp2(mj - m_safe);
        l = l * fa + ml[1] * fb;
        m = m_new;
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) o[nt][dt] = o[nt][dt] * fa + oj[dt] * fb;
      };
      if (n_max > 0) {
        // The first 8 pieces are fetched four at a time with all loads of a batch in flight
        // together.  Indices past a row's last piece are clamped to it (a repeated, finite read
        // that is weighted with zero), which keeps the batches free of per-piece branches.
        constexpr int kBatch = 4;
        int64_t slot[2 * kBatch];
#pragma unroll
        for (int j = 0; j < 2 * kBatch; ++j) {
          const int last = n_other - 1;
          const int e = e0 + max(0, j < last ? j : last);
          slot[j] = static_cast<int64_t>(p.part_base[e]) + static_cast<int64_t>(g) * p.part_hstride[e] + hh;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          if (q * kBatch < n_max) {
            f32x2 ml[kBatch];
            f32x4 oj[kBatch][D / 16];
#pragma unroll
            for (int k = 0; k < kBatch; ++k) {
              ml[k] = *reinterpret_cast<const f32x2 *>(p.part_ml + slot[q * kBatch + k] * 2);
              const float *src = p.part_o + slot[q * kBatch + k] * D + jj * 4;
#pragma unroll
              for (int dt = 0; dt < D / 16; ++dt) oj[k][dt] = *reinterpret_cast<const f32x4 *>(src + dt * 16);
            }
#pragma unroll
            for (int k = 0; k < kBatch; ++k) fold(ml[k], oj[k], q * kBatch + k < n_other);
          }
        }
        for (int j = 2 * kBatch; j < n_max; ++j) {  // deeper paths: one piece at a time
          const int last = n_other - 1;
          const int e = e0 + max(0, j < last ? j : last);
          const int64_t sl = static_cast<int64_t>(p.part_base[e]) + static_cast<int64_t>(g) * p.part_hstride[e] + hh;
          const f32x2 ml = *reinterpret_cast<const f32x2 *>(p.part_ml + sl * 2);
          f32x4 oj[D / 16];
          const float *src = p.part_o + sl * D + jj * 4;
#pragma unroll
          for (int dt = 0; dt < D / 16; ++dt) oj[dt] = *reinterpret_cast<const f32x4 *>(src + dt * 16);
          fold(ml, oj, j < n_other);
        }
      }
    }
    if (finish) {
      const float inv = 1.0f / l;
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) o[nt][dt] *= inv;
      dst_row = static_cast<int64_t>(qtok[nt]) * sh.Hq + g * G + hh;
      if (row_ok && jj == 0 && p.lse) p.lse[dst_row] = (m + __builtin_log2f(l)) * 0.6931471805599453f;
    } else {
      dst_row = static_cast<int64_t>(cur.pbase) + static_cast<int64_t>(g) * rows + r0w + m16;
      if (row_ok && jj == 0) *reinterpret_cast<f32x2 *>(p.part_ml + dst_row * 2) = f32x2{m, l};
    }
    float *dst = finish ? p.out : p.part_o;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
      *reinterpret_cast<f32x4 *>(my + m16 * kRowPad + dt * 16 + jj * 4) = o[nt][dt];
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 16 / kRowsPerInst; ++i) {
      const int row = i * kRowsPerInst + sub;
      const f32x4 v = *reinterpret_cast<const f32x4 *>(my + row * kRowPad + piece * 4);
      // destination row index of tile row `row`, held by lane `row` (k-group 0)
      const int lo = __shfl(static_cast<int>(dst_row & 0xffffffff), row);
      const int hi = __shfl(static_cast<int>(dst_row >> 32), row);
      const int64_t drow = (static_cast<int64_t>(hi) << 32) | static_cast<uint32_t>(lo);
      if (r0w + row < rows) *reinterpret_cast<f32x4 *>(dst + drow * D + piece * 4) = v;
    }
  }
}

// Raw 128-bit pieces of one 32-token block (two pages) of one kv head, as loaded, and the lane's page scales (fp8).
template <int KV, int D>
struct RawBlock {
  static constexpr int NK = (KV == kFP8) ? D / 64 : D / 32;  // loads per K half-tile
  static constexpr int NV = (KV == kFP8) ? D / 32 : D / 16;
  u32x4 k[2][NK];
  u32x4 v[NV];
  float ks = 1.f, vs = 1.f;
};

// ---- split path: items of few rows -------------------------------------------------------------
// The work items of a launch, in up to four lists: workgroup wg_end[k - 1] .. wg_end[k] - 1 belong to
// list k.
struct SplitLists {
  static constexpr int kLists = 4;
  const int32_t *items[kLists];
  int32_t wg_end[kLists];
  int32_t n_items[kLists];
  int32_t span[kLists];     // rows an item of the list covers from its first row on
};
// The list the workgroup belongs to and its index there.
struct ListPos {
  int k, local, n_items, span;
  const int32_t *items;
};
__device__ __forceinline__ ListPos list_of(const SplitLists &ls, int wg) {
  ListPos r = {0, wg, ls.n_items[0], ls.span[0], ls.items[0]};
#pragma unroll
  for (int i = 1; i < SplitLists::kLists; ++i) {  // member by member: as a whole the lists go through scratch memory
    const bool in = wg >= ls.wg_end[i - 1];
    r.k = in ? i : r.k;
    r.local = in ? wg - ls.wg_end[i - 1] : r.local;
    r.n_items = in ? ls.n_items[i] : r.n_items;
    r.span = in ? ls.span[i] : r.span;
    r.items = in ? ls.items[i] : r.items;
  }
  return r;
}

template <int D>
constexpr int wave_fold_floats() { return 4 * (D / 16) * 256 + 4 * 16 * 2; }

// One work item of up to 16 * NT rows.  SPLIT: a workgroup for it.  A launch that is short of work items is
// long on latency (a block costs a memory round trip, then its arithmetic), so the item's blocks
// are split between the four wavefronts, which fold their softmax states through LDS; a chunk of
// 16 pages is then two blocks deep instead of eight.  Otherwise a wavefront takes the item (SUFFIX: rows of a
// private suffix, finished here where it is in one piece).
// DEEP: the K/V loads of block b+1 are in flight while block b is computed, in registers of their own.  The
// steady-state loop is free of conditional loads on purpose: the vector-memory completion counter is in-order, and a
// load that is issued on one path only would force the compiler to wait for everything outstanding at the join.
// Otherwise one set of registers, K's requested behind the score MFMAs of the block before, V's at the start of the
// block (130 and not 216 registers for fp8 heads of 128, 213 and not 392 with two row tiles).  K past the
// last block is requested as well, by all lanes from one address: a copy of the step without it makes the compiler carry
// the state over in 64 moves a step, which wait for the loads.
// CAP: V page scales above v_most are read as v_most, so that a node shared by many rows gives the same values as a row
// tile and through LDS.
template <int KV, int D, int NT, bool TREE, bool SPLIT, bool SUFFIX, bool DEEP, bool CAP = false>
__device__ __forceinline__ void wave_item(const AttnArgs &p, const Shape &sh, const Item &cur, float *lds, float v_most = 0.f) {
  constexpr int ESZ = (KV == kFP8) ? 1 : 2;
  constexpr int TILE_BYTES = 16 * D * ESZ;
  const int lane = threadIdx.x & 63;
  const int m16 = lane & 15;
  const int jj = lane >> 4;
  const int w = uniform(threadIdx.x >> 6);
  const char *kpool = static_cast<const char *>(p.k_pool);
  const char *vpool = static_cast<const char *>(p.v_pool);
  // Byte offset of this lane inside a K half-tile / a V tile.
  const int k_lane_off = jj * 128 + (m16 & 7) * 16;
  const int v_lane_off = (jj & 1) * 256 + m16 * 16;

  const int g = cur.g;
  const int n_all = (cur.pg_count + 1) >> 1;
  const int b_first = SPLIT ? (n_all * w) >> 2 : 0, nblk = SPLIT ? (n_all * (w + 1)) >> 2 : n_all;  // blocks b_first .. nblk - 1

  auto tile_of = [&](int pid) { return static_cast<int64_t>(pid) * sh.page_tiles + g; };
  auto issue_k = [&](RawBlock<KV, D> &rb, const BlockMeta &bm, int64_t tile_a, int64_t tile_b, int msk) {
    if (KV == kFP8) {
      const int sidx = (jj < 2 ? bm.pid_a : bm.pid_b) * sh.Hkv + g;
      rb.ks = p.k_scale[sidx];
      rb.vs = p.v_scale[sidx];
    }
    const char *kp = kpool + (m16 < 8 ? tile_a : tile_b) * TILE_BYTES + (k_lane_off & msk);
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int s = 0; s < RawBlock<KV, D>::NK; ++s)
        rb.k[t][s] = load_kv(kp + t * (TILE_BYTES / 2) + s * 512);
  };
  auto issue_v = [&](RawBlock<KV, D> &rb, int64_t tile_a, int64_t tile_b) {
    const char *vp = vpool + (jj < 2 ? tile_a : tile_b) * TILE_BYTES + v_lane_off;
#pragma unroll
    for (int s = 0; s < RawBlock<KV, D>::NV; ++s) rb.v[s] = load_kv(vp + s * 512);
  };
  auto issue_loads = [&](RawBlock<KV, D> &rb, const BlockMeta &bm) {
    const int64_t tile_a = tile_of(bm.pid_a), tile_b = tile_of(bm.pid_b);
    issue_k(rb, bm, tile_a, tile_b, -1);
    issue_v(rb, tile_a, tile_b);
  };
  // page records of block min(b, nblk - 1)
  auto meta = [&](int b) { return load_block_meta(p.pg_rec, cur, b < nblk ? b : nblk - 1); };

  const bool task_masked = (cur.flags & 1) != 0;
  RowState<D, NT> st;
  load_rows<D, NT>(p, sh, cur, cur.row0, st);

  // One block; refill_k is called where its K registers (and scales) are free.
  auto compute_block = [&](const RawBlock<KV, D> &rb, const BlockMeta &bm, auto refill_k) {
    bf16x8 kf[2][D / 32];
    bf16x8 vf[D / 16];
    if (KV == kFP8) {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < D / 64; ++s) {
          kf[t][2 * s] = fp8x8_to_bf16x8(rb.k[t][s][0], rb.k[t][s][1]);
          kf[t][2 * s + 1] = fp8x8_to_bf16x8(rb.k[t][s][2], rb.k[t][s][3]);
        }
#pragma unroll
      for (int s = 0; s < D / 32; ++s) {
        vf[2 * s] = fp8x8_to_bf16x8(rb.v[s][0], rb.v[s][1]);
        vf[2 * s + 1] = fp8x8_to_bf16x8(rb.v[s][2], rb.v[s][3]);
      }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < D / 32; ++s) kf[t][s] = __builtin_bit_cast(bf16x8, rb.k[t][s]);
#pragma unroll
      for (int s = 0; s < D / 16; ++s) vf[s] = __builtin_bit_cast(bf16x8, rb.v[s]);
    }
    // This lane's score registers cover tokens 8*(jj&1) .. +7 of page A (jj < 2) or B.
    const int vp = jj < 2 ? bm.vp_a : bm.vp_b;
    block_math<TREE, KV == kBF16, D, NT>(st, kf, vf, task_masked || (bm.vp_b & 127) == 0, vp & 127, vp >> 7,
                                         p.scale_log2 * rb.ks, CAP ? fminf(rb.vs, v_most) : rb.vs, refill_k);
  };

  if (b_first < nblk) {
    RawBlock<KV, D> r0;
    BlockMeta m0 = meta(b_first);
    if constexpr (DEEP) {
      const auto nothing = [] {};
      RawBlock<KV, D> r1;
      issue_loads(r0, m0);
      BlockMeta m1 = meta(b_first + 1);
      int b = b_first;
      for (; b + 2 < nblk; b += 2) {  // blocks b, b+1, b+2 all exist
        const BlockMeta m2 = meta(b + 2);
        issue_loads(r1, m1);
        compute_block(r0, m0, nothing);
        const BlockMeta m3 = meta(b + 3);
        issue_loads(r0, m2);
        compute_block(r1, m1, nothing);
        m0 = m2;
        m1 = m3;
      }
      if (b + 1 < nblk) {
        issue_loads(r1, m1);
        compute_block(r0, m0, nothing);
        compute_block(r1, m1, nothing);
      } else {
        compute_block(r0, m0, nothing);
      }
    } else {
      BlockMeta m1 = meta(b_first + 1);
      int64_t tile_a = tile_of(m0.pid_a), tile_b = tile_of(m0.pid_b);
      issue_k(r0, m0, tile_a, tile_b, -1);
      for (int b = b_first; b < nblk; ++b) {
        const BlockMeta m2 = meta(b + 2);
        issue_v(r0, tile_a, tile_b);
        tile_a = tile_of(m1.pid_a);
        tile_b = tile_of(m1.pid_b);
        compute_block(r0, m0, [&] { issue_k(r0, m1, tile_a, tile_b, b + 1 < nblk ? -1 : 0); });
        m0 = m1;
        m1 = m2;
      }
    }
  }

  if constexpr (!SPLIT) {
    float l_tot[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {  // the row sum is spread over the four lane groups
      float l = st.l[nt];
      l += __shfl_xor(l, 16);
      l += __shfl_xor(l, 32);
      l_tot[nt] = l;
    }
    finish_rows<D, NT, SUFFIX>(p, sh, cur, cur.row0, st.o, st.m, l_tot, st.qtok, lds + w * stage_floats<D>());
    return;
  }
  // ---- fold: every wavefront leaves its state in LDS, wavefront w then makes output tiles w, w + 4, ..
  const int rows = cur.qt_count * sh.G;
  f32x4 *fo = reinterpret_cast<f32x4 *>(lds);      // [wavefront][16-dim tile][lane]
  float *fml = lds + 4 * (D / 16) * 256;           // [wavefront][row][m, l]
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if (cur.row0 + nt * 16 >= rows) break;         // uniform over the workgroup
    float l = st.l[nt];                            // the row sum is spread over the four lane groups
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (nt > 0) __syncthreads();
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) fo[(w * (D / 16) + dt) * 64 + lane] = st.o[nt][dt];
    if (jj == 0) *reinterpret_cast<f32x2 *>(fml + (w * 16 + m16) * 2) = f32x2{st.m[nt], l};
    __syncthreads();
    f32x2 ml[4];
    float m_all = kNegInf;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      ml[v] = *reinterpret_cast<const f32x2 *>(fml + (v * 16 + m16) * 2);
      m_all = fmaxf(m_all, ml[v][0]);
    }
    const float m_safe = m_all == kNegInf ? 0.f : m_all;  // a row that sees nothing of the item: l = 0
    float f[4], l_all = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      f[v] = fast_exp2(ml[v][0] - m_safe);
      l_all += ml[v][1] * f[v];
    }
    const int row = cur.row0 + nt * 16 + m16;
    const bool row_ok = row < rows;
    const int64_t dst_row = p.finish ? static_cast<int64_t>(st.qtok[nt]) * sh.Hq + g * sh.G + row % sh.G
                                     : static_cast<int64_t>(cur.pbase) + static_cast<int64_t>(g) * rows + row;
    if (w == 0 && jj == 0 && row_ok) {
      if (!p.finish)
        *reinterpret_cast<f32x2 *>(p.part_ml + dst_row * 2) = f32x2{m_all, l_all};
      else if (p.lse)
        p.lse[dst_row] = (m_all + __builtin_log2f(l_all)) * 0.6931471805599453f;
    }
    const float norm = p.finish ? 1.0f / l_all : 1.0f;
    float *dst = (p.finish ? p.out : p.part_o) + dst_row * D + jj * 4;
#pragma unroll
    for (int i = 0; i < D / 64; ++i) {
      const int dt = i * 4 + w;
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int v = 0; v < 4; ++v) acc += fo[(v * (D / 16) + dt) * 64 + lane] * f[v];
      if (row_ok) *reinterpret_cast<f32x4 *>(dst + dt * 16) = acc * norm;
    }
  }
}

// Block step of items of many rows.  Same contraction as block_math, tuned for many row
// tiles per wavefront, where the vector ALU work of the softmax -- not the matrix cores -- sets
// the pace:
//  * P is rounded once to fp16 (11 significant bits; to nearest, one instruction per pair, because a
//    row's pieces are folded with pieces of the other items, whose weights are not rounded: the
//    mean shortfall of rounding toward zero would weigh this piece 3e-4 too low against them) and
//    V^T arrives as fp16 operand images, so
//    PV is one MFMA per tile instead of a hi and a lo one;
//  * the row sums come from one more MFMA against a tile of ones, which also adds up the four
//    lane groups and uses the same rounded weights as the numerator;
//  * with a page-independent scale (bf16 KV) the running maximum is kept on the raw scores and
//    scale and subtraction fuse into one FMA per score.
// m is in units of raw score for bf16 KV and of scaled score for fp8 KV (c differs per page).
template <bool FP8, bool TREE, int D, int NT>
__device__ __forceinline__ void block_math_f16(const bf16x8 (&qf)[NT][D / 32], const int (&limit)[NT],
                                               const int (&qidx)[NT], const uint32_t (&dmask)[NT],
                                               f32x4 (&o)[NT][D / 16], float (&m)[NT],
                                               f32x4 (&lacc)[NT], const bf16x8 (&kf)[2][D / 32],
                                               const f16x8 (&vh)[D / 16], bool masked, int valid_l,
                                               int pos_l, float c) {
  const _Float16 one = static_cast<_Float16>(1.0f);
  const f16x8 ones = {one, one, one, one, one, one, one, one};
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
      sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][s], qf[nt][s], sa, 0, 0, 0);
      sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[1][s], qf[nt][s], sb, 0, 0, 0);
    }
    float x[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[i] = FP8 ? sa[i] * c : sa[i];
      x[4 + i] = FP8 ? sb[i] * c : sb[i];
    }
    if (masked) mask_scores<TREE>(x, limit[nt], qidx[nt], dmask[nt], valid_l, pos_l, true);
    float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])),
                     fmaxf(fmaxf(x[4], x[5]), fmaxf(x[6], x[7])));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m[nt], mx);
    const float m_safe = m_new == kNegInf ? 0.f : m_new;
    float alpha, pr[8];
    if (FP8) {
      alpha = fast_exp2(m[nt] - m_safe);
#pragma unroll
      for (int i = 0; i < 8; ++i) pr[i] = fast_exp2(x[i] - m_safe);
    } else {
      const float mc = m_safe * c;
      alpha = fast_exp2(m[nt] * c - mc);
#pragma unroll
      for (int i = 0; i < 8; ++i) pr[i] = fast_exp2(__builtin_fmaf(x[i], c, -mc));
    }
    m[nt] = m_new;
    if (!__all(alpha == 1.0f)) {
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) o[nt][dt] *= alpha;
      lacc[nt] *= alpha;
    }
    u32x4 pw;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      pw[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{pr[2 * i], pr[2 * i + 1]}, f16x2));
    const f16x8 ph = __builtin_bit_cast(f16x8, pw);
    lacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, ph, lacc[nt], 0, 0, 0);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
      o[nt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh[dt], ph, o[nt][dt], 0, 0, 0);
  }
}

// Smallest K page scale used in a product with a masked (-inf) score: a scale of 0 (an all-zero
// page) would turn -inf into NaN; with this value the page's scores are 0 to within 1e-27.
constexpr float kMinKScale = 1.0e-30f;

// Eight e4m3 codes times a page scale (finite, 0 <= scale <= kMaxVScaleF16) -> eight fp16.  The
// scale is taken apart as 2^e * m with m in [1, 2): the scaled conversion applies 2^e (exact while
// the result is a normal fp16), a packed fp16 multiply applies m rounded to fp16.  Against
// code * scale in exact arithmetic the result is off by at most 2^-10 relative (two roundings to
// 11 bits), and below 2^-14 in magnitude by less than 2^-23 absolute.  A scale of 0 (or an fp32
// subnormal) gives zeros.
__device__ __forceinline__ u32x4 fp8x8_to_f16x8(uint32_t w0, uint32_t w1, float scale) {
  const uint32_t sb = __builtin_bit_cast(uint32_t, scale);
  const float pow2 = __builtin_bit_cast(float, sb & 0x7f800000u);
  const _Float16 mant = static_cast<_Float16>(__builtin_bit_cast(float, (sb & 0x007fffffu) | 0x3f800000u));
  const f16x2 m2 = {mant, mant};
  u32x4 r;
  r[0] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(static_cast<int>(w0), pow2, false) * m2);
  r[1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(static_cast<int>(w0), pow2, true) * m2);
  r[2] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(static_cast<int>(w1), pow2, false) * m2);
  r[3] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(static_cast<int>(w1), pow2, true) * m2);
  return r;
}

// ---- split path: items of many rows ------------------------------------------------------------
// For groups with many stacked rows.  The workgroup covers up to 64 * NTW rows of one (task, kv
// head); wavefront w owns rows row0 + w*16*NTW .. .  Each 32-token block is fetched from global
// memory once per workgroup -- every wavefront loads a quarter of it -- and is placed in LDS as
// ready-made MFMA operand images (K as bf16, V^T as fp16, fp8 widened on the way and V multiplied
// by its page scale) that all four wavefronts read (lane * 16 B, conflict free).  Two LDS buffers
// and one barrier per block.
template <int D>
constexpr int coop_lds_floats() {
  constexpr int img = 2 * (2 * (D / 32) + D / 16) * 256;
  return img > 4 * stage_floats<D>() ? img : 4 * stage_floats<D>();
}

template <int KV, int D, int NTW, bool TREE>
__device__ __forceinline__ void coop_item(const AttnArgs &p, const Shape &sh, const Item &cur, float *lds) {
  constexpr bool FP8 = KV == kFP8;
  constexpr int ESZ = FP8 ? 1 : 2;
  constexpr int TILE_BYTES = 16 * D * ESZ;
  constexpr int NKI = 2 * (D / 32);        // K operand images per block
  constexpr int NI = NKI + D / 16;         // all operand images per block (1 KiB each)
  constexpr int RAW = FP8 ? NI / 2 : NI;   // 1 KiB global loads per block
  constexpr int RK = FP8 ? NKI / 2 : NKI;  // of which K
  constexpr int PER = RAW / 4;             // global loads per wavefront and block
  static_assert(RAW % 4 == 0, "block must split evenly over four wavefronts");
  u32x4 *img = reinterpret_cast<u32x4 *>(lds);  // [buf][image][lane]

  const int lane = threadIdx.x & 63, m16 = lane & 15, jj = lane >> 4;
  const int w = uniform(threadIdx.x >> 6);
  const int g = cur.g;
  const int nblk = (cur.pg_count + 1) >> 1;
  const int rows = cur.qt_count * sh.G;
  const int row_base = cur.row0 + w * 16 * NTW;
  const bool has_rows = row_base < rows;
  const bool task_masked = (cur.flags & 1) != 0;
  const char *kpool = static_cast<const char *>(p.k_pool);
  const char *vpool = static_cast<const char *>(p.v_pool);
  const int k_lane_off = jj * 128 + (m16 & 7) * 16;
  const int v_lane_off = (jj & 1) * 256 + m16 * 16;

  RowState<D, NTW> st;
  load_rows<D, NTW>(p, sh, cur, row_base, st);
  f32x4 lacc[NTW];
#pragma unroll
  for (int nt = 0; nt < NTW; ++nt) lacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // Wavefront w fetches raw pieces w, w + 4, ... of the block (K pieces first, then V).
  struct Raw {
    u32x4 r[PER];
    float vs;
  };
  auto stage_load = [&](Raw &raw, const BlockMeta &bm) {
    const int64_t tile_a = (static_cast<int64_t>(bm.pid_a) * sh.page_tiles + g);
    const int64_t tile_b = (static_cast<int64_t>(bm.pid_b) * sh.page_tiles + g);
    const char *kp = kpool + (m16 < 8 ? tile_a : tile_b) * TILE_BYTES + k_lane_off;
    const char *vp = vpool + (jj < 2 ? tile_a : tile_b) * TILE_BYTES + v_lane_off;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = k * 4 + w;  // wave-uniform
      const char *src = idx < RK ? kp + (idx / (RK / 2)) * (TILE_BYTES / 2) + (idx % (RK / 2)) * 512
                                 : vp + (idx - RK) * 512;
      raw.r[k] = load_kv(src);
    }
    raw.vs = FP8 ? fminf(p.v_scale[(jj < 2 ? bm.pid_a : bm.pid_b) * sh.Hkv + g], kMaxVScaleF16) : 1.f;
  };
  auto stage_store = [&](const Raw &raw, int buf) {
    u32x4 *dst = img + buf * (NI * 64) + lane;
#pragma unroll
    for (int k = 0; k < PER; ++k) {
      const int idx = k * 4 + w;
      if (FP8) {
        if (idx < RK) {
          dst[(2 * idx) * 64] = __builtin_bit_cast(u32x4, fp8x8_to_bf16x8(raw.r[k][0], raw.r[k][1]));
          dst[(2 * idx + 1) * 64] = __builtin_bit_cast(u32x4, fp8x8_to_bf16x8(raw.r[k][2], raw.r[k][3]));
        } else {
          dst[(2 * idx) * 64] = fp8x8_to_f16x8(raw.r[k][0], raw.r[k][1], raw.vs);
          dst[(2 * idx + 1) * 64] = fp8x8_to_f16x8(raw.r[k][2], raw.r[k][3], raw.vs);
        }
      } else {
        dst[idx * 64] = raw.r[k];  // bf16 pool: K is a bf16 and V an fp16 operand image as stored
      }
    }
  };
  auto compute = [&](int b, const BlockMeta &bm) {
    if (!has_rows) return;
    const u32x4 *src = img + (b & 1) * (NI * 64) + lane;
    bf16x8 kf[2][D / 32];
    f16x8 vh[D / 16];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int s = 0; s < D / 32; ++s)
        kf[t][s] = __builtin_bit_cast(bf16x8, src[(t * (D / 32) + s) * 64]);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) vh[dt] = __builtin_bit_cast(f16x8, src[(NKI + dt) * 64]);
    const int valid_a = bm.vp_a & 127, valid_b = bm.vp_b & 127;
    float c = p.scale_log2;
    if (FP8) c *= fmaxf(p.k_scale[(jj < 2 ? bm.pid_a : bm.pid_b) * sh.Hkv + g], kMinKScale);
    block_math_f16<FP8, TREE, D, NTW>(st.qf, st.limit, st.qidx, st.dmask, st.o, st.m, lacc, kf, vh,
                                task_masked || valid_b == 0, jj < 2 ? valid_a : valid_b,
                                jj < 2 ? (bm.vp_a >> 7) : (bm.vp_b >> 7), c);
  };
  auto meta = [&](int b) { return load_block_meta(p.pg_rec, cur, b < nblk ? b : nblk - 1); };

  // LDS holds block b while it is computed; the pieces of block b+1 are requested before the
  // computation and moved to the other LDS buffer after it.
  Raw x;
  BlockMeta bm = meta(0);
  stage_load(x, bm);
  stage_store(x, 0);
  __syncthreads();
  for (int b = 0; b < nblk; ++b) {
    const bool more = b + 1 < nblk;  // uniform over the workgroup
    const BlockMeta nbm = meta(b + 1);
    if (more) stage_load(x, nbm);
    compute(b, bm);
    if (more) stage_store(x, (b + 1) & 1);
    bm = nbm;
    __syncthreads();
  }
  // The operand images are dead after the last barrier; the same LDS now serves the transposes.
  if (has_rows) {
    float m_out[NTW], l_out[NTW];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) {
      m_out[nt] = FP8 ? st.m[nt] : st.m[nt] * p.scale_log2;
      l_out[nt] = lacc[nt][0];
    }
    finish_rows<D, NTW, false>(p, sh, cur, row_base, st.o, m_out, l_out, st.qtok, lds + w * stage_floats<D>());
  }
}

// All items of the split path in one launch: lists 0 and 1 hold groups of up to 128 and up to 64 rows
// a span, lists 2 and 3 groups of up to 16 rows and private suffixes.
// kSplitLean: for launches of many short items, none in list 0: three workgroups a compute unit where the others hold two
// (heads of 64: five and three).
// kSplitTiles: for launches that leave the chip room: items of many rows go as row tiles of 16 NT, a workgroup each that
// splits the pages between its wavefronts, instead of one through LDS, whose blocks follow each other.  The tiles read the
// pages again, from L2 as far as the tiles of an item run on one XCD at one time: tile t of an item is workgroup item + t * items of
// its list, which is one XCD where the list's items are a multiple of 8.  Bytes past L2 over KV bytes, prompts of 24000 tokens
// under 63 or 64 rows, fp8: 120 items of 2 and of 4 kv heads 1.07 and 1.06, 96 of 8 kv heads 1.6, 188 of 2 kv heads of 64 2.1.
template <int KV, int D, int NT, bool TREE, SplitForm FORM>
__global__ __launch_bounds__(256, split_occupancy(D, FORM)) void spex_split_attn_kernel(AttnArgs p, Shape sh, SplitLists ls) {
  constexpr int kLds = FORM != kSplitTiles && coop_lds_floats<D>() > wave_fold_floats<D>() ? coop_lds_floats<D>() : wave_fold_floats<D>();
  __shared__ __attribute__((aligned(16))) float lds[kLds];
  const ListPos at = list_of(ls, static_cast<int>(blockIdx.x));
  const int tile = FORM == kSplitTiles ? at.local / at.n_items : 0;
  Item cur = load_item(at.items, at.local - tile * at.n_items);
  cur.row0 += tile * 16 * NT;
  if (cur.pg_count == 0 || (FORM == kSplitTiles && cur.row0 >= cur.qt_count * sh.G)) return;  // whole workgroup: padding item, or no such tile
  if (FORM == kSplitFull && at.k == 0)
    coop_item<KV, D, 2, TREE>(p, sh, cur, lds);
  else if (FORM != kSplitTiles && at.k <= 1)
    coop_item<KV, D, 1, TREE>(p, sh, cur, lds);
  else
    wave_item<KV, D, NT, TREE, true, false, NT == 1 && FORM != kSplitLean, KV == kFP8 && FORM == kSplitTiles>(
        p, sh, cur, lds, at.k <= 1 ? kMaxVScaleF16 : __builtin_huge_valf());
}

// The same in launches of their own where there are items enough to fill the chip with a wavefront each (the
// rule and both sides' times stand with the planner's item lengths).
template <int KV, int D, int NT, bool SUFFIX, bool TREE>
__global__ __launch_bounds__(256, 2) void spex_wave_attn_kernel(AttnArgs p, Shape sh) {
  __shared__ __attribute__((aligned(16))) float lds[4 * stage_floats<D>()];
  const int item = uniform(static_cast<int>(blockIdx.x) * 4 + static_cast<int>(threadIdx.x >> 6));
  if (item >= p.n_items) return;
  const Item cur = load_item(p.items, item);
  if (cur.pg_count == 0) return;  // padding item
  wave_item<KV, D, NT, TREE, false, SUFFIX, NT == 1>(p, sh, cur, lds);
}

template <int KV, int D, int NTW, bool TREE>
__global__ __launch_bounds__(256, 2) void spex_coop_attn_kernel(AttnArgs p, Shape sh) {
  __shared__ __attribute__((aligned(16))) float lds[coop_lds_floats<D>()];
  const Item cur = load_item(p.items, static_cast<int>(blockIdx.x));
  if (cur.pg_count == 0) return;  // padding item (whole workgroup)
  coop_item<KV, D, NTW, TREE>(p, sh, cur, lds);
}

// ---- tree-walk kernel: one workgroup carries a block of query rows from the root to the leaves --
// A work item is a row block (up to NW = 4 or 8 wavefronts x 16 * NTW rows of the requested nodes below one
// root, neighbours in the tree next to each other) and a kv head.  Its block list covers every
// page on the rows' paths exactly once, each block with the range of rows whose path contains it.
// Phase 1 walks the blocks whose rows span several wavefronts: the workgroup fetches each block
// once into LDS operand images (as items of many rows do on the split path) and every wavefront contracts it
// with the row tiles inside the range.  Phase 2: every wavefront streams the blocks that only its
// own rows need straight into registers.  The softmax state (m, l, o) of a row stays in registers
// from the first block to the last, so the only global writes are the finished output rows.
struct WalkBlock {
  int pid_a, vp_a, pid_b, vp_b, rows, flags;
  float ka, kb, va, vb;  // fp8: K and V scales of pages a and b for the item's kv head; else unused
};

__device__ __forceinline__ float sload_f(const float *base, int64_t idx) {
  typedef const float __attribute__((address_space(4))) const_f32;
  return ((const_f32 *)(uintptr_t)base)[idx];
}

// The record of a block and, for fp8, the page scales it will need.  Workgroups whose whole
// block list fits (walk_rec_cap blocks) copy it into LDS once, at the start, with ordinary vector
// loads, and read records from there: a scalar load inside the loop misses the scalar cache every
// other record and, because scalar loads return out of order, the next LDS wait of the wavefront
// becomes a wait for that miss -- measured at ~1.4 us per block.  Longer lists fall back to the
// scalar path, requested one or two blocks ahead.
// Eight wavefronts on a path in halves, one workgroup a compute unit: records of up to 1024 blocks (32 thousand
// tokens; fp8 with its scales 768) besides the images.  With 256, 9 prompts of 10000 tokens took 1.5 us a step where
// those of 3000 took 1.06 (bf16 239 -> 210 us, fp8 242 -> 150; head dim 64, 100 prompts of 12000: 228 -> 156, fp8
// 307 -> 150).  Whole paths keep 256: two workgroups a compute unit are bound by memory, and with more records in LDS
// 80 prompts of 12000 tokens took 830 us instead of 621.
constexpr int walk_rec_cap(int kv, int nw, int ks) {
  return ks == 2 && nw == 8 ? (kv == kFP8 ? 768 : 1024) : 256;
}

template <bool FP8>
__device__ __forceinline__ WalkBlock load_walk_block(const WalkArgs &p, int idx, int g, int Hkv,
                                                     bool in_lds, const int32_t *rec, const float *scl,
                                                     int first) {
  WalkBlock b;
  if (in_lds) {
    const int at = uniform(idx) - first;
    const u32x4 lo = *reinterpret_cast<const u32x4 *>(rec + at * 8);
    const u32x2 hi = *reinterpret_cast<const u32x2 *>(rec + at * 8 + 4);
    b.pid_a = uniform(static_cast<int>(lo[0]));
    b.vp_a = uniform(static_cast<int>(lo[1]));
    b.pid_b = uniform(static_cast<int>(lo[2]));
    b.vp_b = uniform(static_cast<int>(lo[3]));
    b.rows = uniform(static_cast<int>(hi[0]));
    b.flags = uniform(static_cast<int>(hi[1]));
    if (FP8) {
      const f32x4 sc = *reinterpret_cast<const f32x4 *>(scl + at * 4);
      b.ka = fmaxf(sc[0], kMinKScale);
      b.kb = fmaxf(sc[1], kMinKScale);
      b.va = fminf(sc[2], kMaxVScaleF16);
      b.vb = fminf(sc[3], kMaxVScaleF16);
    } else {
      b.ka = b.kb = b.va = b.vb = 1.f;
    }
    return b;
  }
  const int64_t r = static_cast<int64_t>(uniform(idx)) * 8;
  b.pid_a = sload(p.blocks, r + 0);
  b.vp_a = sload(p.blocks, r + 1);
  b.pid_b = sload(p.blocks, r + 2);
  b.vp_b = sload(p.blocks, r + 3);
  b.rows = sload(p.blocks, r + 4);
  b.flags = sload(p.blocks, r + 5);
  if (FP8) {
    const int64_t ia = static_cast<int64_t>(b.pid_a) * Hkv + g, ib = static_cast<int64_t>(b.pid_b) * Hkv + g;
    b.ka = fmaxf(sload_f(p.k_scale, ia), kMinKScale);
    b.kb = fmaxf(sload_f(p.k_scale, ib), kMinKScale);
    b.va = fminf(sload_f(p.v_scale, ia), kMaxVScaleF16);
    b.vb = fminf(sload_f(p.v_scale, ib), kMaxVScaleF16);
  } else {
    b.ka = b.kb = b.va = b.vb = 1.f;
  }
  return b;
}

// Scores of one 32-token block for row tiles T0 .. T1 - 1 of the wavefront: S^T = K Q^T (see
// block_math for the operand layout).
template <int T0, int T1, int D, int NT>
__device__ __forceinline__ void walk_scores_of(const bf16x8 (&qf)[NT][D / 32], const bf16x8 (&kf)[2][D / 32],
                                               f32x4 (&sa)[NT], f32x4 (&sb)[NT]) {
#pragma unroll
  for (int nt = T0; nt < T1; ++nt) {
    f32x4 a = {0.f, 0.f, 0.f, 0.f}, b = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
      a = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[0][s], qf[nt][s], a, 0, 0, 0);
      b = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[1][s], qf[nt][s], b, 0, 0, 0);
    }
    sa[nt] = a;
    sb[nt] = b;
  }
}

// Online softmax and O^T += V^T P^T for the same tiles; P rounded to fp16, row sums by MFMA
// against ones (see block_math_f16).  Rows outside [lo, hi) see nothing of the block.
// One path with two branches for all tiles of the wavefront -- masks, which change scores only, and a
// reference that moves -- so that the tiles' weights and MFMAs form one run of instructions: with
// a branch per tile the weights of one tile were made while the matrix cores idled.
template <bool FP8, bool TREE, int T0, int T1, int D, int NT>
__device__ __forceinline__ void walk_softmax_pv_of(const int (&limit)[NT], const int (&qidx)[NT],
                                                const uint32_t (&dmask)[NT], f32x4 (&o)[NT][D / 16],
                                                float (&m)[NT], f32x4 (&lacc)[NT], f32x4 (&sa)[NT],
                                                f32x4 (&sb)[NT], const f16x8 (&vh)[D / 16], bool tok_masked,
                                                int valid_l, int pos_l, float c, float slack, int lo,
                                                int hi, int rows) {
  // With one tile the block is known to touch it; the branch keeps the scores' instructions and the weights'
  // apart, without it the fp8 kernel takes 178 registers instead of 162 and two workgroups run on a
  // compute unit instead of three (150 trees of 6 branches, 600 workgroups, 52.8 -> 38.5 us).
  if (NT == 1 && (hi <= 0 || lo >= 16)) return;
  const int lane = threadIdx.x & 63, m16 = lane & 15, jj = lane >> 4;
  const _Float16 one = static_cast<_Float16>(1.0f);
  const f16x8 ones = {one, one, one, one, one, one, one, one};
  // Scores stay raw; scale and subtraction of the reference fuse into one FMA per score.  With
  // one scale for the whole path (bf16 KV) the reference m is kept on raw scores; with a scale
  // per page (fp8 KV) it is kept in scaled units (log2 e folded in), and the largest scaled score
  // of the lane is c * the largest raw one (c > 0, and rounding is monotonic).
  // Tile rows past the wavefront's last one hold zero queries and are not written: they need no mask.
  if (tok_masked || lo > 16 * T0 || hi < min(rows, 16 * T1)) {  // wave-uniform
#pragma unroll
    for (int nt = T0; nt < T1; ++nt) {
      const int row = nt * 16 + m16;
      const bool row_in = row >= lo && row < hi;
      uint32_t vm = 0xffu;
      int vis = valid_l - 8 * (jj & 1);  // tokens of the lane's 8 that exist
      if (TREE) {
        // Draft tree: positions below base = T - q_len are visible, position base + k iff bit k of
        // the row's mask is set.  The lane's 8 tokens start at relative position rel; shifting
        // {mask, 32 ones} right by rel + 32 puts their visibility into the low 8 bits.
        const int base = limit[nt] - 1 - qidx[nt];
        const int sh = pos_l + 8 * (jj & 1) - base + 32;
        const uint64_t bits = (static_cast<uint64_t>(dmask[nt]) << 32) | 0xffffffffull;
        vm = sh <= 0 ? 0xffu : (sh >= 64 ? 0u : static_cast<uint32_t>(bits >> sh) & 0xffu);
      } else {
        vis = min(vis, limit[nt] - pos_l - 8 * (jj & 1));
      }
      if (!tok_masked) vis = 8;  // a block that its rows see whole: only the row range counts
      if (TREE && !tok_masked) vm = 0xffu;
      vis = row_in ? vis : 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sa[nt][i] = i < vis && (!TREE || ((vm >> i) & 1u)) ? sa[nt][i] : kNegInf;
        sb[nt][i] = 4 + i < vis && (!TREE || ((vm >> (4 + i)) & 1u)) ? sb[nt][i] : kNegInf;
      }
    }
  }
  // Lazy reference: m is the value the row's weights are taken relative to, not its exact
  // running maximum.  It moves (and o and l are rescaled) only when a score of the row exceeds it
  // by more than `slack` (2^8 in weight); until then weights are at most 2^8, which fp16 and
  // the fp32 sums hold.  The decision is taken per row from the row's own scores, so a row's
  // result does not depend on its neighbours in the tile; most blocks skip the cross-lane
  // maximum and the rescaling altogether.  m starts at kWalkMInit (finite, far below any score).
  float mx[NT];
  bool over = false;
#pragma unroll
  for (int nt = T0; nt < T1; ++nt) {
    const float raw = fmaxf(fmaxf(fmaxf(sa[nt][0], sa[nt][1]), fmaxf(sa[nt][2], sa[nt][3])),
                            fmaxf(fmaxf(sb[nt][0], sb[nt][1]), fmaxf(sb[nt][2], sb[nt][3])));
    mx[nt] = FP8 ? raw * c : raw;
    over = over || mx[nt] > m[nt] + slack;
  }
  if (__any(over)) {
#pragma unroll
    for (int nt = T0; nt < T1; ++nt) {
      const float rmax = row_group_max(mx[nt]);
      const float m_new = rmax > m[nt] + slack ? rmax : m[nt];
      const float alpha = fast_exp2(FP8 ? m[nt] - m_new : (m[nt] - m_new) * c);
      m[nt] = m_new;
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) o[nt][dt] *= alpha;
      lacc[nt] *= alpha;
    }
  }
#pragma unroll
  for (int nt = T0; nt < T1; ++nt) {
    const float mc = FP8 ? m[nt] : m[nt] * c;
    u32x4 pw;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float x0 = i < 2 ? sa[nt][2 * i] : sb[nt][2 * i - 4], x1 = i < 2 ? sa[nt][2 * i + 1] : sb[nt][2 * i - 3];
      pw[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{fast_exp2(__builtin_fmaf(x0, c, -mc)),
                                                                         fast_exp2(__builtin_fmaf(x1, c, -mc))}, f16x2));
    }
    const f16x8 ph = __builtin_bit_cast(f16x8, pw);
    lacc[nt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(ones, ph, lacc[nt], 0, 0, 0);
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
      o[nt][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vh[dt], ph, o[nt][dt], 0, 0, 0);
  }
}

// All row tiles of the wavefront together, or (BY_TILE) one after the other, without those that no row
// of the block lies in: the planner chooses by how many of them there are.  One kernel cannot hold both forms
// (the accumulators of either side of the branch are then other registers: 130 spilled).
template <bool BY_TILE, int D, int NT, int T = 0>
__device__ __forceinline__ void walk_scores(const bf16x8 (&qf)[NT][D / 32], const bf16x8 (&kf)[2][D / 32],
                                            f32x4 (&sa)[NT], f32x4 (&sb)[NT], int lo, int hi) {
  if constexpr (!BY_TILE) {
    walk_scores_of<0, NT, D, NT>(qf, kf, sa, sb);
  } else if constexpr (T < NT) {
    if (lo < 16 * T + 16 && hi > 16 * T) walk_scores_of<T, T + 1, D, NT>(qf, kf, sa, sb);
    walk_scores<BY_TILE, D, NT, T + 1>(qf, kf, sa, sb, lo, hi);
  }
}
template <bool BY_TILE, bool FP8, bool TREE, int D, int NT, int T = 0>
__device__ __forceinline__ void walk_softmax_pv(const int (&limit)[NT], const int (&qidx)[NT],
                                                const uint32_t (&dmask)[NT], f32x4 (&o)[NT][D / 16],
                                                float (&m)[NT], f32x4 (&lacc)[NT], f32x4 (&sa)[NT],
                                                f32x4 (&sb)[NT], const f16x8 (&vh)[D / 16], bool tok_masked,
                                                int valid_l, int pos_l, float c, float slack, int lo,
                                                int hi, int rows) {
  if constexpr (!BY_TILE) {
    walk_softmax_pv_of<FP8, TREE, 0, NT, D, NT>(limit, qidx, dmask, o, m, lacc, sa, sb, vh, tok_masked, valid_l, pos_l,
                                                c, slack, lo, hi, rows);
  } else if constexpr (T < NT) {
    if (lo < 16 * T + 16 && hi > 16 * T)
      walk_softmax_pv_of<FP8, TREE, T, T + 1, D, NT>(limit, qidx, dmask, o, m, lacc, sa, sb, vh, tok_masked, valid_l,
                                                     pos_l, c, slack, lo, hi, rows);
    walk_softmax_pv<BY_TILE, FP8, TREE, D, NT, T + 1>(limit, qidx, dmask, o, m, lacc, sa, sb, vh, tok_masked, valid_l,
                                                      pos_l, c, slack, lo, hi, rows);
  }
}

// Normalise and store the finished rows of one wavefront.  As in finish_rows the tile goes through
// a wave-private LDS area so that every store instruction writes whole 4 * D byte rows.
template <int D, int NT>
__device__ __forceinline__ void walk_write_rows(float *out, float *lse, const Shape &sh, int g, int rows,
                                                f32x4 (&o)[NT][D / 16], const float (&m_log2)[NT],
                                                const f32x4 (&lacc)[NT], const int (&qtok)[NT], float *my) {
  constexpr int kRowPad = D + 4;
  constexpr int kLanesPerRow = D / 4;
  constexpr int kRowsPerInst = 64 / kLanesPerRow;
  const int lane = threadIdx.x & 63, m16 = lane & 15, jj = lane >> 4;
  const int sub = lane / kLanesPerRow, piece = lane % kLanesPerRow;
  const int G = sh.G;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int r0w = nt * 16;
    if (r0w >= rows) break;  // wave-uniform
    const bool row_ok = r0w + m16 < rows;
    const float l = lacc[nt][0];
    const float inv = 1.0f / l;
    const int64_t dst_row = static_cast<int64_t>(qtok[nt]) * sh.Hq + g * G + (r0w + m16) % G;
    if (row_ok && jj == 0 && lse) lse[dst_row] = (m_log2[nt] + __builtin_log2f(l)) * 0.6931471805599453f;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt)
      *reinterpret_cast<f32x4 *>(my + m16 * kRowPad + dt * 16 + jj * 4) = o[nt][dt] * inv;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int i = 0; i < 16 / kRowsPerInst; ++i) {
      const int row = i * kRowsPerInst + sub;
      const f32x4 v = *reinterpret_cast<const f32x4 *>(my + row * kRowPad + piece * 4);
      const int lo32 = __shfl(static_cast<int>(dst_row & 0xffffffff), row);
      const int hi32 = __shfl(static_cast<int>(dst_row >> 32), row);
      const int64_t drow = (static_cast<int64_t>(hi32) << 32) | static_cast<uint32_t>(lo32);
      if (r0w + row < rows) *reinterpret_cast<f32x4 *>(out + drow * D + piece * 4) = v;
    }
  }
}

// KS = 1: wavefront w holds rows w * C .. of the row block.  KS = 2: the lists are made for LW = NW / 2
// wavefronts of rows (NW = 8: the lists of four wavefronts, where the planner chooses halves; NW = 4: two,
// only where asked for); wavefronts w and w + LW hold the same rows and split the row block's path between them -- shared blocks alternate between the two halves of the workgroup
// (two blocks per barrier, each staged by the pair that computes on it), a list wavefront's private
// blocks alternate likewise -- and at the end the upper pair hands its softmax state to the lower
// one through LDS.  Per block a wavefront then works on twice the rows, so half as many operand
// images cross the LDS per row, and a row block's longest path takes half as many steps.
//
// CUT: for requests of more rows than a row block holds, whose first row blocks see nothing of the request's last
// tokens: blocks at the end of the lists that none of the workgroup's rows sees are left out (128 queries of 4 heads, four
// row blocks on paths of 36 blocks: 1.5 blocks on average, 1505 -> 1477 us; 256 queries on a prompt of 100: 401 -> 380).
// A kernel of its own, because the test alone, where nothing can be left out, made short launches slower (512
// workgroups of 1 to 3 blocks 15.9 -> 16.4 us).
template <int KV, int D, int NTW, int NW, bool TREE, int KS = 1, bool BY_TILE = false, bool CUT = false>
__global__ __launch_bounds__(64 * NW, (NW == 4 && NTW <= 2) ? 2 : 1) void spex_tree_walk_kernel(WalkArgs p, Shape sh) {
  constexpr bool FP8 = KV == kFP8;
  constexpr int ESZ = FP8 ? 1 : 2;
  constexpr int TILE_BYTES = 16 * D * ESZ;
  constexpr int C = 16 * NTW;              // rows per wavefront
  constexpr int NKI = 2 * (D / 32);        // K operand images per block
  constexpr int NI = NKI + D / 16;         // all operand images per block (1 KiB each)
  constexpr int RAW = FP8 ? NI / 2 : NI;   // 1 KiB global loads per block
  constexpr int RK = FP8 ? NKI / 2 : NKI;  // of which K
  static_assert(KS == 1 || KS == 2, "the path is split between the two halves of the workgroup");
  constexpr int LW = NW / KS;               // wavefronts the lists were made for (each holds C rows)
  constexpr int PER = (RAW + LW - 1) / LW;  // global loads per wavefront and block in the shared phase
  constexpr bool kEven = RAW % LW == 0;     // else the last wavefronts have no piece to fetch
  // When K and V each split evenly over the wavefronts, a wavefront's first KPER pieces are K and
  // the others V whatever its index, so the widening code is chosen at compile time instead of
  // being run for every piece and selected away.
  constexpr bool kSplitKV = RK % LW == 0 && (RAW - RK) % LW == 0;
  constexpr int KPER = kSplitKV ? RK / LW : 0;
  constexpr int kItemInts = LW <= 4 ? 16 : 32;
  constexpr int kImgFloats = NI * 64 * 4;
  // KS = 2: what a wavefront of the upper pair hands over at the end: o, l (as accumulator) and m
  constexpr int kFoldWaveFloats = NTW * (D / 16) * 256 + NTW * 256 + NTW * 64;
  // output staging of the wavefronts that write rows (all, or the lower pair), then the hand-over area
  constexpr int kTailFloats = LW * stage_floats<D>() + (KS == 2 ? LW * kFoldWaveFloats : 0);
  constexpr int kLdsFloats = 2 * KS * kImgFloats > kTailFloats ? 2 * KS * kImgFloats : kTailFloats;
  __shared__ __attribute__((aligned(16))) float lds[kLdsFloats];
  constexpr int kRecCap = walk_rec_cap(KV, NW, KS);
  __shared__ __attribute__((aligned(16))) int32_t rec_lds[kRecCap * 8];
  __shared__ __attribute__((aligned(16))) float scl_lds[FP8 ? kRecCap * 4 : 4];
  u32x4 *img = reinterpret_cast<u32x4 *>(lds);  // [buf][image][lane]

  const int lane = threadIdx.x & 63, m16 = lane & 15, jj = lane >> 4;
  const int w = uniform(threadIdx.x >> 6);
  const int64_t ir = static_cast<int64_t>(blockIdx.x) * kItemInts;
  const int g = sload(p.items, ir + 0);
  const int blk_begin = sload(p.items, ir + 1);
  int n_shared = sload(p.items, ir + 2);
  // per wavefront: private blocks | room << 16; a wavefront's records are followed by the unused
  // part of its room, so n_all spans records that no wavefront walks
  const int rw = KS == 1 ? w : w % LW;  // the list wavefront whose rows this wavefront holds
  const int ks = KS == 1 ? 0 : w / LW;  // which part of the path it walks
  int n_all = n_shared, n_priv = 0, priv_begin = blk_begin + n_shared;
#pragma unroll
  for (int v = 0; v < LW; ++v) {
    const uint32_t packed = static_cast<uint32_t>(sload(p.items, ir + 3 + v));
    const int npv = static_cast<int>(packed & 0xffffu), room = static_cast<int>(packed >> 16);
    n_all += room;
    n_priv = v == rw ? npv : n_priv;
    priv_begin += v < rw ? room : 0;
  }
  if (n_all == 0) return;  // padding item (whole workgroup)
  const bool rec_in_lds = n_all <= kRecCap;  // uniform over the workgroup
  if (rec_in_lds) {
    const u32x4 *src = reinterpret_cast<const u32x4 *>(p.blocks + static_cast<int64_t>(blk_begin) * 8);
    for (int i = threadIdx.x; i < n_all * 2; i += 64 * NW) reinterpret_cast<u32x4 *>(rec_lds)[i] = src[i];
    if (FP8) {
      __syncthreads();
      for (int i = threadIdx.x; i < n_all * 4; i += 64 * NW) {
        const int page = rec_lds[(i >> 2) * 8 + ((i & 1) ? 2 : 0)];
        scl_lds[i] = ((i & 2) ? p.v_scale : p.k_scale)[static_cast<int64_t>(page) * sh.Hkv + g];
      }
    }
    __syncthreads();
  }
  const int qt_begin = sload(p.items, ir + 3 + LW + rw);
  const int qt_count = sload(p.items, ir + 3 + 2 * LW + rw);
  const int rows = qt_count * sh.G;
  // CUT: where the paths of the workgroup's rows end for them, as a maximum over the lanes (with masks an upper
  // bound: 32 drafts).  The workgroup's entries follow each other from its first wavefront's on.
  int seen_end = 0;
  if constexpr (CUT) {
    int entries = 0;
#pragma unroll
    for (int v = 0; v < LW; ++v) entries += sload(p.items, ir + 3 + 2 * LW + v);
    const int32_t *rec = p.qt_rec + 2 * static_cast<int64_t>(sload(p.items, ir + 3 + LW));
    for (int i = lane; i < entries; i += 64) seen_end = max(seen_end, rec[2 * i + 1] + (TREE ? 31 : 0));
  }
  const bool has_rows = rows > 0;
  const char *kpool = static_cast<const char *>(p.k_pool);
  const char *vpool = static_cast<const char *>(p.v_pool);
  const int k_lane_off = jj * 128 + (m16 & 7) * 16;
  const int v_lane_off = (jj & 1) * 256 + m16 * 16;

  // how far a score may exceed a row's softmax reference before the reference moves (log2 units: 8)
  const float slack = FP8 ? 8.f : 8.f / p.scale_log2;
  // ---- rows of this wavefront
  bf16x8 qf[NTW][D / 32];
  int limit[NTW], qtok[NTW], qidx[NTW];
  uint32_t dmask[NTW];
  f32x4 o[NTW][D / 16], lacc[NTW];
  float m[NTW];
#pragma unroll
  for (int nt = 0; nt < NTW; ++nt) {
    const int r = nt * 16 + m16;
    limit[nt] = INT_MAX;
    qtok[nt] = 0;
    qidx[nt] = 0;
    dmask[nt] = 0;
    m[nt] = kWalkMInit;
    lacc[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < D / 16; ++dt) o[nt][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (r < rows) {
      const int2 qr = *reinterpret_cast<const int2 *>(p.qt_rec + 2 * (qt_begin + r / sh.G));
      qtok[nt] = qr.x;
      limit[nt] = qr.y;
      if (TREE) {
        const int2 dm = *reinterpret_cast<const int2 *>(p.qt_mask + 2 * qr.x);
        qidx[nt] = dm.x;
        dmask[nt] = static_cast<uint32_t>(dm.y);
      }
      const uint16_t *qp = static_cast<const uint16_t *>(p.q) +
                           (static_cast<int64_t>(qr.x) * sh.Hq + g * sh.G + r % sh.G) * D + jj * 8;
#pragma unroll
      for (int s = 0; s < D / 32; ++s)
        qf[nt][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4 *>(qp + s * 32));
    } else {
#pragma unroll
      for (int s = 0; s < D / 32; ++s) qf[nt][s] = __builtin_bit_cast(bf16x8, u32x4{0, 0, 0, 0});
    }
  }

  if constexpr (CUT) {  // every wavefront cuts the shared list alike
    auto unseen = [&](int idx) {
      const int32_t *r = rec_lds + (uniform(idx) - blk_begin) * 8;
      const int64_t far = static_cast<int64_t>(uniform(idx)) * 8;
      const int flags = rec_in_lds ? uniform(r[5]) : sload(p.blocks, far + 5);
      if (!(flags & 1)) return false;
      const int pos = (rec_in_lds ? uniform(r[1]) : sload(p.blocks, far + 1)) >> 7;
      return !__any(seen_end > pos);
    };
    while (n_shared > 0 && unseen(blk_begin + n_shared - 1)) --n_shared;
    while (n_priv > 0 && unseen(priv_begin + n_priv - 1)) --n_priv;
  }
  if (KS == 2) n_priv = (n_priv + 1 - ks) >> 1;  // private blocks ks, ks + 2, .. of the list wavefront

  // The two phases run in either order (the online softmax does not care).  The shared phase is
  // bound by the matrix cores and LDS, the private phase by memory; workgroups that start together
  // would all be in the same phase at the same time, so every other pair of workgroups of an XCD
  // (workgroup n runs on XCD n % 8; the pair n, n + 8 are row blocks of one root and kv head when
  // a root has several, and stay in step so that one finds the other's shared blocks in L2),
  // alternating again with every round of 256, takes its private blocks first: the loop below
  // then runs twice, one phase per turn.  Not with four row tiles per wavefront (registers).
  constexpr bool kStagger = NTW <= 2 && (KS == 1 || NW == 8);
  const bool private_first = kStagger && (((blockIdx.x >> 4) ^ (blockIdx.x >> 8)) & 1) != 0;
#pragma nounroll
  for (int ph = 0; ph < (kStagger ? 2 : 1); ++ph) {
  const bool run_shared = !kStagger || (ph == 0) != private_first;
  const bool run_private = !kStagger || (ph == 0) == private_first;
  // ---- phase 1: blocks shared by several wavefronts, through LDS
  if (run_shared && n_shared > 0) {
    struct Raw {
      u32x4 r[PER];
      float vs;
    };
    // A block that another row block reads too (flag bit 1) is loaded with the ordinary cache
    // policy, so that the second reader finds it in the L2 of the XCD both run on; everything
    // else is streamed.
    auto stage_load = [&](Raw &raw, const WalkBlock &bm) {
      const int64_t tile_a = (static_cast<int64_t>(bm.pid_a) * sh.page_tiles + g);
      const int64_t tile_b = (static_cast<int64_t>(bm.pid_b) * sh.page_tiles + g);
      const char *kp = kpool + (m16 < 8 ? tile_a : tile_b) * TILE_BYTES + k_lane_off;
      const char *vp = vpool + (jj < 2 ? tile_a : tile_b) * TILE_BYTES + v_lane_off;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const bool is_k = kSplitKV ? k < KPER : k * LW + rw < RK;
        const int idx = kSplitKV ? (k < KPER ? k * LW + rw : RK + (k - KPER) * LW + rw) : k * LW + rw;  // wave-uniform
        if (!kEven && idx >= RAW) continue;
        const char *src = is_k ? kp + (idx / (RK / 2)) * (TILE_BYTES / 2) + (idx % (RK / 2)) * 512
                               : vp + (idx - RK) * 512;
        raw.r[k] = (bm.flags & 2) ? *reinterpret_cast<const u32x4 *>(src) : load_kv(src);
      }
      raw.vs = jj < 2 ? bm.va : bm.vb;
    };
    auto stage_store = [&](const Raw &raw, int buf) {
      u32x4 *dst = img + (buf * KS + ks) * (NI * 64) + lane;
#pragma unroll
      for (int k = 0; k < PER; ++k) {
        const bool is_k = kSplitKV ? k < KPER : k * LW + rw < RK;
        const int idx = kSplitKV ? (k < KPER ? k * LW + rw : RK + (k - KPER) * LW + rw) : k * LW + rw;
        if (!kEven && idx >= RAW) continue;
        if (FP8) {
          if (is_k) {
            dst[(2 * idx) * 64] = __builtin_bit_cast(u32x4, fp8x8_to_bf16x8(raw.r[k][0], raw.r[k][1]));
            dst[(2 * idx + 1) * 64] = __builtin_bit_cast(u32x4, fp8x8_to_bf16x8(raw.r[k][2], raw.r[k][3]));
          } else {
            dst[(2 * idx) * 64] = fp8x8_to_f16x8(raw.r[k][0], raw.r[k][1], raw.vs);
            dst[(2 * idx + 1) * 64] = fp8x8_to_f16x8(raw.r[k][2], raw.r[k][3], raw.vs);
          }
        } else {
          dst[idx * 64] = raw.r[k];  // bf16 pool: K is a bf16 and V an fp16 operand image as stored
        }
      }
    };
    auto compute = [&](int b, const WalkBlock &bm) {
      const int lo = (bm.rows & 0xffff) - rw * C, hi = (bm.rows >> 16) - rw * C;
      if (!has_rows || hi <= 0 || lo >= C) return;  // wave-uniform: none of this wavefront's rows
      const u32x4 *src = img + ((b & 1) * KS + ks) * (NI * 64) + lane;
      const float c = p.scale_log2 * (jj < 2 ? bm.ka : bm.kb);
      f32x4 sa[NTW], sb[NTW];
      {
        bf16x8 kf[2][D / 32];
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int s = 0; s < D / 32; ++s)
            kf[t][s] = __builtin_bit_cast(bf16x8, src[(t * (D / 32) + s) * 64]);
        walk_scores<BY_TILE, D, NTW>(qf, kf, sa, sb, lo, hi);
      }
      // The V images are fetched only now, into the registers the K images have left, and their
      // LDS latency passes under the softmax arithmetic.
      __builtin_amdgcn_sched_barrier(0);
      f16x8 vh[D / 16];
#pragma unroll
      for (int dt = 0; dt < D / 16; ++dt) vh[dt] = __builtin_bit_cast(f16x8, src[(NKI + dt) * 64]);
      walk_softmax_pv<BY_TILE, FP8, TREE, D, NTW>(limit, qidx, dmask, o, m, lacc, sa, sb, vh, (bm.flags & 1) != 0,
                                   (jj < 2 ? bm.vp_a : bm.vp_b) & 127, (jj < 2 ? bm.vp_a : bm.vp_b) >> 7,
                                   c, slack, lo, hi, rows);
    };
    auto meta = [&](int b) {
      return load_walk_block<FP8>(p, blk_begin + (b < n_shared ? b : n_shared - 1), g, sh.Hkv, rec_in_lds,
                                  rec_lds, scl_lds, blk_begin);
    };

    // Software pipeline, PF blocks deep: while block c is computed from one LDS buffer, blocks
    // c+1 .. c+PF-1 are already in (or on their way to) registers, block c+1 moves to the other
    // LDS buffer after the computation, and the global loads of block c+PF are issued.  The loads
    // are unconditional (indices past the end repeat the last block) because a load issued on
    // one path only would make every later wait a wait for all outstanding loads.  (PF = 4 was
    // measured for one row tile per wavefront and for fp8 with two, where the registers allow it:
    // no gain.)
    constexpr int PFS = NTW == 1 || FP8 ? 2 : 1;
    if (KS == 2) {
      // Two blocks per barrier: step s holds blocks 2 s (lower pair of wavefronts) and 2 s + 1
      // (upper pair); each pair stages and computes its own.  With an odd number of blocks the upper pair's last
      // step only moves a copy of the last block.  Loads two steps ahead where the registers allow it (one row
      // tile, or fp8): 2 to 3 % on paths of 1500 tokens and more, nothing on short ones.
      const int n_steps = (n_shared + 1) >> 1;
      Raw x[PFS];
      WalkBlock bmq[PFS];
#pragma unroll
      for (int k = 0; k < PFS; ++k) {
        bmq[k] = meta(2 * k + ks);
        stage_load(x[k], bmq[k]);
      }
      stage_store(x[0], 0);
      __syncthreads();
      for (int st = 0; st < n_steps; st += PFS) {
#pragma unroll
        for (int k = 0; k < PFS; ++k) {
          const int c = st + k;
          if (k > 0 && c >= n_steps) break;  // uniform; leaves the loop
          const WalkBlock cur = bmq[k];
          bmq[k] = meta(2 * (c + PFS) + ks);
          stage_load(x[k], bmq[k]);
          if (2 * c + ks < n_shared) compute(c, cur);
          stage_store(x[(k + 1) % PFS], (c + 1) & 1);
          __syncthreads();
        }
      }
    }
    constexpr int PF = 2;
    Raw x[PF];
    WalkBlock bmq[PF];
    if (KS == 1) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        bmq[k] = meta(k);
        stage_load(x[k], bmq[k]);
      }
      stage_store(x[0], 0);
      __syncthreads();
    }
    for (int b = 0; KS == 1 && b < n_shared; b += PF) {
#pragma unroll
      for (int k = 0; k < PF; ++k) {
        const int c = b + k;             // block computed in this step; x[k] is free again
        const WalkBlock cur = bmq[k];
        bmq[k] = meta(c + PF);
        stage_load(x[k], bmq[k]);
        // no early exit from the group of PF steps: a step past the end only moves (clamped)
        // data, so that every path through the loop body issues and waits for the same loads
        if (c < n_shared) compute(c, cur);
        // Unconditional: after the last block this stores a copy of that block (the loads are
        // clamped) into the buffer nobody reads any more.  A store skipped on one path would leave
        // its loads unwaited there, and the compiler would then drain every outstanding load at
        // the top of the loop -- the prefetch of the next block included.
        stage_store(x[(k + 1) % PF], (c + 1) & 1);
        __syncthreads();
      }
    }
  }

  // ---- phase 2: blocks of this wavefront alone, straight into registers
  if (run_private && has_rows && n_priv > 0) {
    constexpr int NK = FP8 ? D / 64 : D / 32;  // 128-bit loads per K half-tile
    constexpr int NV = FP8 ? D / 32 : D / 16;
    auto issue_k = [&](u32x4 (&kr)[2][NK], const WalkBlock &bm) {
      const int64_t tile_a = (static_cast<int64_t>(bm.pid_a) * sh.page_tiles + g);
      const int64_t tile_b = (static_cast<int64_t>(bm.pid_b) * sh.page_tiles + g);
      const char *kp = kpool + (m16 < 8 ? tile_a : tile_b) * TILE_BYTES + k_lane_off;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int s = 0; s < NK; ++s) kr[t][s] = load_kv(kp + t * (TILE_BYTES / 2) + s * 512);
    };
    auto issue_v = [&](u32x4 (&vr)[NV], const WalkBlock &bm) {
      const int64_t tile_a = (static_cast<int64_t>(bm.pid_a) * sh.page_tiles + g);
      const int64_t tile_b = (static_cast<int64_t>(bm.pid_b) * sh.page_tiles + g);
      const char *vp = vpool + (jj < 2 ? tile_a : tile_b) * TILE_BYTES + v_lane_off;
#pragma unroll
      for (int s = 0; s < NV; ++s) vr[s] = load_kv(vp + s * 512);
    };
    // One block: scores from the K registers, which are then refilled (with the block `refill`,
    // if `more`) while the softmax runs; the V registers are refilled as soon as they are widened.
    auto step = [&](u32x4 (&kr)[2][NK], u32x4 (&vr)[NV], const WalkBlock &bm, const WalkBlock &refill, bool more) {
      const int lo = (bm.rows & 0xffff) - rw * C, hi = (bm.rows >> 16) - rw * C;
      const float c = p.scale_log2 * (jj < 2 ? bm.ka : bm.kb), vs = jj < 2 ? bm.va : bm.vb;
      bf16x8 kf[2][D / 32];
      if (FP8) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int s = 0; s < D / 64; ++s) {
            kf[t][2 * s] = fp8x8_to_bf16x8(kr[t][s][0], kr[t][s][1]);
            kf[t][2 * s + 1] = fp8x8_to_bf16x8(kr[t][s][2], kr[t][s][3]);
          }
      } else {
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int s = 0; s < D / 32; ++s) kf[t][s] = __builtin_bit_cast(bf16x8, kr[t][s]);
      }
      f32x4 sa[NTW], sb[NTW];
      walk_scores<BY_TILE, D, NTW>(qf, kf, sa, sb, lo, hi);
      if (more) issue_k(kr, refill);
      f16x8 vh[D / 16];
      if (FP8) {
#pragma unroll
        for (int s = 0; s < D / 32; ++s) {
          vh[2 * s] = __builtin_bit_cast(f16x8, fp8x8_to_f16x8(vr[s][0], vr[s][1], vs));
          vh[2 * s + 1] = __builtin_bit_cast(f16x8, fp8x8_to_f16x8(vr[s][2], vr[s][3], vs));
        }
      } else {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) vh[s] = __builtin_bit_cast(f16x8, vr[s]);
      }
      if (more) issue_v(vr, refill);
      walk_softmax_pv<BY_TILE, FP8, TREE, D, NTW>(limit, qidx, dmask, o, m, lacc, sa, sb, vh, (bm.flags & 1) != 0,
                                   (jj < 2 ? bm.vp_a : bm.vp_b) & 127, (jj < 2 ? bm.vp_a : bm.vp_b) >> 7,
                                   c, slack, lo, hi, rows);
    };
    // the j-th private block of this wavefront (past the end: the last one)
    auto rec_at = [&](int j) {
      const int jc = j < n_priv ? j : n_priv - 1;
      return load_walk_block<FP8>(p, priv_begin + ks + KS * jc, g, sh.Hkv, rec_in_lds, rec_lds, scl_lds, blk_begin);
    };
    {
      u32x4 kr[2][NK], vr[NV];
      WalkBlock cur = rec_at(0);
      WalkBlock nxt = rec_at(1);
      issue_k(kr, cur);
      issue_v(vr, cur);
      for (int i = 0; i + 1 < n_priv; ++i) {
        const WalkBlock nxt2 = rec_at(i + 2);
        step(kr, vr, cur, nxt, true);
        cur = nxt;
        nxt = nxt2;
      }
      step(kr, vr, cur, cur, false);
    }
  }
  }  // phases

  // ---- KS = 2: the upper pair hands its state to the lower pair, which folds it into its own
  // (log-sum-exp rule on the two references).  The LDS images are dead after the last barrier of
  // phase 1, and phase 2 does not touch LDS, so the hand-over area may lie behind the output staging.
  if (KS == 2) {
    float *fold = lds + LW * stage_floats<D>() + rw * kFoldWaveFloats;
    f32x4 *fo = reinterpret_cast<f32x4 *>(fold) + lane;                               // [nt][dt][lane]
    f32x4 *fl = reinterpret_cast<f32x4 *>(fold + NTW * (D / 16) * 256) + lane;         // [nt][lane]
    float *fm = fold + NTW * (D / 16) * 256 + NTW * 256 + lane;                        // [nt][lane]
    if (has_rows && ks == 1) {
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) {
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) fo[(nt * (D / 16) + dt) * 64] = o[nt][dt];
        fl[nt * 64] = lacc[nt];
        fm[nt * 64] = m[nt];
      }
    }
    __syncthreads();
    if (has_rows && ks == 0) {
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) {
        const float m1 = fm[nt * 64];
        const float mn = fmaxf(m[nt], m1);
        // a side that saw nothing still has the (finite) start value of m: its factor is 0, or 1
        // where neither saw anything (rows past the end of the wavefront's rows)
        const float a0 = fast_exp2(FP8 ? m[nt] - mn : (m[nt] - mn) * p.scale_log2);
        const float a1 = fast_exp2(FP8 ? m1 - mn : (m1 - mn) * p.scale_log2);
        m[nt] = mn;
        lacc[nt] = lacc[nt] * a0 + fl[nt * 64] * a1;
#pragma unroll
        for (int dt = 0; dt < D / 16; ++dt) o[nt][dt] = o[nt][dt] * a0 + fo[(nt * (D / 16) + dt) * 64] * a1;
      }
    }
  }

  // ---- output.  The LDS images are dead after the last barrier of phase 1.
  if (has_rows && ks == 0) {
    float m_log2[NTW];
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) m_log2[nt] = FP8 ? m[nt] : m[nt] * p.scale_log2;
    walk_write_rows<D, NTW>(p.out, p.lse, sh, g, rows, o, m_log2, lacc, qtok, lds + w * stage_floats<D>());
  }
}

// ---- generic attention (no matrix cores) ------------------------------------------------------
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o));
  return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// One wavefront per (work item, row): blockIdx.y strides over the item's rows.  Lane = token for
// the scores, lane = dim (d, d+64, ..) for the weighted sum.  The loops over dims and tokens fetch
// eight elements before they use them (in the same order as one at a time), so that a lane does not
// sit out a memory latency per element.
template <int KV, int QT, int LAYOUT>
__global__ __launch_bounds__(64) void spex_generic_attn_kernel(AttnArgs p, Shape sh, int rows_per_item) {
  constexpr int kU = 8;  // elements fetched before they are used
  __shared__ float qs[256];
  const int lane = threadIdx.x;
  const int32_t *rec = p.items + static_cast<int64_t>(blockIdx.x) * 8;
  const int pg_begin = rec[0];
  const int pg_count = rec[1];
  const int qt_begin = rec[2];
  const int qt_count = rec[3];
  const int pbase = rec[4];
  const int g = rec[6];
  const int row0 = rec[7];
  if (pg_count == 0) return;  // padding item
  const int D = sh.D, P = sh.P, G = sh.G;
  const int rows = qt_count * G;
  const int64_t tile_elems = static_cast<int64_t>(P) * D;
  const int n_tok_slots = pg_count * P;
  const int r_end = min(rows, row0 + rows_per_item);

  for (int r = row0 + static_cast<int>(blockIdx.y); r < r_end; r += static_cast<int>(gridDim.y)) {
    const int qt = p.qt_rec[2 * (qt_begin + r / G)];
    const int hh = r % G;
    const int limit = p.qt_rec[2 * (qt_begin + r / G) + 1];
    const int d_base = p.qt_mask ? limit - 1 - p.qt_mask[2 * qt] : 0;
    const uint32_t d_mask = p.qt_mask ? static_cast<uint32_t>(p.qt_mask[2 * qt + 1]) : 0u;
    const int64_t qbase = (static_cast<int64_t>(qt) * sh.Hq + g * G + hh) * D;
    __syncthreads();
    for (int d = lane; d < D; d += 64) qs[d] = load_elem<QT>(p.q, qbase + d);
    __syncthreads();

    float m = kNegInf, l = 0.f;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    for (int t0 = 0; t0 < n_tok_slots; t0 += 64) {
      const int ti = t0 + lane;
      const int e = pg_begin + ti / P;
      const int slot = ti % P;
      bool ok = ti < n_tok_slots;
      float s = kNegInf;
      if (ok) {
        const int vp = p.pg_rec[2 * e + 1];
        const int pos = (vp >> 7) + slot;
        bool seen = pos < limit;
        if (p.qt_mask) {  // draft tree: everything before the drafts, then the mask's bits
          const int rel = pos - d_base;
          seen = rel < 0 || (rel < 32 && ((d_mask >> rel) & 1u));
        }
        ok = slot < (vp & 127) && seen;
      }
      if (ok) {
        const int64_t tile = (static_cast<int64_t>(p.pg_rec[2 * e]) * sh.page_tiles + g);
        float dot = 0.f;
        int d = 0;
        for (; d + kU <= D; d += kU) {
          float kv[kU];
#pragma unroll
          for (int u = 0; u < kU; ++u)
            kv[u] = load_elem<KV>(p.k_pool, tile * tile_elems + k_offset<KV, LAYOUT>(slot, d + u, D));
#pragma unroll
          for (int u = 0; u < kU; ++u) dot += qs[d + u] * kv[u];
        }
        for (; d < D; ++d)
          dot += qs[d] * load_elem<KV>(p.k_pool, tile * tile_elems + k_offset<KV, LAYOUT>(slot, d, D));
        if (KV == kFP8) dot *= p.k_scale[p.pg_rec[2 * e] * sh.Hkv + g];
        s = dot * p.scale_log2;
      }
      const float m_new = fmaxf(m, wave_max(s));
      if (m_new == kNegInf) continue;
      const float alpha = fast_exp2(m - m_new);
      const float pw = ok ? fast_exp2(s - m_new) : 0.f;
      l = l * alpha + wave_sum(pw);
      m = m_new;
#pragma unroll
      for (int c = 0; c < 4; ++c) acc[c] *= alpha;
      const int n_here = min(64, n_tok_slots - t0);
      for (int tb = 0; tb < n_here; tb += kU) {
        float wt[kU], vv[kU][4];
#pragma unroll
        for (int u = 0; u < kU; ++u) {
          const int t = tb + u;
          const float pt = t < n_here ? __shfl(pw, t & 63) : 0.f;
          wt[u] = pt;
#pragma unroll
          for (int c = 0; c < 4; ++c) vv[u][c] = 0.f;
          if (pt == 0.f) continue;  // wave-uniform: pt is a broadcast value
          const int e2 = pg_begin + (t0 + t) / P;
          const int slot2 = (t0 + t) % P;
          const int64_t tile = (static_cast<int64_t>(p.pg_rec[2 * e2]) * sh.page_tiles + g);
          if (KV == kFP8) wt[u] = pt * p.v_scale[p.pg_rec[2 * e2] * sh.Hkv + g];
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            const int d = lane + 64 * c;
            if (d < D) vv[u][c] = load_v_elem<KV, LAYOUT>(p.v_pool, tile * tile_elems + v_offset<KV, LAYOUT>(slot2, d, D));
          }
        }
#pragma unroll
        for (int u = 0; u < kU; ++u)
#pragma unroll
          for (int c = 0; c < 4; ++c) acc[c] += wt[u] * vv[u][c];
      }
    }
    const int64_t out_slot = static_cast<int64_t>(pbase) + static_cast<int64_t>(g) * rows + r;
    if (lane == 0) {
      p.part_ml[out_slot * 2] = m;
      p.part_ml[out_slot * 2 + 1] = l;
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int d = lane + 64 * c;
      if (d < D) p.part_o[out_slot * D + d] = acc[c];
    }
  }
}

// ---- row-major pools on the matrix cores --------------------------------------------------------
// One workgroup (four wavefronts) per work item and group of up to 64 of its rows.  A wavefront
// holds one tile of 16 rows; an item with up to 16 (32) rows has its tokens split between four
// (two) wavefronts, which fold their softmax states through LDS at the end.
//
// A row-major tile is an operand as it lies in memory, because a contraction may take its index in
// any order as long as both operands agree:
//   S^T = K Q^T: lane (token m16, group jj) loads 16 bytes of its token's row at a time; every
//     element (fp32) or octet (16-bit, widened fp8) of the load is one MFMA operand whose
//     contraction index is the dim the lane holds, and Q is loaded with the same dims.
//   The result leaves tokens 4 jj .. 4 jj + 3 of row m16 in the lane.
//   fp32 pools: P^T as the B operand of four fp32 MFMA 16x16x4, one per r, whose contraction runs over tokens
//     {4 jj + r}.  Lane (m16, jj) loads VE consecutive dims VE m16 .. of token 4 jj + r; element i is the A
//     operand of O^T += V^T P^T for the tile of dims {VE m + i}.
//   16-bit and fp8 pools: two groups of 16 tokens at a time, which leave eight weights in the lane, the
//     contraction index of a bf16 MFMA 16x16x32.  The lane's V rows of the same eight tokens are turned
//     token-minor by one byte permutation per register.  A weight goes in as three bf16 pieces that add up to
//     the fp32 weight, and V is exact in bf16, so every product is the one the fp32 MFMA would see.
//
// Why this shape: per 32 tokens and row tile at D = 128 a wavefront issues 8 + 24 MFMAs of 16 cycles; P V on the
// fp32 MFMA was 64 of 32 cycles, four times as long as the memory needs for the tokens, and bound the kernel.
// Measured, fp32 P V -> bf16 pieces: 8 ragged queries of 16 branches, bf16 pages of 32 tokens, heads 32/8/128,
// 42.3 -> 37.3 us a call; 32 queries 117 -> 101 (fp8 94 -> 75); heads 16/4/256, fp8, 140 -> 73 (two workgroups
// a compute unit instead of one).  Error against 64 bits 2.9e-7 (3.1e-7 with the fp32 MFMA, 4.7e-7 on the vector ALU).
// A wavefront's K loads for the next tokens are issued right after the score MFMAs, its V loads right after the PV
// MFMAs, page records a step ahead.
template <int KV>
struct RowMajorTraits {};
template <>
struct RowMajorTraits<kF32> { static constexpr int kEsz = 4; };
template <>
struct RowMajorTraits<kBF16> { static constexpr int kEsz = 2; };
template <>
struct RowMajorTraits<kFP8> { static constexpr int kEsz = 1; };

// kRowAny: head dims below DP.  kRowFull: DP itself, whose addresses and bounds are known when compiled (bf16, 128:
// 161 registers instead of 182, three workgroups a compute unit instead of two: 114 -> 101 us for the 32 queries
// above).  kRowHalf: fp8 rows of a multiple of 8 bytes that is none of 16, K loaded 8 bytes at a time (heads 6/3/40,
// 31 prompts of 14000 tokens 2935 us in the generic kernel, 74 here; 32 queries of 16 branches 342 -> 22).
enum RowMode : int { kRowAny, kRowFull, kRowHalf };

// Whether a lane of the wavefront holds a weight, other than 0, below 2^-86: its pieces, or the 2^-40 of it that keeps
// them positive, would be subnormal bf16 numbers, whose last bit is 2^-133 (weights of 2^-118 and 2^-124 then err by
// 1e-5 and 1e-3 instead of 8e-8; below 2^-93 an infinite value gives NaN).  Few steps have one, with a score 59 below
// the row's largest or an fp8 page scale that small, so the smallest of all is looked at first (pages of 32 tokens,
// 16 branches: 37.5 us without the test, 37.7 with it).
__device__ __forceinline__ bool beyond_pieces(const float (&pr)[2][4]) {
  const float lo = fminf(fminf(fminf(pr[0][0], pr[0][1]), fminf(pr[0][2], pr[0][3])), fminf(fminf(pr[1][0], pr[1][1]), fminf(pr[1][2], pr[1][3])));
  if (!__any(lo < 0x1p-86f)) return false;
  uint32_t least = 0xffffffffu;  // weight 0 wraps to the top
#pragma unroll
  for (int i = 0; i < 8; ++i) least = min(least, __builtin_bit_cast(uint32_t, pr[i >> 2][i & 3]) - 1u);
  return __any(least < __builtin_bit_cast(uint32_t, 0x1p-86f) - 1u);
}

// Workgroups per compute unit: as many as the registers allow without spills.  fp32 heads of 64 keep five (91 registers;
// left alone the compiler takes 99, and four: 32 queries of 16 branches 34.1 -> 35.6 us, 8 of 9000 tokens 47.2 -> 49.1).
constexpr int rowmajor_occupancy(int kv, int dp, int mode) {
  if (dp > 128) return kv == kFP8 ? 2 : 1;
  if (dp == 64 && kv == kF32 && mode == kRowFull) return 5;
  return dp == 64 || kv != kF32 || mode == kRowFull ? 3 : 2;
}

template <int KV, int DP, int MODE>
__global__ __launch_bounds__(256, rowmajor_occupancy(KV, DP, MODE)) void spex_rowmajor_attn_kernel(AttnArgs p, Shape sh, SplitLists ls) {
  constexpr int ESZ = RowMajorTraits<KV>::kEsz;
  constexpr int CH = 16 / ESZ;             // elements per 16-byte load
  constexpr int NK = DP / (4 * CH);        // K loads per lane and step
  constexpr int VE = DP / 16 < CH ? DP / 16 : CH;  // V elements per lane and load
  constexpr int NC = DP / (16 * VE);       // V loads per token
  constexpr int NO = DP / 16;              // output tiles
  constexpr int NQ = KV == kF32 ? DP / 4 : DP / 8;  // Q registers
  constexpr int SUB = KV == kF32 ? 1 : 2;  // groups of 16 tokens per step
  constexpr int kFold = NO * 4 + 2;        // floats per lane a wavefront hands over
  // A step's values are requested at its start, or for most fp32 rows at the end of the step before: us a call with values at the
  // start / at the end, heads 8/2/64 290 / 279, 16/2/64 566 / 538, 12/4/96 609 / 574, 12/4/80 587 / 535 (8 branches of 67 queries on
  // 6 prompts of 4400), 6/2/200 77.0 / 73.9 (of 16 on 8 of 512); 32/8/128 1373 / 1407 and 141 / 145, 6/3/40 174 / 178.
  constexpr bool kEarlyV = KV != kF32 || (DP == 128 && MODE == kRowFull) || (DP == 64 && MODE == kRowAny);
  __shared__ float fold[4 * 64 * kFold];

  const int lane = threadIdx.x & 63, m16 = lane & 15, jj = lane >> 4;
  const int w = uniform(threadIdx.x >> 6);
  const ListPos at = list_of(ls, static_cast<int>(blockIdx.x));
  const int span = at.span;
  const int group = at.local / at.n_items; // 64 rows each
  const Item it = load_item(at.items, at.local - group * at.n_items);
  if (it.pg_count == 0) return;            // padding item
  static_assert(MODE != kRowHalf || (KV == kFP8 && DP <= 128), "loads of V rows are 8 bytes at most");
  const int D = MODE == kRowFull ? DP : sh.D, G = sh.G, rows = it.qt_count * G;
  const int row_end = min(rows, it.row0 + span);
  const int row_lo = it.row0 + group * 64;
  if (row_lo >= row_end) return;           // whole workgroup
  const int here = row_end - row_lo;
  const int ks_log = here <= 16 ? 2 : (here <= 32 ? 1 : 0);  // log2 of the wavefronts per row tile
  const int rt = w >> ks_log, ks = w & ((1 << ks_log) - 1);
  const int row_base = row_lo + rt * 16;
  const bool has_rows = row_base < row_end;

  const int logp = 31 - __builtin_clz(sh.P);
  const int n_slots = it.pg_count << logp;
  // 16 tokens a step, SUB steps a turn of the loop; wavefronts share an item by whole turns
  const int n_steps = (n_slots + 15) >> 4, n_turns = (n_steps + SUB - 1) / SUB;
  const int step0 = ((n_turns * ks) >> ks_log) * SUB, step1 = min(n_steps, ((n_turns * (ks + 1)) >> ks_log) * SUB);
  const int slot_end = min(n_slots, step1 << 4);

  // ---- rows
  const int row = row_base + m16;
  const bool row_ok = row < row_end;
  int limit = 0, qt = 0, d_base = 0;
  uint32_t d_mask = 0;
  u32x4 q[NQ / 4];
#pragma unroll
  for (int i = 0; i < NQ / 4; ++i) q[i] = u32x4{0, 0, 0, 0};
  if (row_ok) {
    const int2 qr = *reinterpret_cast<const int2 *>(p.qt_rec + 2 * (it.qt_begin + row / G));
    qt = qr.x;
    limit = qr.y;
    if (p.qt_mask) {
      const int2 dm = *reinterpret_cast<const int2 *>(p.qt_mask + 2 * qt);
      d_base = limit - 1 - dm.x;
      d_mask = static_cast<uint32_t>(dm.y);
    }
    const int64_t qrow = (static_cast<int64_t>(qt) * sh.Hq + it.g * G + row % G) * D;
#pragma unroll
    for (int i = 0; i < NQ / 4; ++i) {
      // fp32: load i covers dims 16 i + 4 jj ..; bf16: 32 i + 8 jj ..; against fp8 K two octets per load
      const int d = KV == kF32 ? 16 * i + 4 * jj : (KV == kBF16 ? 32 * i + 8 * jj : 64 * (i >> 1) + 16 * jj + 8 * (i & 1));
      if (d < D)
        q[i] = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(p.q) + (qrow + d) * (KV == kF32 ? 4 : 2));
    }
  }

  f32x4 o[NO];
#pragma unroll
  for (int i = 0; i < NO; ++i) o[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  float m = kRowMajorMInit, l = 0.f;

  const int64_t tile_bytes = static_cast<int64_t>(D) * ESZ << logp;
  const char *kpool = static_cast<const char *>(p.k_pool), *vpool = static_cast<const char *>(p.v_pool);
  // Page record of the token whose K row the lane loads (token m16 of the step) and of the four
  // tokens whose V rows it loads and whose scores it gets (4 jj .. 4 jj + 3: one page, P >= 4).
  struct Rec {
    int2 k, v;
  };
  auto rec_of = [&](int step) {
    const int last = it.pg_count - 1;
    const int s = min(step, step1 - 1) << 4;
    Rec r;
    r.k = *reinterpret_cast<const int2 *>(p.pg_rec + 2 * (it.pg_begin + min((s + m16) >> logp, last)));
    r.v = *reinterpret_cast<const int2 *>(p.pg_rec + 2 * (it.pg_begin + min((s + 4 * jj) >> logp, last)));
    return r;
  };
  // Dims past D (D < DP) are read from the start of the row instead, so that no load is
  // conditional: in K they meet zeros of Q, in V they make output dims that are not written.
  // Steps past the wavefront's last one are read as well, for the same reason, but by all lanes from the first token of
  // the last step: one cache line (in the modes whose offsets are the lane's own, one row), and one just read, instead of 16 rows.
  // An item of 76 tokens is one turn or none for a
  // wavefront, which used to request its tokens up to four times (8 ragged queries of 16 branches, bf16 pages of 32
  // tokens: 35.7 -> 30.3 us a call, 32 queries 131 -> 116; fp32 heads 28/4/128, 64 prompts of 1024 142 -> 137;
  // the start of the tile instead, a line that may be no wavefront's own: 4 prompts of 12000 tokens 57.4, 52.4 so,
  // 54.1 with whole rows repeated).  Offsets that took part in this were made anew every step: fp32 heads 12/4/80, 8 branches of 67
  // queries on 6 prompts of 4400 610 -> 587 us, 6/3/40 179 -> 174, 6/2/200, 64 prompts of 1024, 96 -> 92.
  u32x4 kr[SUB][NK];
  auto load_k = [&](int j, const Rec &r, int step) {
    const int msk = step < step1 ? -1 : 0;  // uniform
    const int slot = ((min(step, step1 - 1) << 4) + (m16 & msk)) & (sh.P - 1), dj = MODE == kRowFull ? 0 : CH * jj;
    const char *src = kpool + (static_cast<int64_t>(r.k.x) * sh.page_tiles + it.g) * tile_bytes + (slot * D * ESZ + (MODE == kRowFull ? 16 * jj & msk : 0));
#pragma unroll
    for (int i = 0; i < NK; ++i) {
      const int d = 4 * CH * i + dj;
      if constexpr (MODE == kRowHalf) {
        const u32x2 lo = *reinterpret_cast<const u32x2 *>(src + (d < D ? d : 0));
        const u32x2 hi = *reinterpret_cast<const u32x2 *>(src + (d + 8 < D ? d + 8 : 0));
        kr[j][i] = u32x4{lo[0], lo[1], hi[0], hi[1]};
      } else {
        kr[j][i] = *reinterpret_cast<const u32x4 *>(src + (MODE == kRowFull || d < D ? d * ESZ : 0));
      }
    }
  };
  // Page scales of the four tokens of the lane, ahead of their keys: behind the values already on their way they
  // would make the scores wait for those.
  struct Scales {
    float k, v;
  };
  Scales scl[SUB];
  auto load_scales = [&](int j, const Rec &r) {
    scl[j] = {1.f, 1.f};
    if (KV == kFP8) {
      const int64_t at_page = static_cast<int64_t>(r.v.x) * sh.Hkv + it.g;
      scl[j] = {p.k_scale[at_page], p.v_scale[at_page]};
    }
  };
  struct VReg {
    uint32_t w[VE * ESZ / 4];
  };
  VReg vr[SUB][4][NC];
  int v_off[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) v_off[c] = 16 * VE * c + VE * m16 < D ? 16 * VE * c : -VE * m16;
  auto load_v = [&](int j, const Rec &r, int step) {
    const int msk = step < step1 ? -1 : 0;
    const int slot = ((min(step, step1 - 1) << 4) + (4 * jj & msk)) & (sh.P - 1);
    const char *src = vpool + (static_cast<int64_t>(r.v.x) * sh.page_tiles + it.g) * tile_bytes + (slot * D + (MODE == kRowFull ? VE * m16 & msk : VE * m16)) * ESZ;
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int c = 0; c < NC; ++c)
        __builtin_memcpy(&vr[j][t][c], __builtin_assume_aligned(src + (t * D + (MODE == kRowFull ? 16 * VE * c : v_off[c])) * ESZ, VE * ESZ), VE * ESZ);
  };

  if (has_rows && step0 < step1) {
    Rec cur[SUB], nxt[SUB];
#pragma unroll
    for (int j = 0; j < SUB; ++j) {
      cur[j] = rec_of(step0 + j);
      nxt[j] = rec_of(step0 + SUB + j);
      load_scales(j, cur[j]);
      load_k(j, cur[j], step0 + j);
      if constexpr (!kEarlyV) load_v(j, cur[j], step0 + j);
    }
    for (int st = step0; st < step1; st += SUB) {
      // 16-bit and fp8 values go out before the keys are waited for: left to itself the compiler puts them behind the first
      // MFMA (fp8 pages of 32 tokens 27.4 -> 26.6 us, heads 6/3/40 22.8 -> 21.9, bf16 heads of 96 33.6 -> 32.9; fp32
      // 45.1 -> 45.8).
      if constexpr (kEarlyV)
#pragma unroll
        for (int j = 0; j < SUB; ++j) load_v(j, cur[j], st + j);
      if constexpr (KV != kF32) __builtin_amdgcn_sched_barrier(0);
      float x[SUB][4], vs_l[SUB], mx = kNegInf;
#pragma unroll
      for (int j = 0; j < SUB; ++j) {
        vs_l[j] = scl[j].v;
        f32x4 sa = {0.f, 0.f, 0.f, 0.f}, sb = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NK; ++i) {
          const u32x4 &k = kr[j][i];
          if (KV == kF32) {
            const f32x4 kv = __builtin_bit_cast(f32x4, k), qv = __builtin_bit_cast(f32x4, q[i]);
            sa = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[0], qv[0], sa, 0, 0, 0);
            sb = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[1], qv[1], sb, 0, 0, 0);
            sa = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[2], qv[2], sa, 0, 0, 0);
            sb = __builtin_amdgcn_mfma_f32_16x16x4f32(kv[3], qv[3], sb, 0, 0, 0);
          } else if (KV == kBF16) {
            f32x4 &acc = (i & 1) ? sb : sa;
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k), __builtin_bit_cast(bf16x8, q[i]), acc, 0, 0, 0);
          } else {
            sa = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fp8x8_to_bf16x8(k[0], k[1]), __builtin_bit_cast(bf16x8, q[2 * i]), sa, 0, 0, 0);
            sb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fp8x8_to_bf16x8(k[2], k[3]), __builtin_bit_cast(bf16x8, q[2 * i + 1]), sb, 0, 0, 0);
          }
        }
        // ---- what the row sees of the lane's four tokens
        const int s16 = st + j, slot = ((s16 << 4) + 4 * jj) & (sh.P - 1);
        const int pos = (cur[j].v.y >> 7) + slot;
        int have = (s16 << 4) + 4 * jj < slot_end ? (cur[j].v.y & 127) - slot : 0;
        uint32_t vm = 0xfu;
        if (p.qt_mask) {
          const int shift = pos - d_base + 32;
          const uint64_t bits = (static_cast<uint64_t>(d_mask) << 32) | 0xffffffffull;
          vm = shift <= 0 ? 0xfu : (shift >= 64 ? 0u : static_cast<uint32_t>(bits >> shift) & 0xfu);
        } else {
          have = min(have, limit - pos);
        }
        const float c = p.scale_log2 * scl[j].k;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          x[j][r] = (sa[r] + sb[r]) * c;
          x[j][r] = (r < have && ((vm >> r) & 1u)) ? x[j][r] : kNegInf;
        }
        mx = fmaxf(mx, fmaxf(fmaxf(x[j][0], x[j][1]), fmaxf(x[j][2], x[j][3])));
      }
#pragma unroll
      for (int j = 0; j < SUB; ++j) {
        load_scales(j, nxt[j]);
        load_k(j, nxt[j], st + SUB + j);
      }
      // The softmax reference is the running maximum, so that no weight exceeds 1 and a sum of large
      // fp32 values overflows only where the row's own result does.
      if (__any(mx > m)) {
        const float m_new = fmaxf(m, row_group_max(mx));
        const float alpha = fast_exp2(m - m_new);
        m = m_new;
        l *= alpha;
#pragma unroll
        for (int i = 0; i < NO; ++i) o[i] *= alpha;
      }
      float pr[SUB][4];
#pragma unroll
      for (int j = 0; j < SUB; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          pr[j][r] = fast_exp2(x[j][r] - m);
          l += pr[j][r];
          if (KV == kFP8) pr[j][r] *= vs_l[j];
        }
      // Loads past the item's pages (of 4 and 8 tokens) or the wavefront's last group repeated tokens, which may hold
      // infinities: their weight is 0, so their values must be 0 as well.
      if (((st + SUB) << 4) > slot_end) {
#pragma unroll
        for (int j = 0; j < SUB; ++j)
          if (((st + j) << 4) + 4 * jj >= slot_end)
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
              for (int cc = 0; cc < NC; ++cc) vr[j][t][cc] = VReg{};
      }
      if constexpr (SUB == 2)
        if (beyond_pieces(pr)) {  // fp32 weights on the fp32 MFMA; nothing is left for the pieces below
#pragma unroll
          for (int t = 0; t < 8; ++t) {
#pragma unroll
            for (int cc = 0; cc < NC; ++cc) {
              VReg &vv = vr[t >> 2][t & 3][cc];
#pragma unroll
              for (int i = 0; i < VE; ++i) {
                float v;
                if constexpr (KV == kBF16) {
                  v = __builtin_bit_cast(float, (i & 1) ? vv.w[i / 2] & 0xffff0000u : vv.w[i / 2] << 16);
                } else {
                  const int wd = static_cast<int>(vv.w[i / 4]);
                  const f32x2 two = (i & 2) ? __builtin_amdgcn_cvt_pk_f32_fp8(wd, true) : __builtin_amdgcn_cvt_pk_f32_fp8(wd, false);
                  v = two[i & 1];
                }
                o[cc * VE + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, pr[t >> 2][t & 3], o[cc * VE + i], 0, 0, 0);
              }
              vv = VReg{};
            }
            pr[t >> 2][t & 3] = 0.f;
          }
        }
      if constexpr (KV == kF32) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int cc = 0; cc < NC; ++cc)
#pragma unroll
            for (int i = 0; i < VE; ++i)
              o[cc * VE + i] = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, vr[0][t][cc].w[i]), pr[0][t], o[cc * VE + i], 0, 0, 0);
      } else {
        // Three pieces of 8 significant bits, each cut off toward zero: together the whole fp32 weight.  A piece
        // of nothing would turn an infinite value into NaN; 2^-40 of the weight, far below its last bit, keeps it
        // positive.
        u32x4 pc[3];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float a = pr[i >> 1][(i & 1) * 2], b = pr[i >> 1][(i & 1) * 2 + 1];
          const float ta = a * 0x1p-40f, tb = b * 0x1p-40f;
#pragma unroll
          for (int n = 0; n < 3; ++n) {
            pc[n][i] = pack_hi16(a, b);
            a = a - __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, a) & 0xffff0000u) + ta;
            b = b - __builtin_bit_cast(float, __builtin_bit_cast(uint32_t, b) & 0xffff0000u) + tb;
          }
        }
#pragma unroll
        for (int cc = 0; cc < NC; ++cc)
#pragma unroll
          for (int i2 = 0; i2 < VE / 2; ++i2) {
            // dims 2 i2 and 2 i2 + 1 of the lane's eight tokens, turned token-minor
            uint32_t d[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
              if constexpr (KV == kBF16) {
                d[t] = vr[t >> 2][t & 3][cc].w[i2];
              } else {
                const int wd = static_cast<int>(vr[t >> 2][t & 3][cc].w[i2 / 2]);
                d[t] = __builtin_bit_cast(uint32_t, (i2 & 1) ? __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(wd, 1.0f, true)
                                                             : __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(wd, 1.0f, false));
              }
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
              u32x4 v;
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] = __builtin_amdgcn_perm(d[2 * i + 1], d[2 * i], e ? 0x07060302u : 0x05040100u);
              f32x4 &acc = o[cc * VE + 2 * i2 + e];
#pragma unroll
              for (int n = 0; n < 3; ++n)
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pc[n]), acc, 0, 0, 0);
            }
          }
      }
#pragma unroll
      for (int j = 0; j < SUB; ++j) {
        if constexpr (!kEarlyV) load_v(j, nxt[j], st + SUB + j);
        cur[j] = nxt[j];
        nxt[j] = rec_of(st + 2 * SUB + j);
      }
    }
  }
  l += __shfl_xor(l, 16);  // the row sum is spread over the four lane groups
  l += __shfl_xor(l, 32);

  // ---- output.  The wavefronts of one row tile fold their states through LDS: each leaves its own, and folds and stores
  // a share of every row, its quarter or half of the registers r (against the first wavefront alone: heads 16/4/256
  // 40.8 -> 38.4 us, fp8 29.1 -> 28.2; others within 1 %).
  const int n_states = 1 << ks_log;
  const float *states = fold + (rt << ks_log) * (64 * kFold) + lane;
  float f[4] = {1.f, 0.f, 0.f, 0.f};
  if (ks_log > 0) {
    float *own = fold + w * (64 * kFold) + lane;
#pragma unroll
    for (int i = 0; i < NO; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) own[(i * 4 + r) * 64] = o[i][r];
    own[NO * 4 * 64] = m;
    own[(NO * 4 + 1) * 64] = l;
    __syncthreads();
    float mv[4], lv[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int at_v = v < n_states ? v : 0;
      mv[v] = states[at_v * (64 * kFold) + NO * 4 * 64];
      lv[v] = v < n_states ? states[at_v * (64 * kFold) + (NO * 4 + 1) * 64] : 0.f;
    }
    m = fmaxf(fmaxf(mv[0], mv[1]), fmaxf(mv[2], mv[3]));
    l = 0.f;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      f[v] = fast_exp2(mv[v] - m);
      l += lv[v] * f[v];
    }
  }
  if (!row_ok) return;
  const int64_t slot = p.finish ? static_cast<int64_t>(qt) * sh.Hq + it.g * G + row % G
                                : static_cast<int64_t>(it.pbase) + static_cast<int64_t>(it.g) * rows + row;
  if (jj == 0 && ks == 0) {
    if (!p.finish)
      *reinterpret_cast<f32x2 *>(p.part_ml + slot * 2) = f32x2{m, l};
    else if (p.lse)
      p.lse[slot] = (m + __builtin_log2f(l)) * 0.6931471805599453f;
  }
  const float norm = p.finish ? 1.0f / l : 1.0f;
  float *dst = (p.finish ? p.out : p.part_o) + slot * D;
  // the lane holds dims 16 VE c + 4 VE jj .. + 4 VE - 1 of its row
  auto dim_of = [&](int c, int r, int h) { return 16 * VE * c + 4 * VE * jj + VE * r + 4 * h; };
  if (ks_log > 0) {
    const int r_end = (4 * (ks + 1)) >> ks_log;
    for (int r = (4 * ks) >> ks_log; r < r_end; ++r)
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int h = 0; h < VE / 4; ++h) {
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (v < n_states)  // uniform
#pragma unroll
              for (int e = 0; e < 4; ++e) acc[e] += states[v * (64 * kFold) + ((c * VE + 4 * h + e) * 4 + r) * 64] * f[v];
          const int d = dim_of(c, r, h);
          if (d < D) *reinterpret_cast<f32x4 *>(dst + d) = acc * norm;
        }
    return;
  }
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int h = 0; h < VE / 4; ++h) {
        const int d = dim_of(c, r, h);
        if (d < D)
          *reinterpret_cast<f32x4 *>(dst + d) =
              f32x4{o[c * VE + 4 * h][r], o[c * VE + 4 * h + 1][r], o[c * VE + 4 * h + 2][r], o[c * VE + 4 * h + 3][r]} * norm;
      }
}

// ---- merge -----------------------------------------------------------------------------------
// One row (query token, query head) per slices * D / VEC threads, threadIdx = (vector of the row, slice and query token,
// query head): slice s folds pieces s, s + slices, .. of the row, a thread VEC consecutive dims, and the slices are folded
// through LDS.  Bound by latency, not bytes: a piece is a chain of dependent reads (its slot, then m, l and o), so
// four pieces of a slice are requested together and the row's pieces are spread over the slices; where the pieces'
// records lie at a fixed stride the chain is one read shorter than through part_indptr.  One query of 16 branches, 12.2 us
// a call: 11.3 so and without divisions, 10.9 with the kv heads on their XCDs.
// Where a kv head has few query heads a workgroup takes several query tokens, as many as fill its 256 threads: with one the
// LDS arrays let a compute unit hold 26 workgroups of 16 to 64 threads.  4096 query tokens, this kernel alone, us, with one
// token a workgroup / several: heads 32/32/128 71.8 / 41.1, 16/16/64 37.0 / 15.9, 6/3/40 9.7 / 7.2, 8/4/64 11.7 / 9.0,
// 12/4/96 16.6 / 14.3, 24/8/128 37.8 / 32.2.  Up to 128 threads only: 12/4/96 16.9, 24/8/128 38.0, the others the same.
// MANY: several query tokens a workgroup.
template <int VEC, bool MANY>
__global__ __launch_bounds__(kMergeThreads) void spex_lse_merge_kernel(MergeArgs a, Shape sh) {
  __shared__ __attribute__((aligned(16))) float lds_o[kMergeThreads * VEC];
  __shared__ float lds_ml[kMergeThreads][2];
  const int dv = static_cast<int>(blockDim.x), slices = MANY ? 1 << a.slice_log2 : static_cast<int>(blockDim.y);
  const int c = static_cast<int>(threadIdx.x), s = MANY ? static_cast<int>(threadIdx.y) & (slices - 1) : static_cast<int>(threadIdx.y);
  const int tid = (static_cast<int>(threadIdx.z) * static_cast<int>(blockDim.y) + static_cast<int>(threadIdx.y)) * dv + c;
  int qi = static_cast<int>(a.heads_first ? blockIdx.z : blockIdx.x);  // uniform unless MANY: what hangs on it alone are scalar loads
  if (MANY) qi = qi * (static_cast<int>(blockDim.y) >> a.slice_log2) + (static_cast<int>(threadIdx.y) >> a.slice_log2);
  const int g = static_cast<int>(a.heads_first ? blockIdx.x : blockIdx.y);
  const int hh = static_cast<int>((a.heads_first ? blockIdx.y : blockIdx.z) * blockDim.z + threadIdx.z);
  const bool live = hh < sh.G && (!MANY || qi < a.n_qtok);
  const int qt = a.qt_ids && (!MANY || live) ? a.qt_ids[qi] : qi;
  const int64_t orow = static_cast<int64_t>(qt) * sh.Hq + g * sh.G + hh;
  float m = kNegInf, l = 0.f, acc[VEC];
#pragma unroll
  for (int i = 0; i < VEC; ++i) acc[i] = 0.f;
  if (live) {
    const bool at_stride = a.stride > 0;  // uniform
    const int e0 = at_stride ? 0 : a.part_indptr[qt], e1 = at_stride ? a.stride : a.part_indptr[qt + 1];
    const int32_t *rec = a.rec + 2 * static_cast<int64_t>(qt) * a.stride;
    for (int e = e0 + s; e < e1; e += kMergeBatch * slices) {
      // entries past the row's last one are read as some valid one and count nothing
      float mj[kMergeBatch], lj[kMergeBatch], oj[kMergeBatch][VEC];
      int64_t slot[kMergeBatch];
      bool there[kMergeBatch];
#pragma unroll
      for (int k = 0; k < kMergeBatch; ++k) {
        const int ek = e + k * slices < e1 ? e + k * slices : e1 - 1;
        int2 r;
        if (at_stride)
          r = *reinterpret_cast<const int2 *>(rec + 2 * ek);
        else
          r = int2{a.part_base[ek], a.part_hstride[ek]};
        there[k] = e + k * slices < e1 && r.x >= 0;
        slot[k] = max(r.x, 0) + static_cast<int64_t>(g) * r.y + hh;
      }
#pragma unroll
      for (int k = 0; k < kMergeBatch; ++k) {
        const f32x2 ml = *reinterpret_cast<const f32x2 *>(a.part_ml + slot[k] * 2);
        const bool use = there[k] && ml[1] != 0.f;
        mj[k] = use ? ml[0] : kNegInf;
        lj[k] = use ? ml[1] : 0.f;
        const float *op = a.part_o + slot[k] * sh.D + c * VEC;
        if (VEC == 4) {
          const f32x4 o = *reinterpret_cast<const f32x4 *>(op);
#pragma unroll
          for (int i = 0; i < VEC; ++i) oj[k][i] = o[i];
        } else {
#pragma unroll
          for (int i = 0; i < VEC; ++i) oj[k][i] = op[i];
        }
      }
      float m_new = m;
#pragma unroll
      for (int k = 0; k < kMergeBatch; ++k) m_new = fmaxf(m_new, mj[k]);
      if (m_new == kNegInf) continue;  // nothing seen so far
      const float fa = fast_exp2(m - m_new);
      l *= fa;
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] *= fa;
#pragma unroll
      for (int k = 0; k < kMergeBatch; ++k) {
        const float f = fast_exp2(mj[k] - m_new);
        l += lj[k] * f;
        if (lj[k] != 0.f) {
#pragma unroll
          for (int i = 0; i < VEC; ++i) acc[i] += oj[k][i] * f;
        }
      }
      m = m_new;
    }
  }
  if (slices > 1) {
#pragma unroll
    for (int i = 0; i < VEC; ++i) lds_o[tid * VEC + i] = acc[i];
    lds_ml[tid][0] = m;
    lds_ml[tid][1] = l;
    __syncthreads();
    if (!live || s != 0) return;
    float m_all = m;
    for (int k = 1; k < slices; ++k) m_all = fmaxf(m_all, lds_ml[tid + k * dv][0]);
    const float m_safe = m_all == kNegInf ? 0.f : m_all;  // every score of the row is -inf: lse is -inf too
    const float f0 = fast_exp2(m - m_safe);
    l *= f0;
#pragma unroll
    for (int i = 0; i < VEC; ++i) acc[i] *= f0;
    for (int k = 1; k < slices; ++k) {
      const int t = tid + k * dv;
      const float f = fast_exp2(lds_ml[t][0] - m_safe);
      l += lds_ml[t][1] * f;
#pragma unroll
      for (int i = 0; i < VEC; ++i) acc[i] += lds_o[t * VEC + i] * f;
    }
    m = m_all;
  }
  if (!live) return;
  const float inv = 1.0f / l;
  float *out = a.out + orow * sh.D + c * VEC;
  if (VEC == 4) {
    *reinterpret_cast<f32x4 *>(out) = f32x4{acc[0] * inv, acc[1] * inv, acc[2] * inv, acc[3] * inv};
  } else {
#pragma unroll
    for (int i = 0; i < VEC; ++i) out[i] = acc[i] * inv;
  }
  if (a.lse && c == 0) a.lse[orow] = (m + __builtin_log2f(l)) * 0.6931471805599453f;
}

// ---- append scatter / gather -----------------------------------------------------------------
template <int KV, int LAYOUT>
__global__ __launch_bounds__(256) void spex_scatter_kv_kernel(ScatterArgs a, Shape sh) {
  typedef typename std::conditional<KV == kF32, float,
                                    typename std::conditional<KV == kBF16, uint16_t, uint8_t>::type>::type T;
  const int D = sh.D, P = sh.P, H = sh.Hkv;
  const int64_t total = static_cast<int64_t>(a.n_pages) * H * P * D;
  const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (tid >= total) return;
  const int d = static_cast<int>(tid % D);
  const int slot = static_cast<int>((tid / D) % P);
  const int g = static_cast<int>((tid / (static_cast<int64_t>(D) * P)) % H);
  const int pi = static_cast<int>(tid / (static_cast<int64_t>(D) * P * H));
  const bool is_new = pi > 0 || a.first_page_is_new;
  const int tok = pi * P + slot - a.first_slot;  // index among the tokens of this launch
  const int64_t tile = (static_cast<int64_t>(a.page_ids[pi]) * sh.page_tiles + g);
  const int sidx = a.page_ids[pi] * H + g;
  const int64_t tile_elems = static_cast<int64_t>(P) * D;
  T *kp = static_cast<T *>(a.k_pool) + tile * tile_elems + k_offset<KV, LAYOUT>(slot, d, D);
  T *vp = static_cast<T *>(a.v_pool) + tile * tile_elems + v_offset<KV, LAYOUT>(slot, d, D);
  if (tok >= 0 && tok < a.n_tokens) {
    const int64_t src = (static_cast<int64_t>(tok) * H + g) * D + d;
    *kp = static_cast<const T *>(a.k_src)[src];
    const T vx = static_cast<const T *>(a.v_src)[src];
    *vp = v_is_f16<KV, LAYOUT>() ? static_cast<T>(bf16_bits_to_f16_bits(static_cast<uint16_t>(vx))) : vx;
  } else if (tok >= a.n_tokens && is_new) {
    *kp = T(0);
    *vp = T(0);
  }
  if (KV == kFP8 && is_new && d == 0 && slot == 0) {
    const int idx_new = pi - (a.first_page_is_new ? 0 : 1);
    a.k_scale[sidx] = a.k_scale_src[idx_new * H + g];
    a.v_scale[sidx] = a.v_scale_src[idx_new * H + g];
  }
}

// fp32 -> OCP e4m3fn code, round to nearest even, saturating at +-448 (0x7E / 0xFE); NaN -> 0x7F
// with the sign.  Integer arithmetic on the bit pattern, so the result does not depend on
// floating-point compile flags.  Normal range (|y| >= 2^-6): the fp32 mantissa is rounded to 3
// bits with the usual add-half-and-LSB trick, a carry moves into the exponent by itself.  Below
// that the grid is the multiples of 2^-9, and 8 * 2^-9 is the smallest normal (code 0x08).
__device__ __forceinline__ uint32_t encode_e4m3(float y) {
  const uint32_t u = __builtin_bit_cast(uint32_t, y);
  const uint32_t sign = (u >> 24) & 0x80u, a = u & 0x7fffffffu;
  uint32_t code;
  if (a > 0x7f800000u) {
    code = 0x7fu;
  } else if (a >= 0x43e00000u) {  // 448.0f and above (infinity included)
    code = 0x7eu;
  } else if (a >= 0x3c800000u) {  // 2^-6
    const uint32_t r = a + 0x7ffffu + ((a >> 20) & 1u);
    code = (((r >> 23) - 120u) << 3) | ((r >> 20) & 7u);
  } else {
    code = static_cast<uint32_t>(__builtin_rintf(__builtin_bit_cast(float, a) * 512.0f));
  }
  return code | sign;
}

// A run of bf16 tokens of one node into an fp8 pool, quantised on the way: one workgroup per
// (page, kv head).  For a page this append starts, the workgroup first takes the largest magnitude
// of the tokens it puts there, separately for K and V, and sets scale = max(amax / 448, 2^-40);
// a page that was partially filled before keeps its scale.  Then code = e4m3(x * (1 / scale)).
// Unused slots of a started page are zeroed.  Inputs must be finite.
template <int LAYOUT>
__global__ __launch_bounds__(256) void spex_scatter_quant_kernel(ScatterArgs a, Shape sh) {
  const int D = sh.D, P = sh.P, H = sh.Hkv;
  const int g = blockIdx.x % H, pi = blockIdx.x / H;
  const bool is_new = pi > 0 || a.first_page_is_new;
  const int page = a.page_ids[pi];
  const int sidx = page * H + g;
  const uint16_t *ksrc = static_cast<const uint16_t *>(a.k_src), *vsrc = static_cast<const uint16_t *>(a.v_src);
  auto widen = [](uint16_t b) { return __builtin_bit_cast(float, static_cast<uint32_t>(b) << 16); };
  __shared__ float red[2][4];
  float ks, vs;
  if (is_new) {  // uniform over the workgroup
    float ka = 0.f, va = 0.f;
    for (int e = threadIdx.x; e < P * D; e += 256) {
      const int tok = pi * P + e / D - a.first_slot;
      if (tok >= 0 && tok < a.n_tokens) {
        const int64_t src = (static_cast<int64_t>(tok) * H + g) * D + e % D;
        ka = fmaxf(ka, __builtin_fabsf(widen(ksrc[src])));
        va = fmaxf(va, __builtin_fabsf(widen(vsrc[src])));
      }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      ka = fmaxf(ka, __shfl_xor(ka, o));
      va = fmaxf(va, __shfl_xor(va, o));
    }
    if ((threadIdx.x & 63) == 0) {
      red[0][threadIdx.x >> 6] = ka;
      red[1][threadIdx.x >> 6] = va;
    }
    __syncthreads();
    ka = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
    va = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3]));
    ks = fmaxf(ka / 448.0f, 0x1p-40f);
    vs = fmaxf(va / 448.0f, 0x1p-40f);
    if (threadIdx.x == 0) {
      a.k_scale[sidx] = ks;
      a.v_scale[sidx] = vs;
    }
  } else {
    ks = a.k_scale[sidx];
    vs = a.v_scale[sidx];
  }
  const float kinv = 1.0f / ks, vinv = 1.0f / vs;
  const int64_t tile = (static_cast<int64_t>(page) * sh.page_tiles + g) * (static_cast<int64_t>(P) * D);
  uint8_t *kp = static_cast<uint8_t *>(a.k_pool) + tile, *vp = static_cast<uint8_t *>(a.v_pool) + tile;
  for (int e = threadIdx.x; e < P * D; e += 256) {
    const int slot = e / D, d = e % D;
    const int tok = pi * P + slot - a.first_slot;
    if (tok >= 0 && tok < a.n_tokens) {
      const int64_t src = (static_cast<int64_t>(tok) * H + g) * D + d;
      kp[k_offset<kFP8, LAYOUT>(slot, d, D)] = static_cast<uint8_t>(encode_e4m3(widen(ksrc[src]) * kinv));
      vp[v_offset<kFP8, LAYOUT>(slot, d, D)] = static_cast<uint8_t>(encode_e4m3(widen(vsrc[src]) * vinv));
    } else if (tok >= a.n_tokens && is_new) {
      kp[k_offset<kFP8, LAYOUT>(slot, d, D)] = 0;
      vp[v_offset<kFP8, LAYOUT>(slot, d, D)] = 0;
    }
  }
}

// ---- whole pages in and out ---------------------------------------------------------------------
// One workgroup per (page, kv head).  Both sides are bound by memory, and by the launch for a step
// of a few pages, so every access of a tile or of a token's row is 16 bytes (8 where an fp8 chunk
// has to be put together), V crosses LDS because a tile holds it token-minor, and one launch takes
// up to kMaxPagesPerScatter pages.  The element kernels above moved 2 bytes per access and
// 64 pages per launch; they remain for rows or buffers that are not 16-byte aligned.
// Slots [lo, fill) of the page are written: tokens up to hi, zeros from there to the end of a page
// the append starts.
struct PageSpan {
  int pi, g, lo, hi, fill, tok0;  // token of slot s: s - tok0
  bool is_new;
};
__device__ __forceinline__ PageSpan page_span(const ScatterArgs &a, const Shape &sh) {
  PageSpan s;
  s.g = static_cast<int>(blockIdx.x) % sh.Hkv;
  s.pi = static_cast<int>(blockIdx.x) / sh.Hkv;
  s.is_new = s.pi > 0 || a.first_page_is_new;
  s.tok0 = a.first_slot - s.pi * sh.P;
  s.lo = s.pi == 0 ? a.first_slot : 0;
  s.hi = min(sh.P, s.tok0 + a.n_tokens);
  s.fill = s.is_new ? sh.P : s.hi;
  return s;
}

__device__ __forceinline__ uint16_t half_word(const u32x4 &v, int i) {
  return static_cast<uint16_t>(v[i >> 1] >> (16 * (i & 1)));
}

// Page scales of a quantising append: from the largest magnitudes of the workgroup's tokens for a
// page it starts, else the page's own.  Also writes the scales of a started page.
struct Scales {
  float k, v;
};
__device__ __forceinline__ Scales quant_scales(const ScatterArgs &a, bool is_new, int sidx, float ka, float va) {
  __shared__ float red[2][4];
  Scales s;
  if (is_new) {  // uniform over the workgroup
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
      ka = fmaxf(ka, __shfl_xor(ka, o));
      va = fmaxf(va, __shfl_xor(va, o));
    }
    if ((threadIdx.x & 63) == 0) {
      red[0][threadIdx.x >> 6] = ka;
      red[1][threadIdx.x >> 6] = va;
    }
    __syncthreads();
    ka = fmaxf(fmaxf(red[0][0], red[0][1]), fmaxf(red[0][2], red[0][3]));
    va = fmaxf(fmaxf(red[1][0], red[1][1]), fmaxf(red[1][2], red[1][3]));
    s.k = fmaxf(ka / 448.0f, 0x1p-40f);
    s.v = fmaxf(va / 448.0f, 0x1p-40f);
    if (threadIdx.x == 0) {
      a.k_scale[sidx] = s.k;
      a.v_scale[sidx] = s.v;
    }
  } else {
    s.k = a.k_scale[sidx];
    s.v = a.v_scale[sidx];
  }
  return s;
}
__device__ __forceinline__ float abs_max8(const u32x4 &x) {
  float m = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) m = fmaxf(m, __builtin_fabsf(bf16_bits_to_float(half_word(x, i))));
  return m;
}
__device__ __forceinline__ u32x2 encode8(const u32x4 &x, float inv) {
  u32x2 r = {0, 0};
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i >> 2] |= encode_e4m3(bf16_bits_to_float(half_word(x, i)) * inv) << (8 * (i & 3));
  return r;
}

// Tiled pools.  bf16: K chunks of 8 dims of a token go straight to their place, V through LDS as
// fp16.  fp8: K and V codes (given, or encoded here with QUANT) through LDS.
template <int KV, int D, bool QUANT>
__global__ __launch_bounds__(256) void spex_write_tiles_kernel(ScatterArgs a, Shape sh) {
  constexpr bool FP8 = KV == kFP8;
  constexpr int CH = (FP8 && !QUANT) ? 16 : 8;       // elements per 16-byte piece of a source row
  constexpr int ESZ = FP8 ? 1 : 2, SSZ = (FP8 && !QUANT) ? 1 : 2;
  constexpr int N = 16 * D / CH;                      // source pieces of a page, <= 256
  constexpr int ROW = D * ESZ + 16;                   // LDS bytes per token
  __shared__ __attribute__((aligned(16))) char ldsk[FP8 ? 16 * ROW : 16];
  __shared__ __attribute__((aligned(16))) char ldsv[16 * ROW];
  const PageSpan ps = page_span(a, sh);
  const int page = a.page_ids[ps.pi], H = sh.Hkv, tid = threadIdx.x;
  char *kt = static_cast<char *>(a.k_pool) + (static_cast<int64_t>(page) * sh.page_tiles + ps.g) * (16 * D * ESZ);
  char *vt = static_cast<char *>(a.v_pool) + (static_cast<int64_t>(page) * sh.page_tiles + ps.g) * (16 * D * ESZ);
  const int slot = tid / (D / CH), d = tid % (D / CH) * CH;
  u32x4 kx = {0, 0, 0, 0}, vx = {0, 0, 0, 0};
  if (tid < N && slot >= ps.lo && slot < ps.hi) {
    const int64_t src = ((static_cast<int64_t>(slot - ps.tok0) * H + ps.g) * D + d) * SSZ;
    kx = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.k_src) + src);
    vx = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(a.v_src) + src);
  }
  const int sidx = page * H + ps.g;
  if (QUANT) {
    const Scales s = quant_scales(a, ps.is_new, sidx, abs_max8(kx), abs_max8(vx));
    if (tid < N) {  // zeros of unused slots encode to zero codes
      *reinterpret_cast<u32x2 *>(ldsk + slot * ROW + d) = encode8(kx, 1.0f / s.k);
      *reinterpret_cast<u32x2 *>(ldsv + slot * ROW + d) = encode8(vx, 1.0f / s.v);
    }
  } else if (FP8) {
    if (tid < N) {
      *reinterpret_cast<u32x4 *>(ldsk + slot * ROW + d) = kx;
      *reinterpret_cast<u32x4 *>(ldsv + slot * ROW + d) = vx;
    }
    if (ps.is_new && tid == 0) {
      const int idx_new = ps.pi - (a.first_page_is_new ? 0 : 1);
      a.k_scale[sidx] = a.k_scale_src[idx_new * H + ps.g];
      a.v_scale[sidx] = a.v_scale_src[idx_new * H + ps.g];
    }
  } else if (tid < N) {
    if (slot >= ps.lo && slot < ps.fill)
      *reinterpret_cast<u32x4 *>(kt + 2 * k_offset<KV, kMfmaTiled>(slot, d, D)) = kx;
    u32x4 h;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      h[i] = bf16_bits_to_f16_bits(half_word(vx, 2 * i)) | static_cast<uint32_t>(bf16_bits_to_f16_bits(half_word(vx, 2 * i + 1))) << 16;
    *reinterpret_cast<u32x4 *>(ldsv + slot * ROW + 2 * d) = h;
  }
  __syncthreads();
  // 16-byte pieces of the tiles, in memory order
  constexpr int NT = 16 * D * ESZ / 16;
  if (tid >= NT) return;
  if (FP8) {
    const int half = tid / (D / 2), rem = tid % (D / 2), s = rem / 32, j = rem / 8 % 4, tt = rem % 8;
    const int t = (tt >> 2) * 8 + 4 * half + (tt & 3);
    if (t >= ps.lo && t < ps.fill) {
      const u32x2 lo = *reinterpret_cast<const u32x2 *>(ldsk + t * ROW + 64 * s + 8 * j);
      const u32x2 hi = *reinterpret_cast<const u32x2 *>(ldsk + t * ROW + 64 * s + 32 + 8 * j);
      *reinterpret_cast<u32x4 *>(kt + 16 * tid) = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
    const int vd = tid / 32 * 32 + tid % 16, t0 = tid / 16 % 2 * 8;  // dims vd and vd + 16 of tokens t0 .. t0 + 7
    uint32_t b[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 16; ++i)
      b[i >> 2] |= static_cast<uint32_t>(static_cast<uint8_t>(ldsv[(t0 + (i & 7)) * ROW + vd + (i >> 3) * 16])) << (8 * (i & 3));
    if (t0 >= ps.lo && t0 + 8 <= ps.fill) {
      *reinterpret_cast<u32x4 *>(vt + 16 * tid) = u32x4{b[0], b[1], b[2], b[3]};
    } else {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int t1 = t0 + (i & 7);
        if (t1 >= ps.lo && t1 < ps.fill) vt[16 * tid + i] = static_cast<char>(b[i >> 2] >> (8 * (i & 3)));
      }
    }
  } else {
    const int vd = tid / 32 * 16 + tid % 16, t0 = tid / 16 % 2 * 8;
    uint32_t b[4] = {0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 8; ++i)
      b[i >> 1] |= static_cast<uint32_t>(*reinterpret_cast<const uint16_t *>(ldsv + (t0 + i) * ROW + 2 * vd)) << (16 * (i & 1));
    if (t0 >= ps.lo && t0 + 8 <= ps.fill) {
      *reinterpret_cast<u32x4 *>(vt + 16 * tid) = u32x4{b[0], b[1], b[2], b[3]};
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (t0 + i >= ps.lo && t0 + i < ps.fill)
          *reinterpret_cast<uint16_t *>(vt + 16 * tid + 2 * i) = static_cast<uint16_t>(b[i >> 1] >> (16 * (i & 1)));
    }
  }
}

// Row-major pools: rows are copied (or encoded, 8 dims at a time) as they are.
template <int KV, bool QUANT>
__global__ __launch_bounds__(256) void spex_write_rows_kernel(ScatterArgs a, Shape sh) {
  constexpr int ESZ = RowMajorTraits<KV>::kEsz, SSZ = QUANT ? 2 : ESZ, CH = 16 / SSZ;
  constexpr int kMaxRounds = 64 * 256 / 8 / 256;      // pieces per thread of the largest quantised page
  const PageSpan ps = page_span(a, sh);
  const int page = a.page_ids[ps.pi], H = sh.Hkv, D = sh.D, tid = threadIdx.x;
  const int per = D / CH, n = sh.P * per;
  const int64_t tile = (static_cast<int64_t>(page) * sh.page_tiles + ps.g) * (static_cast<int64_t>(sh.P) * D * ESZ);
  char *kt = static_cast<char *>(a.k_pool) + tile, *vt = static_cast<char *>(a.v_pool) + tile;
  const int sidx = page * H + ps.g;
  auto source = [&](int c, const void *base) {
    const int slot = c / per;
    u32x4 x = {0, 0, 0, 0};
    if (slot >= ps.lo && slot < ps.hi)
      x = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(base) +
                                           ((static_cast<int64_t>(slot - ps.tok0) * H + ps.g) * D + c % per * CH) * SSZ);
    return x;
  };
  if (QUANT) {
    u32x4 kx[kMaxRounds], vx[kMaxRounds];
    float ka = 0.f, va = 0.f;
#pragma unroll
    for (int r = 0; r < kMaxRounds; ++r) {
      kx[r] = vx[r] = u32x4{0, 0, 0, 0};
      if (r * 256 + tid < n) {
        kx[r] = source(r * 256 + tid, a.k_src);
        vx[r] = source(r * 256 + tid, a.v_src);
      }
      ka = fmaxf(ka, abs_max8(kx[r]));
      va = fmaxf(va, abs_max8(vx[r]));
    }
    const Scales s = quant_scales(a, ps.is_new, sidx, ka, va);
#pragma unroll
    for (int r = 0; r < kMaxRounds; ++r) {
      const int c = r * 256 + tid, slot = c / per;
      if (c < n && slot >= ps.lo && slot < ps.fill) {
        *reinterpret_cast<u32x2 *>(kt + c * 8) = encode8(kx[r], 1.0f / s.k);
        *reinterpret_cast<u32x2 *>(vt + c * 8) = encode8(vx[r], 1.0f / s.v);
      }
    }
  } else {
    for (int c = tid; c < n; c += 256) {
      const int slot = c / per;
      const u32x4 kx = source(c, a.k_src), vx = source(c, a.v_src);
      if (slot >= ps.lo && slot < ps.fill) {
        *reinterpret_cast<u32x4 *>(kt + c * 16) = kx;
        *reinterpret_cast<u32x4 *>(vt + c * 16) = vx;
      }
    }
    if (KV == kFP8 && ps.is_new && tid == 0) {
      const int idx_new = ps.pi - (a.first_page_is_new ? 0 : 1);
      a.k_scale[sidx] = a.k_scale_src[idx_new * H + ps.g];
      a.v_scale[sidx] = a.v_scale_src[idx_new * H + ps.g];
    }
  }
}

// Tokens of a page back in logical order (the inverse of the two kernels above).
template <int KV, int LAYOUT>
__global__ __launch_bounds__(256) void spex_read_pages_kernel(GatherArgs a, Shape sh) {
  constexpr bool TILED = LAYOUT == kMfmaTiled;
  constexpr int ESZ = RowMajorTraits<KV>::kEsz, CH = 16 / ESZ;
  constexpr int kRowMax = 128 * ESZ + 16;             // LDS bytes per token, tiled pools
  __shared__ __attribute__((aligned(16))) char ldsv[TILED ? 16 * kRowMax : 16];
  const int H = sh.Hkv, D = sh.D, tid = threadIdx.x;
  const int g = static_cast<int>(blockIdx.x) % H, pi = static_cast<int>(blockIdx.x) / H;
  const int page = a.page_ids[pi], tok0 = a.first_slot - pi * sh.P;
  const int lo = pi == 0 ? a.first_slot : 0, hi = min(sh.P, tok0 + a.n_tokens);
  const int64_t tile = (static_cast<int64_t>(page) * sh.page_tiles + g) * (static_cast<int64_t>(sh.P) * D * ESZ);
  const char *kt = static_cast<const char *>(a.k_pool) + tile, *vt = static_cast<const char *>(a.v_pool) + tile;
  char *ko = static_cast<char *>(a.k_out), *vo = static_cast<char *>(a.v_out);
  auto dst = [&](int slot, int d) { return ((static_cast<int64_t>(slot - tok0) * H + g) * D + d) * ESZ; };
  if (KV == kFP8 && tid < sh.P && tid >= lo && tid < hi) {
    const int64_t at = static_cast<int64_t>(tid - tok0) * H + g;
    if (a.k_scale_out) a.k_scale_out[at] = a.k_scale[page * H + g];
    if (a.v_scale_out) a.v_scale_out[at] = a.v_scale[page * H + g];
  }
  if (!TILED) {
    const int per = D / CH, n = sh.P * per;
    for (int c = tid; c < n; c += 256) {
      const int slot = c / per;
      if (slot < lo || slot >= hi) continue;
      *reinterpret_cast<u32x4 *>(ko + dst(slot, c % per * CH)) = *reinterpret_cast<const u32x4 *>(kt + c * 16);
      *reinterpret_cast<u32x4 *>(vo + dst(slot, c % per * CH)) = *reinterpret_cast<const u32x4 *>(vt + c * 16);
    }
    return;
  }
  const int n = 16 * D * ESZ / 16, row = D * ESZ + 16;  // <= 256 pieces of 16 bytes
  if (tid < n) {
    const u32x4 kx = *reinterpret_cast<const u32x4 *>(kt + 16 * tid), vx = *reinterpret_cast<const u32x4 *>(vt + 16 * tid);
    if (KV == kFP8) {
      const int half = tid / (D / 2), rem = tid % (D / 2), s = rem / 32, j = rem / 8 % 4, tt = rem % 8;
      const int t = (tt >> 2) * 8 + 4 * half + (tt & 3);
      if (t >= lo && t < hi) {
        *reinterpret_cast<u32x2 *>(ko + dst(t, 64 * s + 8 * j)) = u32x2{kx[0], kx[1]};
        *reinterpret_cast<u32x2 *>(ko + dst(t, 64 * s + 32 + 8 * j)) = u32x2{kx[2], kx[3]};
      }
      const int vd = tid / 32 * 32 + tid % 16, t0 = tid / 16 % 2 * 8;
#pragma unroll
      for (int i = 0; i < 16; ++i)
        ldsv[(t0 + (i & 7)) * row + vd + (i >> 3) * 16] = static_cast<char>(vx[i >> 2] >> (8 * (i & 3)));
    } else {
      const int half = tid / D, rem = tid % D, s = rem / 32, j = rem / 8 % 4, tt = rem % 8;
      const int t = (tt >> 2) * 8 + 4 * half + (tt & 3);
      if (t >= lo && t < hi) *reinterpret_cast<u32x4 *>(ko + dst(t, 32 * s + 8 * j)) = kx;
      const int vd = tid / 32 * 16 + tid % 16, t0 = tid / 16 % 2 * 8;
#pragma unroll
      for (int i = 0; i < 8; ++i) *reinterpret_cast<uint16_t *>(ldsv + (t0 + i) * row + 2 * vd) = f16_bits_to_bf16_bits(half_word(vx, i));
    }
  }
  __syncthreads();
  const int slot = tid / (D / CH), d = tid % (D / CH) * CH;
  if (tid < n && slot >= lo && slot < hi)
    *reinterpret_cast<u32x4 *>(vo + dst(slot, d)) = *reinterpret_cast<const u32x4 *>(ldsv + slot * row + d * ESZ);
}

// One appended token per node: thread = (node, kv head, dim).  Writes the token's K and V element
// into its slot; where the token starts a page it also zeroes the page's other slots (so that
// nothing stale can be read from a partial page) and stores the page's fp8 scales.  The first
// n_patches threads also write one length patch each into the device copy of the cached plan.  QUANT (fp8
// pools): the source holds bf16 values and the code is encode_e4m3(x * (1 / scale)), scale being
// the one given for a page the token starts, else the one the page already has.
template <int KV, int LAYOUT, bool QUANT>
__global__ __launch_bounds__(256) void spex_append_tokens_kernel(AppendTokensArgs a, Shape sh) {
  typedef typename std::conditional<KV == kF32, float,
                                    typename std::conditional<KV == kBF16, uint16_t, uint8_t>::type>::type T;
  const int D = sh.D, P = sh.P, H = sh.Hkv;
  const int64_t total = static_cast<int64_t>(a.n_nodes) * H * D;
  const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (tid >= total) return;
  // the cached launch lists follow the append in the same launch: new valid counts and limits
  if (tid < a.n_patches) a.plan[a.patches[2 * tid]] = a.patches[2 * tid + 1];
  const int d = static_cast<int>(tid % D);
  const int g = static_cast<int>((tid / D) % H);
  const int node = static_cast<int>(tid / (static_cast<int64_t>(D) * H));
  const int page = a.dst[2 * node], code = a.dst[2 * node + 1];
  const int slot = code & 0xff;
  const bool is_new = (code >> 8) != 0;
  const int64_t tile = (static_cast<int64_t>(page) * sh.page_tiles + g) * (static_cast<int64_t>(P) * D);
  T *kp = static_cast<T *>(a.k_pool) + tile, *vp = static_cast<T *>(a.v_pool) + tile;
  T kx, vx;
  if (QUANT) {
    const float ks = is_new ? a.k_scale_src[node * H + g] : a.k_scale[page * H + g];
    const float vs = is_new ? a.v_scale_src[node * H + g] : a.v_scale[page * H + g];
    const float kf = __builtin_bit_cast(float, static_cast<uint32_t>(static_cast<const uint16_t *>(a.k_src)[tid]) << 16);
    const float vf = __builtin_bit_cast(float, static_cast<uint32_t>(static_cast<const uint16_t *>(a.v_src)[tid]) << 16);
    kx = static_cast<T>(encode_e4m3(kf * (1.0f / ks)));
    vx = static_cast<T>(encode_e4m3(vf * (1.0f / vs)));
  } else {
    kx = static_cast<const T *>(a.k_src)[tid];
    vx = static_cast<const T *>(a.v_src)[tid];
    if (v_is_f16<KV, LAYOUT>()) vx = static_cast<T>(bf16_bits_to_f16_bits(static_cast<uint16_t>(vx)));
  }
  kp[k_offset<KV, LAYOUT>(slot, d, D)] = kx;
  vp[v_offset<KV, LAYOUT>(slot, d, D)] = vx;
  if (is_new) {
    for (int s2 = 0; s2 < P; ++s2)
      if (s2 != slot) {
        kp[k_offset<KV, LAYOUT>(s2, d, D)] = T(0);
        vp[v_offset<KV, LAYOUT>(s2, d, D)] = T(0);
      }
    if (KV == kFP8 && d == 0) {
      a.k_scale[page * H + g] = a.k_scale_src[node * H + g];
      a.v_scale[page * H + g] = a.v_scale_src[node * H + g];
    }
  }
}

template <int KV, int LAYOUT>
__global__ __launch_bounds__(256) void spex_gather_kv_kernel(GatherArgs a, Shape sh) {
  typedef typename std::conditional<KV == kF32, float,
                                    typename std::conditional<KV == kBF16, uint16_t, uint8_t>::type>::type T;
  const int D = sh.D, P = sh.P, H = sh.Hkv;
  const int64_t total = static_cast<int64_t>(a.n_tokens) * H * D;
  const int64_t tid = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (tid >= total) return;
  const int d = static_cast<int>(tid % D);
  const int g = static_cast<int>((tid / D) % H);
  const int tok = static_cast<int>(tid / (static_cast<int64_t>(D) * H));
  const int pi = (tok + a.first_slot) / P;
  const int slot = (tok + a.first_slot) % P;
  const int64_t tile = (static_cast<int64_t>(a.page_ids[pi]) * sh.page_tiles + g);
  const int sidx = a.page_ids[pi] * H + g;
  const int64_t tile_elems = static_cast<int64_t>(P) * D;
  static_cast<T *>(a.k_out)[tid] =
      static_cast<const T *>(a.k_pool)[tile * tile_elems + k_offset<KV, LAYOUT>(slot, d, D)];
  const T vx = static_cast<const T *>(a.v_pool)[tile * tile_elems + v_offset<KV, LAYOUT>(slot, d, D)];
  static_cast<T *>(a.v_out)[tid] =
      v_is_f16<KV, LAYOUT>() ? static_cast<T>(f16_bits_to_bf16_bits(static_cast<uint16_t>(vx))) : vx;
  if (KV == kFP8 && d == 0) {
    if (a.k_scale_out) a.k_scale_out[static_cast<int64_t>(tok) * H + g] = a.k_scale[sidx];
    if (a.v_scale_out) a.v_scale_out[static_cast<int64_t>(tok) * H + g] = a.v_scale[sidx];
  }
}

template <int KV, int QT>
hipError_t launch_generic(const Shape &sh, const AttnArgs &a, int rows_per_item, hipStream_t stream) {
  const dim3 grid(a.n_items, rows_per_item), block(64);
  if (sh.layout == kMfmaTiled)
    hipLaunchKernelGGL((spex_generic_attn_kernel<KV, QT, kMfmaTiled>), grid, block, 0, stream, a, sh,
                       rows_per_item);
  else
    hipLaunchKernelGGL((spex_generic_attn_kernel<KV, QT, kRowMajor>), grid, block, 0, stream, a, sh,
                       rows_per_item);
  return hipGetLastError();
}

}  // namespace

bool has_mfma_kernel(const Shape &sh) {
  return sh.layout == kMfmaTiled && sh.q_dtype == kBF16 &&
         (sh.kv_dtype == kBF16 || sh.kv_dtype == kFP8) && sh.P == 16 && (sh.D == 64 || sh.D == 128);
}

hipError_t launch_generic_attention(const Shape &sh, const AttnArgs &a, int rows_per_item, hipStream_t stream) {
  if (a.n_items <= 0) return hipSuccess;
  if (sh.kv_dtype == kF32 && sh.q_dtype == kF32) return launch_generic<kF32, kF32>(sh, a, rows_per_item, stream);
  if (sh.kv_dtype == kBF16 && sh.q_dtype == kBF16) return launch_generic<kBF16, kBF16>(sh, a, rows_per_item, stream);
  if (sh.kv_dtype == kFP8 && sh.q_dtype == kBF16) return launch_generic<kFP8, kBF16>(sh, a, rows_per_item, stream);
  return hipErrorInvalidValue;
}

bool has_rowmajor_kernel(const Shape &sh, const AttnArgs &a) {
  // 16-byte loads of whole rows: rows and buffers must be 16-byte aligned (fp8 up to 128 dims: rows 8-byte
  // aligned, see kRowHalf); four tokens of a lane must share a page.  Anything else goes to the generic kernel.
  const int ch = sh.kv_dtype == kF32 ? 4 : (sh.kv_dtype == kBF16 || sh.D <= 128 ? 8 : 16);
  const bool types = sh.kv_dtype == kF32 ? sh.q_dtype == kF32 : sh.q_dtype == kBF16;
  auto aligned = [](const void *x) { return (reinterpret_cast<uintptr_t>(x) & 15) == 0; };
  return sh.layout == kRowMajor && types && sh.P >= 4 && sh.D % ch == 0 && sh.D <= 256 && aligned(a.k_pool) &&
         aligned(a.v_pool) && aligned(a.q);
}

template <int KV>
static hipError_t launch_rowmajor_kv(const Shape &sh, const AttnArgs &a, const SplitLists &ls, int n_wg, hipStream_t stream) {
  const dim3 grid(n_wg), block(256);
  const auto launch = [&](auto dp) {
    constexpr int DP = decltype(dp)::value;
    if (sh.D == DP) {
      hipLaunchKernelGGL((spex_rowmajor_attn_kernel<KV, DP, kRowFull>), grid, block, 0, stream, a, sh, ls);
      return;
    }
    if constexpr (KV == kFP8 && DP <= 128)
      if (sh.D % 16 != 0) {
        hipLaunchKernelGGL((spex_rowmajor_attn_kernel<KV, DP, kRowHalf>), grid, block, 0, stream, a, sh, ls);
        return;
      }
    hipLaunchKernelGGL((spex_rowmajor_attn_kernel<KV, DP, kRowAny>), grid, block, 0, stream, a, sh, ls);
  };
  if (sh.D <= 64)
    launch(std::integral_constant<int, 64>());
  else if (sh.D <= 128)
    launch(std::integral_constant<int, 128>());
  else
    launch(std::integral_constant<int, 256>());
  return hipGetLastError();
}

// rows_per_wg: rows of an item one workgroup takes.  n_wg < 0: too many.
static SplitLists make_lists(const ItemLists &l, int rows_per_wg, int64_t *n_wg) {
  SplitLists ls{};
  *n_wg = 0;
  for (int k = 0; k < SplitLists::kLists; ++k) {
    ls.items[k] = l.items[k];
    ls.n_items[k] = l.n_items[k] > 0 ? l.n_items[k] : 1;  // a divisor
    ls.span[k] = l.span[k];
    *n_wg += static_cast<int64_t>(l.n_items[k]) * ((l.span[k] + rows_per_wg - 1) / rows_per_wg);
    ls.wg_end[k] = static_cast<int32_t>(*n_wg);
    if (*n_wg > INT32_MAX) {
      *n_wg = -1;
      break;
    }
  }
  return ls;
}

template <int KV, int D, int NT, SplitForm FORM>
static hipError_t launch_split_form(const Shape &sh, const AttnArgs &a, const SplitLists &ls, int n_wg, hipStream_t stream) {
  const dim3 grid(n_wg), block(256);
  if (a.qt_mask)  // draft token trees: visibility masks per query
    hipLaunchKernelGGL((spex_split_attn_kernel<KV, D, NT, true, FORM>), grid, block, 0, stream, a, sh, ls);
  else
    hipLaunchKernelGGL((spex_split_attn_kernel<KV, D, NT, false, FORM>), grid, block, 0, stream, a, sh, ls);
  return hipGetLastError();
}

template <int KV, int D, int NT>
static hipError_t launch_split_nt(const Shape &sh, const AttnArgs &a, const ItemLists &l, hipStream_t stream) {
  int64_t n_wg = 0;
  const SplitLists ls = make_lists(l, l.form == kSplitTiles ? 16 * NT : 128, &n_wg);
  if (n_wg < 0) return hipErrorInvalidValue;
  if (n_wg == 0) return hipSuccess;
  const int n = static_cast<int>(n_wg);
  if (l.form == kSplitTiles) return launch_split_form<KV, D, NT, kSplitTiles>(sh, a, ls, n, stream);
  if constexpr (NT == 1 && !(KV == kBF16 && D == 128))
    if (l.form == kSplitLean && l.n_items[0] == 0) return launch_split_form<KV, D, NT, kSplitLean>(sh, a, ls, n, stream);
  return l.form == kSplitFull ? launch_split_form<KV, D, NT, kSplitFull>(sh, a, ls, n, stream) : hipErrorInvalidValue;
}

template <int KV, int D>
static hipError_t launch_split_d(const Shape &sh, const AttnArgs &a, const ItemLists &l, hipStream_t stream) {
  return l.span[2] <= 16 && l.span[3] <= 16 ? launch_split_nt<KV, D, 1>(sh, a, l, stream) : launch_split_nt<KV, D, 2>(sh, a, l, stream);
}

template <int KV, int D, bool TREE>
static hipError_t launch_phases_tree(const Shape &sh, AttnArgs a, const ItemLists &l, hipStream_t stream) {
  const dim3 block(256);
  for (int k : {2, 0, 1, 3}) {
    if (l.n_items[k] <= 0) continue;
    a.items = l.items[k];
    a.n_items = l.n_items[k];
    const dim3 waves((l.n_items[k] + 3) / 4), groups(l.n_items[k]);
    if (k == 0)
      hipLaunchKernelGGL((spex_coop_attn_kernel<KV, D, 2, TREE>), groups, block, 0, stream, a, sh);
    else if (k == 1)
      hipLaunchKernelGGL((spex_coop_attn_kernel<KV, D, 1, TREE>), groups, block, 0, stream, a, sh);
    else if (k == 2 && l.span[k] <= 16)
      hipLaunchKernelGGL((spex_wave_attn_kernel<KV, D, 1, false, TREE>), waves, block, 0, stream, a, sh);
    else if (k == 2)
      return hipErrorInvalidValue;
    else if (l.span[k] <= 16)
      hipLaunchKernelGGL((spex_wave_attn_kernel<KV, D, 1, true, TREE>), waves, block, 0, stream, a, sh);
    else
      hipLaunchKernelGGL((spex_wave_attn_kernel<KV, D, 2, true, TREE>), waves, block, 0, stream, a, sh);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int KV, int D>
static hipError_t launch_phases_d(const Shape &sh, const AttnArgs &a, const ItemLists &l, hipStream_t stream) {
  return a.qt_mask ? launch_phases_tree<KV, D, true>(sh, a, l, stream) : launch_phases_tree<KV, D, false>(sh, a, l, stream);
}

hipError_t launch_split_phases(const Shape &sh, const AttnArgs &a, const ItemLists &l, hipStream_t stream) {
  if (!has_mfma_kernel(sh) || l.span[0] > 128 || l.span[1] > 64 || l.span[2] > 32 || l.span[3] > 32) return hipErrorInvalidValue;
  if (sh.kv_dtype == kBF16)
    return sh.D == 64 ? launch_phases_d<kBF16, 64>(sh, a, l, stream) : launch_phases_d<kBF16, 128>(sh, a, l, stream);
  return sh.D == 64 ? launch_phases_d<kFP8, 64>(sh, a, l, stream) : launch_phases_d<kFP8, 128>(sh, a, l, stream);
}

hipError_t launch_split(const Shape &sh, const AttnArgs &a, const ItemLists &l, hipStream_t stream) {
  const bool tiled = has_mfma_kernel(sh);
  if (!tiled && !has_rowmajor_kernel(sh, a)) return hipErrorInvalidValue;
  if (l.span[0] > 128 || l.span[1] > 64 || l.span[2] > 32 || l.span[3] > 32) return hipErrorInvalidValue;
  if (tiled && sh.kv_dtype == kBF16)
    return sh.D == 64 ? launch_split_d<kBF16, 64>(sh, a, l, stream) : launch_split_d<kBF16, 128>(sh, a, l, stream);
  if (tiled) return sh.D == 64 ? launch_split_d<kFP8, 64>(sh, a, l, stream) : launch_split_d<kFP8, 128>(sh, a, l, stream);
  int64_t n_wg = 0;
  const SplitLists ls = make_lists(l, 64, &n_wg);
  if (n_wg < 0) return hipErrorInvalidValue;
  if (n_wg == 0) return hipSuccess;
  const int n = static_cast<int>(n_wg);
  if (sh.kv_dtype == kF32) return launch_rowmajor_kv<kF32>(sh, a, ls, n, stream);
  if (sh.kv_dtype == kBF16) return launch_rowmajor_kv<kBF16>(sh, a, ls, n, stream);
  return launch_rowmajor_kv<kFP8>(sh, a, ls, n, stream);
}

template <int KV, int D, int NW, bool TREE>
static hipError_t launch_walk_ntw(const Shape &sh, const WalkArgs &a, int ntw, bool by_tile, hipStream_t stream) {
  const dim3 grid(a.n_items), block(64 * NW);
  // fp8 with two tiles and either type with four; eight wavefronts with four tiles always (straight on,
  // their accumulators spill: 1044 us where one tile in four is touched, by tile 386)
  if (ntw == 1)
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 1, NW, TREE>), grid, block, 0, stream, a, sh);
  else if (ntw == 2 && KV == kFP8 && by_tile)
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 2, NW, TREE, 1, KV == kFP8>), grid, block, 0, stream, a, sh);
  else if (ntw == 2 && NW == 4 && a.cut)
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 2, NW, TREE, 1, false, NW == 4>), grid, block, 0, stream, a, sh);
  else if (ntw == 2)
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 2, NW, TREE>), grid, block, 0, stream, a, sh);
  else if (NW == 8 || by_tile)
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 4, NW, TREE, 1, true>), grid, block, 0, stream, a, sh);
  else
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 4, NW, TREE, 1, NW == 8>), grid, block, 0, stream, a, sh);
  return hipGetLastError();
}

template <int KV, int D, int NW, bool TREE>
static hipError_t launch_walk_halves(const Shape &sh, const WalkArgs &a, int ntw, hipStream_t stream) {
  const dim3 grid(a.n_items), block(64 * NW);
  if (ntw == 1)
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 1, NW, TREE, 2>), grid, block, 0, stream, a, sh);
  else if (ntw == 2 && NW == 8 && a.cut)
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 2, NW, TREE, 2, false, NW == 8>), grid, block, 0, stream, a, sh);
  else if (ntw == 2)
    hipLaunchKernelGGL((spex_tree_walk_kernel<KV, D, 2, NW, TREE, 2>), grid, block, 0, stream, a, sh);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int KV, int D>
static hipError_t launch_walk_nw(const Shape &sh, const WalkArgs &a, int ntw, int waves, bool halves, bool by_tile, hipStream_t stream) {
  if (halves) {  // lists for four wavefronts of rows, walked by eight
    if (waves != 4) return hipErrorInvalidValue;
    return a.qt_mask ? launch_walk_halves<KV, D, 8, true>(sh, a, ntw, stream)
                     : launch_walk_halves<KV, D, 8, false>(sh, a, ntw, stream);
  }
  if (a.qt_mask) {  // draft-tree masks: not in the kernel that splits the path
    if (waves == 2) return hipErrorInvalidValue;
    return waves == 4 ? launch_walk_ntw<KV, D, 4, true>(sh, a, ntw, by_tile, stream)
                      : launch_walk_ntw<KV, D, 8, true>(sh, a, ntw, by_tile, stream);
  }
  // lists for two wavefronts of rows, walked by four: the path is split in two
  if (waves == 2) return launch_walk_halves<KV, D, 4, false>(sh, a, ntw, stream);
  return waves == 4 ? launch_walk_ntw<KV, D, 4, false>(sh, a, ntw, by_tile, stream)
                    : launch_walk_ntw<KV, D, 8, false>(sh, a, ntw, by_tile, stream);
}

hipError_t launch_tree_walk(const Shape &sh, const WalkArgs &a, int ntw, int waves, bool halves, bool by_tile, hipStream_t stream) {
  if (a.n_items <= 0) return hipSuccess;
  if (!has_mfma_kernel(sh) || (ntw != 1 && ntw != 2 && ntw != 4) || (waves != 2 && waves != 4 && waves != 8))
    return hipErrorInvalidValue;
  if (sh.kv_dtype == kBF16)
    return sh.D == 64 ? launch_walk_nw<kBF16, 64>(sh, a, ntw, waves, halves, by_tile, stream)
                      : launch_walk_nw<kBF16, 128>(sh, a, ntw, waves, halves, by_tile, stream);
  return sh.D == 64 ? launch_walk_nw<kFP8, 64>(sh, a, ntw, waves, halves, by_tile, stream)
                    : launch_walk_nw<kFP8, 128>(sh, a, ntw, waves, halves, by_tile, stream);
}

namespace {
// blob[pairs[2i]] = pairs[2i + 1]: brings the device copy of a plan up to date after appends.
__global__ __launch_bounds__(256) void spex_patch_plan_kernel(int32_t *blob, const int32_t *pairs, int n) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) blob[pairs[2 * i]] = pairs[2 * i + 1];
}
}  // namespace

hipError_t launch_patch(int32_t *blob, const int32_t *pairs, int32_t n, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(spex_patch_plan_kernel, dim3((n + 255) / 256), dim3(256), 0, stream, blob, pairs, n);
  return hipGetLastError();
}

hipError_t launch_merge(const Shape &sh, const MergeArgs &args, hipStream_t stream) {
  MergeArgs a = args;
  if (a.n_qtok <= 0) return hipSuccess;
  const MergeShape m = merge_shape(sh.Hkv, sh.G, sh.D, a.n_qtok, a.avg_pieces);
  a.heads_first = m.heads_first;
  a.slice_log2 = m.slice_log2;
  const unsigned n = static_cast<unsigned>((static_cast<int64_t>(a.n_qtok) + m.tokens - 1) / m.tokens), heads = static_cast<unsigned>(sh.Hkv), parts = static_cast<unsigned>(m.parts);
  const dim3 grid = m.heads_first ? dim3(heads, parts, n) : dim3(n, heads, parts), block(m.dv, m.tokens << m.slice_log2, m.rows);
  const auto kernel = m.vec == 4 ? (m.tokens > 1 ? spex_lse_merge_kernel<4, true> : spex_lse_merge_kernel<4, false>)
                                 : (m.tokens > 1 ? spex_lse_merge_kernel<1, true> : spex_lse_merge_kernel<1, false>);
  hipLaunchKernelGGL(kernel, grid, block, 0, stream, a, sh);
  return hipGetLastError();
}

template <int KV>
static hipError_t scatter_layout(const Shape &sh, const ScatterArgs &a, hipStream_t stream) {
  const int64_t total = static_cast<int64_t>(a.n_pages) * sh.Hkv * sh.P * sh.D;
  const dim3 grid(static_cast<unsigned>((total + 255) / 256)), block(256);
  if (sh.layout == kMfmaTiled)
    hipLaunchKernelGGL((spex_scatter_kv_kernel<KV, kMfmaTiled>), grid, block, 0, stream, a, sh);
  else
    hipLaunchKernelGGL((spex_scatter_kv_kernel<KV, kRowMajor>), grid, block, 0, stream, a, sh);
  return hipGetLastError();
}

// 16-byte accesses of token rows and tiles: every buffer and row 16-byte aligned.
static bool aligned16(const void *x) { return (reinterpret_cast<uintptr_t>(x) & 15) == 0; }
static bool wide_rows(const Shape &sh, int src_esz, const void *kp, const void *vp, const void *ks, const void *vs) {
  const int esz = sh.kv_dtype == kF32 ? 4 : (sh.kv_dtype == kBF16 ? 2 : 1);
  // an encoded row needs 8 bytes per 16 of its source; everything else moves 16 as they are
  const bool row = sh.D * src_esz % 16 == 0 && (src_esz != esz || sh.D * esz % 16 == 0);
  return row && aligned16(kp) && aligned16(vp) && aligned16(ks) && aligned16(vs);
}

hipError_t launch_scatter_quantise(const Shape &sh, const ScatterArgs &a, hipStream_t stream) {
  if (a.n_pages <= 0) return hipSuccess;
  if (sh.kv_dtype != kFP8) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>(a.n_pages * sh.Hkv)), block(256);
  if (wide_rows(sh, 2, a.k_pool, a.v_pool, a.k_src, a.v_src)) {
    if (sh.layout != kMfmaTiled)
      hipLaunchKernelGGL((spex_write_rows_kernel<kFP8, true>), grid, block, 0, stream, a, sh);
    else if (sh.D == 64)
      hipLaunchKernelGGL((spex_write_tiles_kernel<kFP8, 64, true>), grid, block, 0, stream, a, sh);
    else
      hipLaunchKernelGGL((spex_write_tiles_kernel<kFP8, 128, true>), grid, block, 0, stream, a, sh);
  } else if (sh.layout == kMfmaTiled) {
    hipLaunchKernelGGL((spex_scatter_quant_kernel<kMfmaTiled>), grid, block, 0, stream, a, sh);
  } else {
    hipLaunchKernelGGL((spex_scatter_quant_kernel<kRowMajor>), grid, block, 0, stream, a, sh);
  }
  return hipGetLastError();
}

template <int KV>
static hipError_t write_tiles(const Shape &sh, const ScatterArgs &a, hipStream_t stream) {
  const dim3 grid(static_cast<unsigned>(a.n_pages * sh.Hkv)), block(256);
  if (sh.D == 64)
    hipLaunchKernelGGL((spex_write_tiles_kernel<KV, 64, false>), grid, block, 0, stream, a, sh);
  else
    hipLaunchKernelGGL((spex_write_tiles_kernel<KV, 128, false>), grid, block, 0, stream, a, sh);
  return hipGetLastError();
}

template <int KV>
static hipError_t write_rows(const Shape &sh, const ScatterArgs &a, hipStream_t stream) {
  const dim3 grid(static_cast<unsigned>(a.n_pages * sh.Hkv)), block(256);
  hipLaunchKernelGGL((spex_write_rows_kernel<KV, false>), grid, block, 0, stream, a, sh);
  return hipGetLastError();
}

hipError_t launch_scatter(const Shape &sh, const ScatterArgs &a, hipStream_t stream) {
  if (a.n_pages <= 0) return hipSuccess;
  const int esz = sh.kv_dtype == kF32 ? 4 : (sh.kv_dtype == kBF16 ? 2 : 1);
  if (wide_rows(sh, esz, a.k_pool, a.v_pool, a.k_src, a.v_src)) {
    if (sh.layout == kMfmaTiled) return sh.kv_dtype == kBF16 ? write_tiles<kBF16>(sh, a, stream) : write_tiles<kFP8>(sh, a, stream);
    switch (sh.kv_dtype) {
      case kF32: return write_rows<kF32>(sh, a, stream);
      case kBF16: return write_rows<kBF16>(sh, a, stream);
      case kFP8: return write_rows<kFP8>(sh, a, stream);
    }
  }
  switch (sh.kv_dtype) {
    case kF32: return scatter_layout<kF32>(sh, a, stream);
    case kBF16: return scatter_layout<kBF16>(sh, a, stream);
    case kFP8: return scatter_layout<kFP8>(sh, a, stream);
  }
  return hipErrorInvalidValue;
}

template <int KV>
static hipError_t gather_layout(const Shape &sh, const GatherArgs &a, hipStream_t stream) {
  if (wide_rows(sh, RowMajorTraits<KV>::kEsz, a.k_pool, a.v_pool, a.k_out, a.v_out)) {
    const dim3 wgrid(static_cast<unsigned>(a.n_pages * sh.Hkv)), wblock(256);
    if (KV != kF32 && sh.layout == kMfmaTiled)  // fp32 pools are row-major
      hipLaunchKernelGGL((spex_read_pages_kernel<KV, KV == kF32 ? kRowMajor : kMfmaTiled>), wgrid, wblock, 0, stream, a, sh);
    else
      hipLaunchKernelGGL((spex_read_pages_kernel<KV, kRowMajor>), wgrid, wblock, 0, stream, a, sh);
    return hipGetLastError();
  }
  const int64_t total = static_cast<int64_t>(a.n_tokens) * sh.Hkv * sh.D;
  const dim3 grid(static_cast<unsigned>((total + 255) / 256)), block(256);
  if (sh.layout == kMfmaTiled)
    hipLaunchKernelGGL((spex_gather_kv_kernel<KV, kMfmaTiled>), grid, block, 0, stream, a, sh);
  else
    hipLaunchKernelGGL((spex_gather_kv_kernel<KV, kRowMajor>), grid, block, 0, stream, a, sh);
  return hipGetLastError();
}

hipError_t launch_gather(const Shape &sh, const GatherArgs &a, hipStream_t stream) {
  if (a.n_tokens <= 0) return hipSuccess;
  switch (sh.kv_dtype) {
    case kF32: return gather_layout<kF32>(sh, a, stream);
    case kBF16: return gather_layout<kBF16>(sh, a, stream);
    case kFP8: return gather_layout<kFP8>(sh, a, stream);
  }
  return hipErrorInvalidValue;
}

template <int KV, bool QUANT>
static hipError_t append_tokens_layout(const Shape &sh, const AppendTokensArgs &a, hipStream_t stream) {
  const int64_t total = static_cast<int64_t>(a.n_nodes) * sh.Hkv * sh.D;
  const dim3 grid(static_cast<unsigned>((total + 255) / 256)), block(256);
  if (sh.layout == kMfmaTiled)
    hipLaunchKernelGGL((spex_append_tokens_kernel<KV, kMfmaTiled, QUANT>), grid, block, 0, stream, a, sh);
  else
    hipLaunchKernelGGL((spex_append_tokens_kernel<KV, kRowMajor, QUANT>), grid, block, 0, stream, a, sh);
  return hipGetLastError();
}

hipError_t launch_append_tokens(const Shape &sh, const AppendTokensArgs &a, hipStream_t stream) {
  if (a.n_nodes <= 0) return hipSuccess;
  if (a.quantise)
    return sh.kv_dtype == kFP8 ? append_tokens_layout<kFP8, true>(sh, a, stream) : hipErrorInvalidValue;
  switch (sh.kv_dtype) {
    case kF32: return append_tokens_layout<kF32, false>(sh, a, stream);
    case kBF16: return append_tokens_layout<kBF16, false>(sh, a, stream);
    case kFP8: return append_tokens_layout<kFP8, false>(sh, a, stream);
  }
  return hipErrorInvalidValue;
}

}  // namespace spex
