// disc_device.h -- hand-written, shape-generic kernel schedules for gfx950 (CDNA4).
//
// This header is compiled at pattern-registration time together with ONE generated
// `struct Pat` that holds the fused per-element expression of the pattern.  Everything
// that decides performance lives here and is written by hand: how rows are mapped to
// lanes, how data moves through registers / LDS, how reductions are combined.  The
// schedules never see a shape as a compile-time constant; every extent arrives in the
// kernel-argument block that the host fills at launch (the paper's host-side shape
// calculation and launch-dimension selection, Sections 4.2.1 and 4.3).  (The one exception is
// the single-shape module built for the gap-to-static comparison, see DISC_STATIC_ARGS.)
//
// The two templates of Section 4.3 -- loop fusion, and input fusion rooted at a reduction -- are
// kloop_kernel and the row_* / col_* kernels; each exists in
// several versions (vector / scalar access, 32 / 64-bit index, register-resident / streamed
// row, ...) which the host selects per incoming shape.
//
// Interface expected from the generated `Pat` (all members static, __device__, inlined):
//   struct Args            kernel-argument block (pointers, extents, fast-division constants)
//   struct RowCtx          per-row state: operand base offsets and per-row values
//   template<int V> struct Slot      V consecutive elements of every per-element operand
//   template<int V> struct OutSlot   V consecutive elements of every per-element output
//   row_begin(A,row,rc)                        fill RowCtx for `row` (loads per-row operands)
//   load<V>(A,rc,col,span,slot)                load a slot (span: elements of the slot inside the row)
//   template<int P> struct Acc                 accumulator of reduction phase P
//   acc_init<P>(acc)  acc_merge<P>(a,b)  acc_xchg<P,S>(acc)   (S: lane_xchg step)
//   template<int V> struct Keep                per-element values carried between phases
//   phase<P,V,KEEP>(A,acc,slot,keep,span,col,rc)   fold one slot into acc (row reduce);
//                                              KEEP=false recomputes instead of using `keep`
//   accum<P,V>(A,acc,slot,e,col,rc)            fold element e of a slot into acc (column reduce)
//   row_after<P>(A,rc,acc)                     per-row values that become known after phase P
//   epilogue<V,KEEP>(A,rc,slot,keep,col,span,out)  per-element results of all outputs
//   store<V>(A,rc,col,span,out)                store a slot of outputs
//   row_store(A,row,rc)                        store per-row outputs (one lane per row calls it)
//   NPHASE, MAX_ACC_BYTES
#pragma once

// A module specialised for one shape defines these before this header: they assign the shape's
// constants to the by-value kernel arguments, and the compiler folds them through the kernel.
#ifndef DISC_STATIC_ARGS
#define DISC_STATIC_ARGS(A)
#define DISC_STATIC_PLAN(rp)
#endif

namespace disc {

typedef unsigned char u8;
typedef unsigned short u16;
typedef unsigned int u32;
typedef long long i64;
typedef unsigned long long u64;

#define DISC_DEV __device__ __forceinline__

template <int N>
struct IntC {
  static constexpr int value = N;
};

// ---------------------------------------------------------------------------------------
// Vectors of N storage elements, loaded and stored with ELEMENT alignment only.  gfx950
// runs with unaligned global access enabled, so the compiler still emits one wide access
// (global_load_dwordx4 for 16 bytes) and the hardware serves rows that start at any element.
// This is why no separate "aligned" kernel version is needed for rows whose length is not a
// multiple of the vector width.  The payload is a native vector value (never a byte copy
// into a struct), so it always lives in registers.
// ---------------------------------------------------------------------------------------
template <class T, int N, bool PACKED = (sizeof(T) == 1 && N >= 4)>
struct Vec {
  typedef T vec_t __attribute__((ext_vector_type(N)));
  typedef vec_t unaligned_t __attribute__((aligned(alignof(T))));
  vec_t v;
  DISC_DEV void clear() { v = vec_t(T(0)); }
  DISC_DEV T get(int e) const { return v[e]; }
  DISC_DEV void set(int e, T x) { v[e] = x; }
};
// One-byte elements are kept as whole 32-bit words: a vector of bytes is not a register type, and
// the compiler would carry it around loops one byte per register, packing and unpacking each time.
template <class T, int N>
struct Vec<T, N, true> {
  typedef unsigned vec_t __attribute__((ext_vector_type(N / 4)));
  typedef vec_t unaligned_t __attribute__((aligned(1)));
  vec_t v;
  DISC_DEV void clear() { v = vec_t(0u); }
  DISC_DEV T get(int e) const { return (T)((v[e / 4] >> (8 * (e % 4))) & 0xffu); }
  DISC_DEV void set(int e, T x) {   // the byte must still be zero (clear() first)
    v[e / 4] |= (unsigned)(unsigned char)x << (8 * (e % 4));
  }
};

// The first n elements of a slot belong to the row (n = N everywhere but at the end of a row).
// The per-element test e < n is made where it is used: keeping the 8 or 16 lane masks of every
// slot alive across the phases was measured slower -- they do not fit the scalar registers next
// to the kernel arguments and were spilled to vector-register lanes on every path.
struct Span {
  int n;
  static DISC_DEV Span upto(int n) {
    Span s;
    s.n = n;
    return s;
  }
  DISC_DEV bool full(int N) const { return n >= N; }
  DISC_DEV bool has(int e) const { return e < n; }
  DISC_DEV bool any() const { return n > 0; }
};
// The span of a slot in a launch whose rows are a whole number of slots (row length a multiple of
// the vector width): a slot is either all inside the row or not there at all, which the compiler
// knows -- every ragged-tail path (predicated bodies, piecewise loads and stores, the wave-wide
// "all full?" vote) drops out of the kernel versions built on it.
struct EvenSpan {
  int n;
  static DISC_DEV EvenSpan upto(int n) {
    EvenSpan s;
    s.n = n;
    return s;
  }
  DISC_DEV bool full(int) const { return true; }
  DISC_DEV bool has(int) const { return true; }
  DISC_DEV bool any() const { return n > 0; }
};

// The same of a slot that is not the first of its tensor (compaction tiles): an operand read one
// element earlier has that element too.
struct InnerSpan : EvenSpan {
  static DISC_DEV InnerSpan upto(int n) {
    InnerSpan s;
    s.n = n;
    return s;
  }
};

// Element offset of a slot relative to the base row of the access.  A caller that passes the
// column as `unsigned` promises that lane_base + col, scaled to bytes, fits 32 bits (the
// register-resident row kernels: a wavefront's rows span at most 3 * 1024 slots); the access can
// then use a scalar base register plus a 32-bit lane offset.  Any other column type: 64 bits.
DISC_DEV unsigned off(int lane_base, unsigned col) { return (unsigned)lane_base + col; }
DISC_DEV i64 off(int lane_base, int col) { return (i64)lane_base + col; }
DISC_DEV i64 off(int lane_base, i64 col) { return lane_base + col; }

// A ragged slot (n < N elements) moves as the power-of-two pieces of n's binary expansion: the
// piece of width W covers [(q-1)W, qW) when n / W == q is odd.  Every lane of a launch has the
// same ragged length, so a wavefront issues at most log2(N) narrow accesses per ragged slot.
template <int W, class T, int N, class I>
DISC_DEV void ld_pieces(Vec<T, N>& d, const T* __restrict__ p, I off, int n) {
  if constexpr (W >= 1) {
#pragma unroll
    for (int q = 1; q * W < N; q += 2)
      if (n / W == q) {
        Vec<T, W> piece;
        piece.v = *reinterpret_cast<const typename Vec<T, W>::unaligned_t*>(p + off + (q - 1) * W);
#pragma unroll
        for (int i = 0; i < W; ++i) d.set((q - 1) * W + i, piece.get(i));
      }
    ld_pieces<W / 2>(d, p, off, n);
  }
}
template <int W, class T, int N, class I>
DISC_DEV void st_pieces(T* __restrict__ p, I off, const Vec<T, N>& s, int n) {
  if constexpr (W >= 1) {
#pragma unroll
    for (int q = 1; q * W < N; q += 2)
      if (n / W == q) {
        Vec<T, W> piece;
        piece.clear();
#pragma unroll
        for (int i = 0; i < W; ++i) piece.set(i, s.get((q - 1) * W + i));
        *reinterpret_cast<typename Vec<T, W>::unaligned_t*>(p + off + (q - 1) * W) = piece.v;
      }
    st_pieces<W / 2>(p, off, s, n);
  }
}

// `whole_ok`: all N elements lie inside the tensor even though only part of them belong to this
// row (the rest are the tail of the previous / head of the next row).  Then the wide load is
// still taken and the caller ignores the surplus elements; only a slot that would leave the
// tensor is read element by element.  This keeps ragged rows on the wide-load path.
// address of element `off` of p; a 32-bit unsigned offset is scaled in 32 bits, so that the
// address is base + zero-extended byte offset -- the form that takes a scalar base register
template <class T, class I>
DISC_DEV const T* at(const T* p, I off) {
  if constexpr (__is_same(I, unsigned))
    return reinterpret_cast<const T*>(reinterpret_cast<const char*>(p) + (unsigned)(off * (unsigned)sizeof(T)));
  else
    return p + off;
}
template <class T, class I>
DISC_DEV T* at(T* p, I off) {
  return const_cast<T*>(at(const_cast<const T*>(p), off));
}

// NT: non-temporal access, a compile-time constant of the kernel version (a run-time choice
// between the two accesses is merged into one plain access by the optimiser).  For operands
// and results that are touched exactly once the hint keeps them from displacing each other in the
// L2 and the memory-side cache; the host picks the version per launch (the hint hurts short or
// misaligned rows, whose cache lines are shared by neighbouring rows and so ARE touched twice).
template <bool NT = false, class T, int N, class I, class SP>
DISC_DEV void ld(Vec<T, N>& d, const T* __restrict__ p, I off, SP sp, bool whole_ok = false) {
  if (sp.full(N) || whole_ok) {
    const auto* q = reinterpret_cast<const typename Vec<T, N>::unaligned_t*>(at(p, off));
    if constexpr (NT) d.v = __builtin_nontemporal_load(q);
    else d.v = *q;
  } else {
    d.clear();
    ld_pieces<N / 2>(d, p, off, sp.n);
    // s_waitcnt vmcnt(0): the pieces are complete before the branches rejoin.  Otherwise the
    // compiler has to assume a piece may still be in flight into d's registers and makes the
    // wide load above wait for every earlier load of the wavefront -- on the path where no
    // lane took this branch at all, serialising the loads of full slots.
    __builtin_amdgcn_s_waitcnt(0x0F70);
  }
}

template <bool NT = false, class T, int N, class I, class SP>
DISC_DEV void st(T* __restrict__ p, I off, const Vec<T, N>& s, SP sp) {
  if (sp.full(N)) {
    auto* q = reinterpret_cast<typename Vec<T, N>::unaligned_t*>(at(p, off));
    if constexpr (NT) __builtin_nontemporal_store(s.v, q);
    else *q = s.v;
  } else {
    st_pieces<N / 2>(p, off, s, sp.n);
  }
}

// Slot of a padded operand: elements whose column lies in [wlo, whi) of a row that lies inside the
// operand (row_ok) come from memory, the others are the padding value.  A slot wholly inside
// takes the ordinary wide load; one that straddles an edge of the operand is read element by
// element (two slots per row at most).
template <class T>
DISC_DEV T pad_const(float x) {
  if constexpr (sizeof(T) == 1) return (T)(x != 0.0f);
  else return (T)x;
}
template <class T, int N, class I, class SP>
DISC_DEV void ld_win(Vec<T, N>& d, const T* __restrict__ p, I off, SP sp, i64 col, bool row_ok, i64 wlo, i64 whi, T padv) {
  const i64 lo = wlo - col, hi = whi - col;        // the operand's columns in slot coordinates
  if (row_ok && lo <= 0 && hi >= sp.n) {
    ld(d, p, off, sp);
  } else {
    d.clear();
#pragma unroll
    for (int e = 0; e < N; ++e) {
      T x = padv;
      if (row_ok && sp.has(e) && e >= lo && e < hi) x = at(p, off)[e];
      d.set(e, x);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);
  }
}

// Slot of an operand read one element earlier: d[e] = p[off + e - 1].  The very first slot of the
// tensor (!has_prev) has no element in front of it: its element 0 stays zero (the caller never looks
// at it) and the rest is read one by one.
template <class T, int N, class I, class SP>
DISC_DEV void ld_prev(Vec<T, N>& d, const T* __restrict__ p, I off, SP sp, bool has_prev) {
  if (__is_same(SP, InnerSpan) || has_prev) {
    ld(d, p - 1, off, sp);
  } else {
    d.clear();
#pragma unroll
    for (int e = 1; e < N; ++e)
      if (sp.has(e)) d.set(e, at(p, off)[e - 1]);
    __builtin_amdgcn_s_waitcnt(0x0F70);
  }
}

// The same where the operand itself is in the slot too: d[0] is all that is loaded, and the others are copied from there
// when the slot is used (prev_from; carried along with the slot they would take registers twice).
template <class T, int N, class I, class SP>
DISC_DEV void ld_prev_first(Vec<T, N>& d, const T* __restrict__ p, I off, SP, bool has_prev) {
  d.clear();
  T first = T(0);
  if (__is_same(SP, InnerSpan) || has_prev) first = at(p - 1, off)[0];
  d.set(0, first);
}
template <class T, int N>
DISC_DEV void prev_from(Vec<T, N>& d, const Vec<T, N>& same) {
  const T first = d.get(0);
  d.clear();
  d.set(0, first);
#pragma unroll
  for (int e = 1; e < N; ++e) d.set(e, same.get(e - 1));
}

// storage <-> register conversions (float values live in fp32 registers; one rounding,
// to nearest even, at the store)
DISC_DEV float to_f32(float x) { return x; }
DISC_DEV float to_f32(_Float16 x) { return (float)x; }
DISC_DEV float to_f32(__bf16 x) { return (float)x; }
DISC_DEV float to_f32(int x) { return (float)x; }
DISC_DEV float to_f32(i64 x) { return (float)x; }
DISC_DEV float to_f32(bool x) { return x ? 1.f : 0.f; }
template <class T> DISC_DEV T from_f32(float x);
template <> DISC_DEV float from_f32<float>(float x) { return x; }
template <> DISC_DEV _Float16 from_f32<_Float16>(float x) { return (_Float16)x; }
template <> DISC_DEV __bf16 from_f32<__bf16>(float x) { return (__bf16)x; }

// fp32 results -> storage vector, two elements per conversion where the type has a packed
// convert (v_cvt_pk_bf16_f32 on gfx950 rounds to nearest even and delivers the packed pair)
template <class T, int N>
DISC_DEV void cvt_vec(Vec<T, N>& d, const float (&y)[N]) {
  if constexpr (N % 2 == 0 && sizeof(T) == 2) {
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef T t2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int e = 0; e < N; e += 2) {
      const f2 p = {y[e], y[e + 1]};
      const t2 q = __builtin_convertvector(p, t2);
      d.v[e] = q[0];
      d.v[e + 1] = q[1];
    }
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) d.v[e] = from_f32<T>(y[e]);
  }
}

// Per-element transcendental math on the hardware approximation units (about 1 ulp each):
// the fused kernels have roughly 40 VALU lane-operations per element to spend before they stop
// being HBM-bound, which IEEE-correct expf / division would use up several times over.
DISC_DEV float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
DISC_DEV float fast_rsqrt(float x) { return __builtin_amdgcn_rsqf(x); }
DISC_DEV float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }
DISC_DEV float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
DISC_DEV float fast_exp(float x) { return __builtin_amdgcn_exp2f(x * 1.44269504088896341f); }
DISC_DEV float fast_log(float x) { return __builtin_amdgcn_logf(x) * 0.693147180559945309f; }
DISC_DEV float fast_sigmoid(float x) { return fast_rcp(1.0f + fast_exp(-x)); }
// a sum whose operands are rounded first, whatever they are (never part of a fused multiply-add)
DISC_DEV float add_apart(float x, float y) {
#pragma clang fp contract(off)
  return x + y;
}
// tanh(x) = 1 - 2 / (exp(2x) + 1): exact limits at +-inf, absolute error ~1e-7 everywhere
DISC_DEV float fast_tanh(float x) { return 1.0f - 2.0f * fast_rcp(fast_exp(2.0f * x) + 1.0f); }

// ---------------------------------------------------------------------------------------
// Division by a runtime extent with constants the host precomputes from the shape
// (round-up multiply-shift method of Granlund & Montgomery): for 0 <= n < 2^31,
//   n / d == (umulhi(n, m) + n) >> s   with s = ceil(log2 d), m = floor(2^32 (2^s - d) / d) + 1.
// ---------------------------------------------------------------------------------------
struct FastDiv {
  u32 d, m, s, pad;
};
DISC_DEV u32 fdiv(u32 n, const FastDiv& f) { return (__umulhi(n, f.m) + n) >> f.s; }

// ---------------------------------------------------------------------------------------
// Cross-lane exchange inside a 64-wide wavefront, all on the VALU (no LDS crossbar):
// lane_xchg<S>(v) returns v of a partner lane such that combining a value with its partner
// for S = 1, 2, 4, 8, 16, 32 in turn leaves every lane of each aligned 2S-lane group with
// the combination of the whole group.  S = 1, 2: DPP quad permutes; S = 4, 8: DPP mirror
// within 8 / 16 lanes (after the quad steps every quad is uniform, so mirroring pairs the
// right quads); S = 16, 32: gfx950's permlane16 / permlane32 swaps, called with both operands
// equal, which hand back the partner row / half as the second result.
// ---------------------------------------------------------------------------------------
template <int S>
DISC_DEV u32 lane_xchg_u32(u32 v) {
  if constexpr (S == 1) return (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);        // quad_perm [1,0,3,2]
  else if constexpr (S == 2) return (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true);   // quad_perm [2,3,0,1]
  else if constexpr (S == 4) return (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true);  // row_half_mirror
  else if constexpr (S == 8) return (u32)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true);  // row_mirror
  else if constexpr (S == 16) {
    auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const bool odd_row = (threadIdx.x >> 4) & 1;
    return odd_row ? r[0] : r[1];
  } else {
    auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    const bool upper = (threadIdx.x >> 5) & 1;
    return upper ? r[0] : r[1];
  }
}
template <int S> DISC_DEV float lane_xchg(float v) { return __builtin_bit_cast(float, lane_xchg_u32<S>(__builtin_bit_cast(u32, v))); }
template <int S> DISC_DEV int lane_xchg(int v) { return (int)lane_xchg_u32<S>((u32)v); }
template <int S> DISC_DEV i64 lane_xchg(i64 v) {
  const u32 lo = lane_xchg_u32<S>((u32)(u64)v), hi = lane_xchg_u32<S>((u32)((u64)v >> 32));
  return (i64)(((u64)hi << 32) | lo);
}
template <int S> DISC_DEV double lane_xchg(double v) { return __builtin_bit_cast(double, lane_xchg<S>(__builtin_bit_cast(i64, v))); }

// true when the predicate holds in every active lane of the wavefront (scalar result)
DISC_DEV bool wave_all(bool p) { return __builtin_amdgcn_ballot_w64(!p) == 0; }

// all-reduce of an accumulator over aligned groups of G lanes (G a power of two, <= 64)
template <class Pat, int P, int S>
DISC_DEV void group_step(typename Pat::template Acc<P>& acc) {
  typename Pat::template Acc<P> o = acc;
  Pat::template acc_xchg<P, S>(o);
  Pat::template acc_merge<P>(acc, o);
}
// nested on purpose: one scalar test per level, nothing re-derived after the branches rejoin.
// The empty asm makes G opaque at each call: the tests are then scalar compares at the point of
// use; otherwise the compiler evaluates all six once per kernel and keeps them as lane masks in
// twelve scalar registers across the row loop, which does not have them to spare.
template <class Pat, int P>
DISC_DEV void group_allreduce(typename Pat::template Acc<P>& acc, int G) {
  asm volatile("" : "+s"(G));
  if (G > 1) {
    group_step<Pat, P, 1>(acc);
    if (G > 2) {
      group_step<Pat, P, 2>(acc);
      if (G > 4) {
        group_step<Pat, P, 4>(acc);
        if (G > 8) {
          group_step<Pat, P, 8>(acc);
          if (G > 16) {
            group_step<Pat, P, 16>(acc);
            if (G > 32) group_step<Pat, P, 32>(acc);
          }
        }
      }
    }
  }
}

// =======================================================================================
// Loop fusion (kLoop).  The iteration space is [rows, inner]; it is cut into slots of V
// consecutive elements of one row.  Consecutive lanes take consecutive slots, so every wave
// reads and writes one contiguous stretch of memory whatever `inner` is; a block walks the
// slot list with a grid stride, U slots in flight per lane to keep enough bytes in flight
// for HBM.  (row, col) of a slot come from one multiply-shift division per slot.
// =======================================================================================
// NT: bit 0 = non-temporal loads of the full-size operands, bit 1 = non-temporal stores
template <class Pat, int V, int U, bool I64, int NT = 0>
DISC_DEV void kloop_body(const typename Pat::Args& A) {
  if constexpr (!I64) {
    const u32 nslots = (u32)A.nslots;
    const u32 stride = gridDim.x * blockDim.x;
    const u32 inner = (u32)A.inner;
    for (u32 s0 = blockIdx.x * blockDim.x + threadIdx.x; s0 < nslots; s0 += stride * U) {
      typename Pat::template Slot<V> slot[U];
      typename Pat::RowCtx rc[U];
      int col[U], nv[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const u32 s = s0 + u * stride;
        nv[u] = 0;
        if (s < nslots) {
          const u32 row = fdiv(s, A.spr_div);
          col[u] = (int)((s - row * A.spr_div.d) * V);
          nv[u] = min((int)V, (int)(inner - (u32)col[u]));
          Pat::row_begin(A, (i64)row, rc[u]);
          Pat::template load<V, NT>(A, rc[u], col[u], Span::upto(nv[u]), slot[u]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (nv[u] > 0) {
          typename Pat::template OutSlot<V> o;
          typename Pat::template Keep<V> kp;
          Pat::template epilogue<V, false>(A, rc[u], slot[u], kp, col[u], Span::upto(nv[u]), o);
          Pat::template store<V, NT>(A, rc[u], col[u], Span::upto(nv[u]), o);
        }
      }
    }
  } else {
    const i64 nslots = A.nslots;
    const i64 stride = (i64)gridDim.x * blockDim.x;
    const i64 spr = A.spr;
    for (i64 s = (i64)blockIdx.x * blockDim.x + threadIdx.x; s < nslots; s += stride) {
      const i64 row = s / spr;
      const i64 col = (s - row * spr) * V;
      const i64 rem = A.inner - col;
      const int nv = rem < (i64)V ? (int)rem : V;
      typename Pat::template Slot<V> slot;
      typename Pat::RowCtx rc;
      Pat::row_begin(A, row, rc);
      Pat::template load<V, NT>(A, rc, col, Span::upto(nv), slot);
      typename Pat::template OutSlot<V> o;
      typename Pat::template Keep<V> kp;
      Pat::template epilogue<V, false>(A, rc, slot, kp, col, Span::upto(nv), o);
      Pat::template store<V, NT>(A, rc, col, Span::upto(nv), o);
    }
  }
}

// =======================================================================================
// Input fusion with a row reduction as root (kInput, reduce over the innermost axis).
//
// Register-resident version: a row is owned by a group of G lanes chosen by the host per shape:
// a power of two 1..32 = several rows per wavefront for short rows, 64 = a wavefront per row,
// a multiple of 64 up to 1024 = G/64 wavefronts per row (the host picks block sizes whose
// wavefront count is a multiple of four, so the four SIMDs of a CU get equal shares).  Lane l of the group holds
// slots l, l+G, l+2G, ... (NV of them, V elements each), loaded ONCE; every reduction phase
// and the epilogue run out of registers, so the row makes exactly one trip from HBM and one
// back.  Within a wavefront partial results are combined with xor-shuffles; across the
// wavefronts of a row through a double-buffered LDS exchange (one barrier per phase).
// =======================================================================================
// The span of a slot in the kernel versions that take the ragged ends of a row as single elements:
// whole like EvenSpan, but the slot may start at ANY column (the vector slots of a row may be
// shifted to 16-byte boundaries of memory, and single elements sit anywhere).
struct TailSpan : EvenSpan {
  static DISC_DEV TailSpan upto(int n) {
    TailSpan s;
    s.n = n;
    return s;
  }
};
template <bool EVEN, bool TAIL = false> struct SpanSel { typedef Span type; };
template <> struct SpanSel<true, false> { typedef EvenSpan type; };
template <> struct SpanSel<true, true> { typedef TailSpan type; };
struct RowPlan {
  int G;        // lanes per row: a power of two <= 64, or a multiple of 64 (whole wavefronts)
  int log2G;    // meaningful for G <= 64
  int nv;       // slots per lane actually needed at this shape (<= NV of the instantiation)
  int flags;    // bit 0: the launched kernel is the version that stages row-vector operands in LDS
                // bit 1: the slot grid is not turned from row to row
                // bit 2: (_t versions) vector slots on boundaries of the tensor, every (flags >> 8) elements
                // bit 3: (_t versions) non-temporal accesses of the vector slots
  int rpb;      // rows per block = blockDim.x / G
};

// Row-vector operands (bias, gamma, beta, ...) are the same for every row a block processes:
// when the host grants the LDS, each block copies them once into dynamic LDS, padded with V
// zero elements, and every slot reads them from there with one aligned LDS vector read --
// no per-slot trip through the vector memory pipeline and no ragged-tail path for them.
extern __shared__ __attribute__((aligned(16))) char disc_stage_lds[];

// Slots that start at a boundary of the tensor and not of the row (TAIL versions, below) start at a column
// head + k * V; every lane group of the block has a head of its own, and keeps it.  An LDS access
// of 8 or 16 bytes off its own alignment is served one lane a cycle (64 cycles, 6 aligned), and as single dwords
// the slots of a wavefront's lanes meet on the same banks (40), so the copies are shifted instead: element i of a row
// vector lies at i + shift, which makes every slot start on 16 bytes (E elements; less where V elements are less).
// A copy for every lane group, or for every shift where these are fewer (which of them pay is the host's rule).  Mixed
// chain of bf16, us, single dwords / shifted copies: 46773 x 5739 253.5 / 243.5, 4000 x 8191 35.4 / 32.2.
struct StagePlan {
  int groups;   // lane groups of the block, 0: unshifted slots
  i64 row0;     // row of the first one
  i64 rows;
  int inner, al;
  DISC_DEV int head(int grp) const {
    const i64 r = row0 + grp < rows ? row0 + grp : rows - 1;
    const int e0 = ((int)(r & (al - 1)) * (inner & (al - 1))) & (al - 1);   // (row * inner) mod al
    return (al - e0) & (al - 1);
  }
  DISC_DEV int copies(int E) const { return groups == 0 ? 1 : groups < E ? groups : E; }
  DISC_DEV int shift(int E, int copy) const { return groups == 0 ? 0 : groups <= E ? -head(copy) & (E - 1) : copy; }
  DISC_DEV int copy_of(int E, int grp) const { return groups == 0 ? 0 : groups <= E ? grp : -head(grp) & (E - 1); }
};
// elements of a slot's access that have to start on its alignment
template <int V, class T>
constexpr int stage_align() { return V * (int)sizeof(T) < 16 ? V : 16 / (int)sizeof(T); }
// cooperative copy of n elements (+ PAD zero elements) into LDS: 16-byte pieces, then the tail; or several shifted ones
// of `bytes` each, in 16-byte pieces that lie on 16 bytes there, four of a lane's loads in flight at once
template <int PAD, class T>
DISC_DEV void stage_copy(T* dst, const T* __restrict__ src, int n, int bytes, const StagePlan& sp, int tid, int nthreads) {
  constexpr int N = 16 / (int)sizeof(T), E = stage_align<PAD, T>();
  if (sp.groups == 0) {
    const int nvec = n / N;
    for (int i = tid; i < nvec; i += nthreads)
      reinterpret_cast<typename Vec<T, N>::vec_t*>(dst)[i] =
          *reinterpret_cast<const typename Vec<T, N>::unaligned_t*>(src + (i64)i * N);
    for (int i = nvec * N + tid; i < n + PAD; i += nthreads) dst[i] = i < n ? src[i] : T(0);
    return;
  }
  const int copies = sp.copies(E), log2 = 31 - __builtin_clz(copies);
  const int pieces = (n + PAD + N - 1) / N * copies;
  for (int w0 = tid; w0 < pieces; w0 += 4 * nthreads) {
    Vec<T, N> x[4];
    int from[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int w = w0 + u * nthreads;
      from[u] = (w >> log2) * N - sp.shift(E, w & (copies - 1));
      if (w < pieces && from[u] >= 0 && from[u] + N <= n)
        x[u].v = *reinterpret_cast<const typename Vec<T, N>::unaligned_t*>(src + from[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int w = w0 + u * nthreads;
      if (w < pieces) {
        if (from[u] < 0 || from[u] + N > n) {      // the ends of a copy
          x[u].clear();
#pragma unroll
          for (int e = 0; e < N; ++e)
            if (from[u] + e >= 0 && from[u] + e < n) x[u].set(e, src[from[u] + e]);
        }
        *reinterpret_cast<typename Vec<T, N>::vec_t*>(reinterpret_cast<char*>(dst) + (w & (copies - 1)) * bytes + (w >> log2) * 16) = x[u].v;
      }
    }
  }
}
// where a lane group's copy of a row vector begins: its byte `at`, copies of `bytes`
template <int V, class T>
DISC_DEV int stage_place(int at, int bytes, const StagePlan& sp, int grp) {
  constexpr int E = stage_align<V, T>();
  if (sp.groups == 0) return at;
  return at + sp.copy_of(E, grp) * bytes + (-sp.head(grp) & (E - 1)) * (int)sizeof(T);
}

// slot at column `col` of the copy that begins at byte_off
template <class T, int N>
DISC_DEV void ld_lds(Vec<T, N>& d, const char* base, int byte_off, int col) {
  typedef typename Vec<T, N>::vec_t aligned_t __attribute__((aligned(sizeof(T) * N < 16 ? sizeof(T) * N : 16)));
  d.v = *reinterpret_cast<const aligned_t*>(base + byte_off + col * (int)sizeof(T));
}

// Sums over the rows carried along by a row reduce (Pat::NCOLSUM of them): every lane adds the
// values of its own columns, row after row, into fp32 registers; at the end of the kernel each
// wavefront (rows of at most a wavefront) or lane group (longer rows) writes one row of partial
// sums per summed output into the workspace, plane q at ws + q * n_partial_rows * inner, and a
// second launch adds the partial rows up in a fixed order.
DISC_DEV float lane_xor_f32(float v, int s) {
  const int lane = (int)threadIdx.x & 63;
  return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute((lane ^ s) << 2, __builtin_bit_cast(int, v)));
}
// x[i] summed over the lanes of a wavefront whose numbers agree mod G, in every lane.  On the vector ALU, one step for
// all values before the next one (rotations within 16 lanes, which a sum of period 2 S completes to one of period S; then
// the halves that permlane swaps hand back).  With a lane permutation through the LDS crossbar per value and step, each
// waiting for the one before, it was 22.4 us for LayerNorm backward of
// 10000 x 300, 19.6 now, and 18.3 for 3000 x 130, 12.9 now.
template <int N>
DISC_DEV void lanes_sum(float (&x)[N], int G) {
  auto rotated = [](float v, auto s) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), 0x120 + s.value, 0xf, 0xf, true));
  };
  asm volatile("" : "+s"(G));
  if (G <= 8) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += rotated(x[i], IntC<8>{});
    if (G <= 4) {
#pragma unroll
      for (int i = 0; i < N; ++i) x[i] += rotated(x[i], IntC<4>{});
      if (G <= 2) {
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] += rotated(x[i], IntC<2>{});
        if (G <= 1) {
#pragma unroll
          for (int i = 0; i < N; ++i) x[i] += rotated(x[i], IntC<1>{});
        }
      }
    }
  }
  if (G <= 16) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const u32 v = __builtin_bit_cast(u32, x[i]);
      auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
      x[i] = __builtin_bit_cast(float, (u32)r[0]) + __builtin_bit_cast(float, (u32)r[1]);
    }
  }
  if (G <= 32) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const u32 v = __builtin_bit_cast(u32, x[i]);
      auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
      x[i] = __builtin_bit_cast(float, (u32)r[0]) + __builtin_bit_cast(float, (u32)r[1]);
    }
  }
}

// The end of a row behind its last whole slot, taken as slots of ONE element by the first lanes of
// the row (TAIL versions of the row kernels): the lane's element, what it keeps between the
// phases, and its column (-1: this lane has none).
template <class Pat>
struct TailSlot {
  typename Pat::template Slot<1> s;
  typename Pat::template Keep<1> k;
  int col;
};
struct NoTail {
  int col;
};
template <class Pat, bool TAIL>
struct TailSel {
  typedef NoTail type;
};
template <class Pat>
struct TailSel<Pat, true> {
  typedef TailSlot<Pat> type;
};

// `after_first` runs once, after the slots have been folded into the accumulator of phase 0 and
// before the lanes combine: the place where the caller issues the loads of the next row.
template <class Pat, int P, int V, int NV, class Hook, class SP, class TS>
DISC_DEV void row_phases(const typename Pat::Args& A, const RowPlan& rp, typename Pat::RowCtx& rc,
                         const typename Pat::template Slot<V> (&slot)[NV],
                         typename Pat::template Keep<V> (&keep)[NV], const SP (&span)[NV],
                         int col0, char* lds, int& parity, Hook& after_first, TS& ts) {
  if constexpr (P < Pat::NPHASE) {
    typename Pat::template Acc<P> acc;
    Pat::template acc_init<P>(acc);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int col = col0 + j * rp.G * V;
      if (span[j].any()) Pat::template phase<P, V, true>(A, acc, slot[j], keep[j], span[j], col, rc);
    }
    if constexpr (!__is_same(TS, NoTail)) {
      if (ts.col >= 0) Pat::template phase<P, 1, true>(A, acc, ts.s, ts.k, TailSpan::upto(1), ts.col, rc);
    }
    if constexpr (P == 0) after_first();
    // lanes of one wavefront
    group_allreduce<Pat, P>(acc, rp.G < 64 ? rp.G : 64);
    // wavefronts of one row
    if (rp.G > 64) {
      typedef typename Pat::template Acc<P> AccT;
      AccT* ex = reinterpret_cast<AccT*>(lds + parity * 16 * Pat::MAX_ACC_BYTES);
      parity ^= 1;
      const int wave = threadIdx.x >> 6;
      if ((threadIdx.x & 63) == 0) ex[wave] = acc;
      __syncthreads();
      const int wpr = rp.G >> 6;               // wavefronts per row
      const int w0 = (wave / wpr) * wpr;       // first wavefront of this row
      if ((wpr & (wpr - 1)) == 0) {
        // every lane fetches one partial (lane i the one of wavefront i mod wpr) and the lanes
        // combine them with the butterfly: one LDS read instead of a chain of wpr dependent ones
        acc = ex[w0 + ((int)threadIdx.x & (wpr - 1))];
        group_allreduce<Pat, P>(acc, wpr);
      } else {
        acc = ex[w0];
        for (int w = 1; w < wpr; ++w) {
          AccT o = ex[w0 + w];
          Pat::template acc_merge<P>(acc, o);
        }
      }
    }
    Pat::template row_after<P>(A, rc, acc);
    row_phases<Pat, P + 1, V, NV>(A, rp, rc, slot, keep, span, col0, lds, parity, after_first, ts);
  }
}

// NT: bit 0 = non-temporal loads of the full-size operands, bit 1 = non-temporal stores
// EVEN: every vector slot is whole -- the host promises that the row length is a multiple of V, or
// TAIL: (with EVEN) the elements behind the last whole slot of a row, inner % V of them, are taken
//       one per lane by the lanes that hold the row's first columns, as slots of ONE element that
//       go through the same phases, the same accumulators and the same epilogue.  Against a
//       ragged last slot this costs one element's work in one wavefront of the row instead of a
//       predicated pass over a whole slot in every lane of that wavefront, no access moves in
//       pieces, and the row needs capacity for its whole slots only.  Needs G >= V lanes per row.
template <class Pat, int V, int NV, bool PIPE = true, int NT = 0, bool EVEN = false, bool TAIL = false>
DISC_DEV void row_reg_body(const typename Pat::Args& A, const RowPlan& rp) {
  static_assert(!TAIL || (EVEN && Pat::NCOLSUM == 0), "single-element tails: whole vector slots, no sums over the rows");
  typedef typename SpanSel<EVEN, TAIL>::type SP;
  __shared__ __attribute__((aligned(16))) char lds[2 * 16 * Pat::MAX_ACC_BYTES];
  // G <= 64: a power of two; G > 64: a multiple of 64
  const int grp = rp.G <= 64 ? (int)threadIdx.x >> rp.log2G : ((int)threadIdx.x >> 6) / (rp.G >> 6);
  const int lane = (int)threadIdx.x - grp * rp.G;
  const int rpb = rp.rpb;
  const i64 rows = A.rows;
  const int inner = (int)A.inner;
  int parity = 0;
  const char* staged = nullptr;
  typename Pat::Staged placed{};
  if constexpr (Pat::STAGED) {
    const StagePlan sp{TAIL && (rp.flags & 4) ? rpb : 0, (i64)blockIdx.x * rpb, rows, inner, TAIL ? rp.flags >> 8 : 0};
    Pat::stage(A, disc_stage_lds, threadIdx.x, blockDim.x, sp);
    Pat::stage_at(A, sp, grp, placed);
    __syncthreads();
    staged = disc_stage_lds;
  }
  // A group past the last row (last block, several rows per block) works on the last row again
  // and stores nothing, so that no branch depends on it.
  //
  // Rows of several wavefronts: the wavefront that gets the ragged extra slots of a row does up
  // to twice the work of the others, and it would always be the first one -- on the same SIMD
  // of the CU for every row.  The slot grid is therefore turned by one wavefront from row to
  // row (lane l takes the columns of lane l + rot), which spreads the extra work evenly.
  // (a lane that sums its columns over the rows keeps its columns: no turning then)
  const int wpr = (Pat::NCOLSUM == 0 && rp.G > 64 && !(rp.flags & 2)) ? rp.G >> 6 : 1;   // flags bit 1: grid not turned (experiments)
  int rot = wpr > 1 ? (int)(blockIdx.x % (unsigned)wpr) * 64 : 0;
  // Row bookkeeping in scalar registers: rw = row of the first lane group of this wavefront in
  // the current row group, sbw = its element offset; both advance by a constant per iteration
  // (no 64-bit products in the loop).  A lane's row is rw + dgrp.
  const int grp_w = __builtin_amdgcn_readfirstlane(grp);
  const int dgrp = grp - grp_w;
  const i64 rstep = (i64)gridDim.x * rpb;
  const i64 sbstep = rstep * A.inner;
  i64 rw = (i64)blockIdx.x * rpb + grp_w;
  i64 sbw = rw * A.inner;
  // TAIL versions, flags bit 2: the vector slots of a row are shifted to the boundaries of
  // al = flags >> 8 elements (a power of two, V at least) of the TENSOR (row * inner + column a
  // multiple of al), so that every wide access of a full-size operand whose base is aligned is aligned
  // itself, whatever the row length: the `head` elements in front of the first boundary are single
  // elements like those behind the last whole slot, one per lane (head + V - 1 lanes at most).
  // The host launches a grid that puts rows of equal alignment on a lane group (the distance
  // between its rows times the row length is a multiple of al), so `head` is worked out once.  It is
  // an alignment matter only: any value 0 .. al-1 addresses the row correctly.
  int head = 0;
  if constexpr (TAIL) {
    if (rp.flags & 4) head = StagePlan{rpb, (i64)blockIdx.x * rpb, rows, inner, rp.flags >> 8}.head(grp);
  }
  int col0 = lane * V;
  int nvalid[NV];
  int tcol = -1;                        // column of this lane's single element (TAIL versions), -1: none
  auto place = [&](int r, int head, int& c0, int (&n)[NV], int& tc) {
    int l = lane + r;
    if (l >= rp.G) l -= rp.G;
    if constexpr (TAIL) {
      // [head single elements | whole slots | single elements behind them]
      const int whole = (inner - head) / V;
      const int behind = head + whole * V;         // first column behind the whole slots
      c0 = head + l * V;
#pragma unroll
      for (int j = 0; j < NV; ++j) n[j] = (j < rp.nv && l + j * rp.G < whole) ? V : 0;
      tc = l < head ? (l < inner ? l : -1) : (behind + (l - head) < inner ? behind + (l - head) : -1);
    } else {
      c0 = l * V;
      tc = -1;
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        const int col = c0 + j * rp.G * V;
        const int hi = inner - col > V ? V : inner - col;
        n[j] = (j < rp.nv && hi > 0) ? hi : 0;
      }
    }
  };
  place(rot, head, col0, nvalid, tcol);
  // Where a row has several wavefronts the head is the same in all lanes: a scalar where copies take registers too (mixed chain,
  // 86369 x 777: 71.8 -> 68.2 us), but not without them: fp32 softmax over 8207 x 8177 takes 107 us with a scalar and 91.9 without.
  int head_w = head;
  if constexpr (Pat::STAGED) head_w = __builtin_amdgcn_readfirstlane(head);
  // Software pipeline over the rows of a block: the loads of the next row are issued as soon as
  // the first reduction phase has consumed the current row's slots (every load issued so far
  // has landed by then, so no wait in the rest of the iteration touches the new loads); they
  // complete behind the lane reductions, the later phases, the epilogue and the stores.
  // (Where the row vectors are is set here, for this row and the next one alike, and not where a row is loaded: merged
  // with a context that was not filled in, the pointer is no longer known to be one to LDS, and every read through it
  // is a flat load, which waits for the row loads in flight too.  us, flat / LDS reads: LayerNorm of fp32 rows with one
  // vector 21592 x 777 51.1 / 37.4, bf16 43184 x 777 49.2 / 41.2.)
  typename Pat::RowCtx rc{};
  rc.sl = staged;
  rc.so = placed;
  typename Pat::template Slot<V> slot[NV];
  typedef typename TailSel<Pat, TAIL>::type TS;
  TS ts, tsn;
  typename Pat::template ColAcc<V> cacc[NV]{};
  // reductions of per-row values over the rows: every lane of a lane group keeps the running values
  // of the group's rows
  float racc[Pat::NROWRED > 0 ? Pat::NROWRED : 1];
  if constexpr (Pat::NROWRED > 0) {
#pragma unroll
    for (int q = 0; q < Pat::NROWRED; ++q) racc[q] = Pat::rr_identity(q);
  }
  // rows past the end (last row group only) are replaced by the last row; their lanes compute
  // along and store nothing
  auto begin_row = [&](i64 rwv, i64 sbv, typename Pat::RowCtx& c) {
    if (rwv + (rpb - grp_w) <= rows) {
      Pat::row_begin3(A, rwv, dgrp, sbv, c);
    } else {
      const i64 last = rows - 1;
      const i64 b = rwv < last ? rwv : last;
      const i64 r = rwv + dgrp < last ? rwv + dgrp : last;
      Pat::row_begin3(A, b, (int)(r - b), b * A.inner, c);
    }
  };
  auto load_row = [&]() {
    begin_row(rw, sbw, rc);
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (nvalid[j] > 0) Pat::template load<V, NT>(A, rc, (unsigned)(col0 + j * rp.G * V), SP::upto(nvalid[j]), slot[j]);
    if constexpr (TAIL) {
      ts.col = tcol;
      if (tcol >= 0) Pat::template load<1, 0>(A, rc, (unsigned)tcol, TailSpan::upto(1), ts.s);
    }
  };
  // the row group of the block starts at row rw - grp_w; the block is done when that is past the end
  if (PIPE && rw - grp_w < rows) load_row();
  while (rw - grp_w < rows) {
    if constexpr (!PIPE) load_row();
    SP span[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) span[j] = SP::upto(nvalid[j]);
    const i64 row = rw + dgrp;
    const bool active = row < rows;
    typename Pat::RowCtx rcn{};
    rcn.sl = staged;
    rcn.so = placed;
    typename Pat::template Slot<V> nxt[NV];
    int col0n = col0, tcoln = tcol;
    int nvalidn[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) nvalidn[j] = nvalid[j];
    auto prefetch = [&]() {
      if (PIPE && rw + rstep - grp_w < rows) {
        if (wpr > 1) {
          rot = rot + 64 < rp.G ? rot + 64 : 0;
          place(rot, head_w, col0n, nvalidn, tcoln);
        }
        begin_row(rw + rstep, sbw + sbstep, rcn);
#pragma unroll
        for (int j = 0; j < NV; ++j)
          if (nvalidn[j] > 0) {
            SP sn;              // the loads look at the element count only
            sn.n = nvalidn[j];
            Pat::template load<V, NT>(A, rcn, (unsigned)(col0n + j * rp.G * V), sn, nxt[j]);
          }
        if constexpr (TAIL) {
          tsn.col = tcoln;
          if (tcoln >= 0) Pat::template load<1, 0>(A, rcn, (unsigned)tcoln, TailSpan::upto(1), tsn.s);
        }
      }
      // keep the loads here: without a fence the compiler is free to sink them below the
      // stores of this row (to save registers), which undoes the pipeline
      asm volatile("" ::: "memory");
    };
    typename Pat::template Keep<V> keep[NV];
    row_phases<Pat, 0, V, NV>(A, rp, rc, slot, keep, span, col0, lds, parity, prefetch, ts);
    if constexpr (Pat::NPHASE == 0) prefetch();   // (no reduction phase to hide the next row's loads behind)
    if constexpr (Pat::NROWRED > 0) {
      if (active) Pat::row_reds(A, rc, racc);
    }
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      if (span[j].any()) {
        const int col = col0 + j * rp.G * V;
        typename Pat::template OutSlot<V> o;
        Pat::template epilogue<V, true>(A, rc, slot[j], keep[j], col, span[j], o);
        // Loads and stores share one in-order counter, and with both kinds in flight the only
        // wait the compiler can express is "all of them".  Waiting for the next row's loads HERE,
        // before the first store of this row (they were issued a reduction phase ago and have
        // landed), means the first use of those loads in the next iteration needs no wait at all
        // -- otherwise that wait sits right behind these stores and exposes their full latency
        // in every iteration.  The stores then have a whole iteration to drain.
        if (PIPE && j == 0) __builtin_amdgcn_s_waitcnt(0x0F70);
        if (active) Pat::template store<V, NT>(A, rc, (unsigned)col, span[j], o);
        if constexpr (Pat::NCOLSUM > 0) {
          if (active) Pat::template col_sums<V, true>(A, rc, slot[j], keep[j], col, span[j], cacc[j]);
        }
      }
    }
    if constexpr (TAIL) {
      if (ts.col >= 0) {
        typename Pat::template OutSlot<1> o;
        Pat::template epilogue<1, true>(A, rc, ts.s, ts.k, ts.col, TailSpan::upto(1), o);
        if (active) Pat::template store<1, 0>(A, rc, (unsigned)ts.col, TailSpan::upto(1), o);
      }
    }
    if (active && lane == 0) Pat::row_store(A, row, rc);
    rw += rstep;
    sbw += sbstep;
    if constexpr (PIPE) {
      rc = rcn;
#pragma unroll
      for (int j = 0; j < NV; ++j) slot[j] = nxt[j];
      if constexpr (TAIL) ts = tsn;
      if (wpr > 1) {
        col0 = col0n;
        tcol = tcoln;
#pragma unroll
        for (int j = 0; j < NV; ++j) nvalid[j] = nvalidn[j];
      }
    } else if (wpr > 1) {
      rot = rot + 64 < rp.G ? rot + 64 : 0;
      place(rot, head_w, col0, nvalid, tcol);
    }
  }
  if constexpr (Pat::NCOLSUM > 0) {
    // lane groups of one wavefront hold the same columns: add them up across the groups
    if (rp.G < 64) {
#pragma unroll
      for (int j = 0; j < NV; ++j)
#pragma unroll
        for (int q = 0; q < Pat::NCOLSUM; ++q) {
          float x[V];
#pragma unroll
          for (int e = 0; e < V; ++e) x[e] = cacc[j].c[q][e];
          lanes_sum(x, rp.G);
#pragma unroll
          for (int e = 0; e < V; ++e) cacc[j].c[q][e] = x[e];
        }
    }
    // lane sets of the block that hold the same columns (the wavefronts of short rows, the lane
    // groups of rows of two wavefronts): in blocks of 256 threads they meet in LDS, one slot of
    // one sum at a time, so that a block writes a single row of partial sums
    const int period = rp.G > 64 ? rp.G : 64;
    const int copies = (int)blockDim.x / period;
    const int copy = (int)threadIdx.x / period;
    const bool merge = copies > 1 && blockDim.x <= 256;
    if (merge) {
      __shared__ typename Vec<float, V>::vec_t cbuf[2][256];      // (in turn: one barrier for each)
#pragma unroll
      for (int j = 0; j < NV; ++j)
#pragma unroll
        for (int q = 0; q < Pat::NCOLSUM; ++q) {
          auto& buf = cbuf[(j * Pat::NCOLSUM + q) & 1];
          if (copy > 0) buf[threadIdx.x] = cacc[j].c[q];
          __syncthreads();
          if (copy == 0)
            for (int k = 1; k < copies; ++k) cacc[j].c[q] += buf[(int)threadIdx.x + k * period];
        }
    }
    const int ppb = merge ? 1 : copies;                                 // rows of partial sums per block
    const bool writer = (merge ? copy == 0 : true) && (rp.G >= 64 || ((int)threadIdx.x & 63) < rp.G);
    float* ws = reinterpret_cast<float*>(A.ws0);
    const i64 prow = (i64)blockIdx.x * ppb + (merge ? 0 : copy);
    if (writer) {
#pragma unroll
      for (int j = 0; j < NV; ++j)
        if (nvalid[j] > 0) {
#pragma unroll
          for (int q = 0; q < Pat::NCOLSUM; ++q) {
            Vec<float, V> t;
            t.v = cacc[j].c[q];
            st(ws + ((i64)q * A.aux0 + prow) * A.inner, (i64)(col0 + j * rp.G * V), t, SP::upto(nvalid[j]));
          }
        }
    }
  }
  if constexpr (Pat::NROWRED > 0) {
    // The lanes of a lane group hold the same values, the groups of a wavefront different rows:
    // combine across the groups, then across the wavefronts of the block through LDS (the
    // wavefronts of one lane group of a long row hold the same rows: one of them counts), and
    // write one partial result per block and reduction: ws1[q * blocks + block].
    if (rp.G < 64) {
#pragma unroll
      for (int q = 0; q < Pat::NROWRED; ++q)
        for (int sft = rp.G; sft < 64; sft <<= 1) racc[q] = Pat::rr_merge(q, racc[q], lane_xor_f32(racc[q], sft));
    }
    __shared__ float rbuf[16][Pat::NROWRED];
    const int wave = (int)threadIdx.x >> 6, nw = (int)blockDim.x >> 6;
    const int wpg = rp.G > 64 ? rp.G >> 6 : 1;
    if (((int)threadIdx.x & 63) == 0) {
#pragma unroll
      for (int q = 0; q < Pat::NROWRED; ++q) rbuf[wave][q] = racc[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      float* ws = reinterpret_cast<float*>(A.ws1);
#pragma unroll
      for (int q = 0; q < Pat::NROWRED; ++q) {
        float t = rbuf[0][q];
        for (int w = wpg; w < nw; w += wpg) t = Pat::rr_merge(q, t, rbuf[w][q]);
        ws[(i64)q * A.aux1 + blockIdx.x] = t;
      }
    }
  }
}

// _t versions: one entry point, both kinds of access (behind a branch inside the body the compiler would
// merge them into one plain access).
template <class Pat, int V, int NV, bool PIPE>
DISC_DEV void row_tail_body(const typename Pat::Args& A, const RowPlan& rp) {
  if (rp.flags & 8) row_reg_body<Pat, V, NV, PIPE, 3, true, true>(A, rp);
  else row_reg_body<Pat, V, NV, PIPE, 0, true, true>(A, rp);
}

// Streaming version for rows that do not fit the register-resident versions: one block per row.  The
// first NR slots of every lane stay in registers, as loaded (no values carried between the phases, no
// second register set for the next row: with blocks of 1024 threads two of them can share a CU, and
// one loads while the other computes); what lies behind them is read again, from L2 / Infinity Cache
// when it fits, once per reduction phase and once for the epilogue.  The elements behind the last
// whole slot of a row go one each to the first lanes, as slots of one element.  Any row length below
// 2^31 works.
//
// as_loaded: a slot's registers with their contents unknown to the compiler, in place (a copy would cost a move
// per register and phase).  It would otherwise convert a slot to fp32 once and keep that, twice the
// registers, through all phases.  Operand by operand: a slot as a whole has words that are only padding, and
// each of those would take a register too (log-sum-exp, eight slots a lane: 99 registers, 75 without them).
template <class T, int N>
DISC_DEV void opaque(Vec<T, N>& x) {
  constexpr int W = (int)sizeof(x.v) / 4;
  if constexpr (W > 0) {
    u32 w[W];
    __builtin_memcpy(w, &x.v, W * 4);
#pragma unroll
    for (int i = 0; i < W; ++i) asm volatile("" : "+v"(w[i]));
    __builtin_memcpy(&x.v, w, W * 4);
  }
}
template <class Pat, int V>
DISC_DEV typename Pat::template Slot<V>& as_loaded(typename Pat::template Slot<V>& s) {
  Pat::template opaque<V>(s);
  return s;
}
// The same as a copy, for the streaming version of four slots a lane, where the padding is a word or two: dot product of
// bf16 rows 58 registers, 63 in place, maximum with position 63 / 71, residual + LayerNorm 93 / 106.
template <class S>
DISC_DEV S copied(const S& s) {
  constexpr int W = (int)(sizeof(S) - sizeof(int)) / 4;      // (the last member is a placeholder)
  u32 w[W > 0 ? W : 1];
  __builtin_memcpy(w, &s, W * 4);
#pragma unroll
  for (int i = 0; i < W; ++i) asm volatile("" : "+v"(w[i]));
  S r;
  __builtin_memcpy(&r, w, W * 4);
  return r;
}
template <class Pat, int V, int NR>
struct StreamRow {
  typename Pat::template Slot<V> held[NR > 0 ? NR : 1];
  typename Pat::template Slot<1> end;
  int end_col;            // column of this lane's single element, -1: none
};
// The row of `rc` as held slots, and the elements behind the last whole slot one each to the first lanes.  A macro: filled
// through a reference (stream_fill) the row takes 15 to 35 registers more, and so fewer wavefronts: log-sum-exp with eight
// slots a lane 75, 63 like this; maximum with position 127 / 95 (4096 x 32000 62 us / 45), dot product of bf16 rows with four
// 78 / 58 (270 x 20800 6.8 / 6.2), LayerNorm backward 128 with 12 spilled / 105 (3000 x 30000 381 / 365).
#define DISC_STREAM_FILL(r, NT)                                                                               \
  do {                                                                                                        \
    _Pragma("unroll") for (int j = 0; j < NR; ++j) {                                                          \
      const int col = (int)(j * blockDim.x + threadIdx.x) * V;                                                \
      if (col < whole) Pat::template load<V, NT>(A, rc, col, TailSpan::upto(V), r.held[j]);                   \
    }                                                                                                         \
    r.end_col = whole + (int)threadIdx.x < inner ? whole + (int)threadIdx.x : -1;                             \
    if (r.end_col >= 0) Pat::template load<1>(A, rc, r.end_col, TailSpan::upto(1), r.end);                    \
    if constexpr (NR > 0) asm volatile("" ::: "memory");     /* all of these loads before the first phase */  \
  } while (0)
// Patterns that write an element per element and sum nothing over the rows are faster with the fewer wavefronts (5000 x
// 26000: residual + LayerNorm 185 us, 190 through the macro; mixed chain 187 / 194; softmax the same).
template <class Pat, int V, int NR>
DISC_DEV void stream_fill(const typename Pat::Args& A, const typename Pat::RowCtx& rc, int inner, int whole, StreamRow<Pat, V, NR>& r) {
  DISC_STREAM_FILL(r, 0);
}
// The block's partial results of reductions of per-row values over the rows
template <class Pat>
DISC_DEV void stream_row_reds(const typename Pat::Args& A, const float (&racc)[Pat::NROWRED]) {
  if (threadIdx.x == 0) {
#pragma unroll
    for (int q = 0; q < Pat::NROWRED; ++q) reinterpret_cast<float*>(A.ws1)[(i64)q * A.aux1 + blockIdx.x] = racc[q];
  }
}

// S: held slots that a sum adds up in one chain; more of them meet as partial sums.
template <class Pat, int P, int V, int NR, int S>
DISC_DEV void row_stream_phases(const typename Pat::Args& A, typename Pat::RowCtx& rc, int whole,
                                StreamRow<Pat, V, NR>& r, char* lds, int& parity) {
  if constexpr (P < Pat::NPHASE) {
    typedef typename Pat::template Acc<P> AccT;
    constexpr bool split = S < NR && (Pat::SUM_PHASES >> P & 1);
    AccT acc, part;
    Pat::template acc_init<P>(acc);
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int col = (int)(j * blockDim.x + threadIdx.x) * V;
      typename Pat::template Keep<V> kp;
      if (split && j % S == 0) Pat::template acc_init<P>(part);
      if (col < whole) {
        if constexpr (S < NR) Pat::template phase<P, V, false>(A, split ? part : acc, as_loaded<Pat, V>(r.held[j]), kp, TailSpan::upto(V), col, rc);
        else Pat::template phase<P, V, false>(A, acc, copied(r.held[j]), kp, TailSpan::upto(V), col, rc);
      }
      if (split && (j % S == S - 1 || j == NR - 1)) Pat::template acc_merge<P>(acc, part);
    }
    for (int col = (int)(NR * blockDim.x + threadIdx.x) * V; col < whole; col += blockDim.x * V) {
      typename Pat::template Slot<V> slot;
      Pat::template load<V>(A, rc, col, TailSpan::upto(V), slot);
      typename Pat::template Keep<V> kp;
      Pat::template phase<P, V, false>(A, acc, slot, kp, TailSpan::upto(V), col, rc);
    }
    if (r.end_col >= 0) {
      typename Pat::template Keep<1> kp;
      Pat::template phase<P, 1, false>(A, acc, r.end, kp, TailSpan::upto(1), r.end_col, rc);
    }
    group_allreduce<Pat, P>(acc, 64);
    AccT* ex = reinterpret_cast<AccT*>(lds + parity * 16 * Pat::MAX_ACC_BYTES);
    parity ^= 1;
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) ex[wave] = acc;
    __syncthreads();
    const int nw = __builtin_amdgcn_readfirstlane((int)(blockDim.x >> 6));         // a power of two
    acc = ex[(int)threadIdx.x & (nw - 1)];
    group_allreduce<Pat, P>(acc, nw);
    Pat::template row_after<P>(A, rc, acc);
    row_stream_phases<Pat, P + 1, V, NR, S>(A, rc, whole, r, lds, parity);
  }
}

// The same for patterns that write nothing per element and sum nothing over the rows.  Bound by the reads.
// There is no store for a block's loads to hide behind, so what counts is how many rows a CU holds in
// different phases: the least block that holds the row, down to one wavefront, with NR = 8 slots a lane
// in place of the four of row_stream_body (blocks of 512 threads at most: at 1024 only one would fit a CU).
// bf16 log-sum-exp, four slots / eight: 8000 x 16000 54 us / 45 (5.7 TB/s), 4096 x 32000 57 / 50,
// 16384 x 8000 54 / 48, 16384 x 4096 34 / 28.5.  Loading the next row while one is worked on took 44.4, 51.2, 50.4
// and, in blocks of 1024, 61.8 us where four slots take 62 (2096 x 64000); 16 slots on half the threads 53 and
// 51.6; 80 registers (28 of them spilled) 70 and 63.
// Twice the slots on a lane would be a chain of fp32 additions twice as long (sums of squares of 16013 bf16 values: 5.3e-8
// off, 4.0e-8 with four slots a lane): two slots to a chain, whose sums meet.
template <class Pat, int V, int NR, int NT>
DISC_DEV void row_held_run(const typename Pat::Args& A) {
  __shared__ __attribute__((aligned(16))) char lds[2 * 16 * Pat::MAX_ACC_BYTES];
  const int inner = (int)A.inner, whole = inner / V * V;
  int parity = 0;
  float racc[Pat::NROWRED > 0 ? Pat::NROWRED : 1];
  if constexpr (Pat::NROWRED > 0) {
#pragma unroll
    for (int q = 0; q < Pat::NROWRED; ++q) racc[q] = Pat::rr_identity(q);
  }
  for (i64 row = blockIdx.x; row < A.rows; row += gridDim.x) {
    typename Pat::RowCtx rc;
    Pat::row_begin(A, row, rc);
    rc.sl = nullptr;
    StreamRow<Pat, V, NR> r;
    DISC_STREAM_FILL(r, NT);
    row_stream_phases<Pat, 0, V, NR, 2>(A, rc, whole, r, lds, parity);
    if constexpr (Pat::NROWRED > 0) Pat::row_reds(A, rc, racc);   // (every lane holds the row's values)
    if (threadIdx.x == 0) Pat::row_store(A, row, rc);
  }
  if constexpr (Pat::NROWRED > 0) stream_row_reds<Pat>(A, racc);
}
// A.aux2: non-temporal loads of the held slots (behind a branch inside the body the compiler would merge the
// two kinds of access into a plain one)
template <class Pat, int V, int NR>
DISC_DEV void row_held_body(const typename Pat::Args& A) {
  if (A.aux2) row_held_run<Pat, V, NR, 1>(A);
  else row_held_run<Pat, V, NR, 0>(A);
}

template <class Pat, int V, int NR>
DISC_DEV void row_stream_body(const typename Pat::Args& A) {
  __shared__ __attribute__((aligned(16))) char lds[2 * 16 * Pat::MAX_ACC_BYTES];
  const int inner = (int)A.inner, whole = inner / V * V;
  int parity = 0;
  bool first = true;
  float racc[Pat::NROWRED > 0 ? Pat::NROWRED : 1];
  if constexpr (Pat::NROWRED > 0) {
#pragma unroll
    for (int q = 0; q < Pat::NROWRED; ++q) racc[q] = Pat::rr_identity(q);
  }
  for (i64 row = blockIdx.x; row < A.rows; row += gridDim.x) {
    typename Pat::RowCtx rc;
    Pat::row_begin(A, row, rc);
    rc.sl = nullptr;
    StreamRow<Pat, V, NR> r;
    if constexpr (Pat::HAS_ELEM_OUT && Pat::NCOLSUM == 0) stream_fill<Pat, V, NR>(A, rc, inner, whole, r);
    else DISC_STREAM_FILL(r, 0);
    row_stream_phases<Pat, 0, V, NR, NR>(A, rc, whole, r, lds, parity);
    if constexpr (Pat::NROWRED > 0) Pat::row_reds(A, rc, racc);   // (every lane holds the row's values)
    auto finish = [&](auto slot, auto width, int col) {
      constexpr int W = decltype(width)::value;
      typename Pat::template OutSlot<W> o;
      typename Pat::template Keep<W> kp;
      Pat::template epilogue<W, false>(A, rc, slot, kp, col, TailSpan::upto(W), o);
      Pat::template store<W>(A, rc, col, TailSpan::upto(W), o);
      if constexpr (Pat::NCOLSUM > 0) {
        // sums over the rows: the block's row of partial sums lives in the workspace (the rows are
        // too long for registers); every lane owns its columns there, so no other lane touches them
        typename Pat::template ColAcc<W> ca{};
        Pat::template col_sums<W, false>(A, rc, slot, kp, col, TailSpan::upto(W), ca);
#pragma unroll
        for (int q = 0; q < Pat::NCOLSUM; ++q) {
          float* dst = reinterpret_cast<float*>(A.ws0) + ((i64)q * A.aux0 + blockIdx.x) * A.inner;
          Vec<float, W> t;
          t.v = ca.c[q];
          if (!first) {
            Vec<float, W> old;
            ld(old, dst, (i64)col, TailSpan::upto(W));
            t.v += old.v;
          }
          st(dst, (i64)col, t, TailSpan::upto(W));
        }
      }
    };
    if constexpr (Pat::HAS_ELEM_OUT || Pat::NCOLSUM > 0) {
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const int col = (int)(j * blockDim.x + threadIdx.x) * V;
        if (col < whole) finish(copied(r.held[j]), IntC<V>{}, col);
      }
      for (int col = (int)(NR * blockDim.x + threadIdx.x) * V; col < whole; col += blockDim.x * V) {
        typename Pat::template Slot<V> slot;
        Pat::template load<V>(A, rc, col, TailSpan::upto(V), slot);
        finish(slot, IntC<V>{}, col);
      }
      if (r.end_col >= 0) finish(r.end, IntC<1>{}, r.end_col);
    }
    if (threadIdx.x == 0) Pat::row_store(A, row, rc);
    first = false;
  }
  if constexpr (Pat::NROWRED > 0) stream_row_reds<Pat>(A, racc);
}

#undef DISC_STREAM_FILL

// An element-wise pattern with sums over the rows (no reduction along the rows: NPHASE = 0) does not need
// a row in one block.  A block of 256 threads is TX = A.aux1 lanes along the columns (a power of two;
// 256 for long rows, which then take gridDim.y blocks) times TY = 256 / TX rows; a lane keeps its
// columns, U rows in flight, and its sums in registers.  Nothing is exchanged between the lanes until
// the end, where the TY lanes of a column meet in LDS and the block writes its part of one row of
// partial sums.  Rows are dealt out one by one, so that the blocks of a launch stream through the
// tensor side by side.  Few blocks mean that a lane adds up many rows (hundreds, in wide tensors), so
// all of it is in fp64, and a few partial rows, or those of few rows, go to the workspace in fp64 too
// (A.aux2): a sum is then rounded once, however the rows were split.  Relative rms error of the sums
// of normally distributed values (half an ulp of the result alone is 2.5e-8), fp32 rows of partial sums of
// fp32 chains in runs of 16 / as it is here: 4000 x 200000 1.5e-7 / 2.5e-8, 700 x 8192 4.8e-8 / 2.5e-8, 32768 x 512
// 9.1e-8 / 3.5e-8.  GELU backward, the same: 8192 x 16384 137.2 us / 135.3, 32768 x 512 22.4 / 22.4.
template <class Pat, int V, int U, int NT, class SP>
DISC_DEV void row_cols_body(const typename Pat::Args& A) {
  __shared__ double cbuf[V][256 + 8];                          // (pitch: the V columns of a slot on other banks)
  const int TX = (int)A.aux1, TY = 256 / TX;
  const int tx = (int)threadIdx.x & (TX - 1);
  // (whole wavefronts along a row: the row number is a scalar)
  int ty = (int)threadIdx.x / TX;
  const int col = ((int)blockIdx.y * TX + tx) * V;
  const i64 rem = A.inner - col;
  const bool mine = rem > 0;
  const SP sp = SP::upto(rem < (i64)V ? (int)rem : V);
  double acc[Pat::NCOLSUM][V];
#pragma unroll
  for (int q = 0; q < Pat::NCOLSUM; ++q)
#pragma unroll
    for (int e = 0; e < V; ++e) acc[q][e] = 0.0;
  auto walk = [&](i64 row) {
    typename Pat::template Late<V> same;          // operands that are the same in every row
    {
      typename Pat::RowCtx rc;
      Pat::row_begin(A, 0, rc);
      Pat::template load_late<V>(A, rc, col, sp, same);
    }
    const char* held = reinterpret_cast<const char*>(&same);
    auto begin = [&](i64 r, typename Pat::RowCtx& rc, typename Pat::template Slot<V>& slot) {
      Pat::row_begin(A, r, rc);
      rc.sl = held;
      Pat::template load<V, NT>(A, rc, col, sp, slot);
    };
    auto finish = [&](const typename Pat::RowCtx& rc, const typename Pat::template Slot<V>& slot) {
      typename Pat::template OutSlot<V> o;
      typename Pat::template Keep<V> keep;
      Pat::template epilogue<V, false>(A, rc, slot, keep, col, sp, o);
      Pat::template store<V, NT>(A, rc, col, sp, o);
      typename Pat::template ColAcc<V> one;        // (-0 + x is x, which the compiler knows)
#pragma unroll
      for (int q = 0; q < Pat::NCOLSUM; ++q) one.c[q] = -0.0f;
      Pat::template col_sums<V, false>(A, rc, slot, keep, col, sp, one);
#pragma unroll
      for (int q = 0; q < Pat::NCOLSUM; ++q)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[q][e] += (double)one.c[q][e];
    };
    const i64 step = (i64)gridDim.x * TY;
    for (; row + (U - 1) * step < A.rows; row += U * step) {
      typename Pat::RowCtx rc[U];
      typename Pat::template Slot<V> slot[U];
#pragma unroll
      for (int u = 0; u < U; ++u) begin(row + u * step, rc[u], slot[u]);
      asm volatile("" ::: "memory");     // all loads of the batch before its first row
#pragma unroll
      for (int u = 0; u < U; ++u) finish(rc[u], slot[u]);
    }
    for (; row < A.rows; row += step) {
      typename Pat::RowCtx rc;
      typename Pat::template Slot<V> slot;
      begin(row, rc, slot);
      finish(rc, slot);
    }
  };
  if (mine) {
    if (TX >= 64) walk((i64)blockIdx.x * TY + __builtin_amdgcn_readfirstlane(ty));
    else walk((i64)blockIdx.x * TY + ty);
  }
  int filled = TY;                                           // (a power of two) lanes of a column that may have had a row
  while (filled > 1 && filled / 2 >= A.rows) filled >>= 1;
  const i64 tile = (i64)blockIdx.y * TX * V;                 // first column of the block
  const int cols = A.inner - tile < (i64)TX * V ? (int)(A.inner - tile) : TX * V;
#pragma unroll
  for (int q = 0; q < Pat::NCOLSUM; ++q) {
#pragma unroll
    for (int e = 0; e < V; ++e) cbuf[e][threadIdx.x] = acc[q][e];
    // more than 16 rows: halves fold onto each other, every step a lane adds what lies s rows behind it
    int left = filled;
    for (; left > 16; left >>= 1) {
      __syncthreads();
      const int s = left >> 1;
      if (ty < s) {
#pragma unroll
        for (int e = 0; e < V; ++e) cbuf[e][threadIdx.x] += cbuf[e][(int)threadIdx.x + s * TX];
      }
    }
    __syncthreads();
    const i64 at = ((i64)q * A.aux0 + blockIdx.x) * A.inner + tile;
    for (int c = (int)threadIdx.x; c < cols; c += 256) {
      double t = cbuf[c % V][c / V];
      for (int k = 1; k < left; ++k) t += cbuf[c % V][c / V + k * TX];
      if (A.aux2) reinterpret_cast<double*>(A.ws0)[at + c] = t;
      else reinterpret_cast<float*>(A.ws0)[at + c] = (float)t;
    }
    if (q + 1 < Pat::NCOLSUM) __syncthreads();
  }
}

// Last launch of a row reduce with reductions of per-row values over the rows: one block of 1024
// threads folds the per-block partial results of every reduction in a fixed order (sums in fp64)
// and stores them.  All reductions advance together and two strides are in flight per lane, so a
// lane makes one or two dependent trips to memory for the couple of thousand partial results of a
// large launch (a 256-thread block that took the reductions one after the other needed 14 us).
template <class Pat>
DISC_DEV void rowred_finish_body(const typename Pat::Args& A) {
  constexpr int NQ = Pat::NROWRED;
  __shared__ double red[NQ][1024];
  const float* ws = reinterpret_cast<const float*>(A.ws1);
  const i64 P = A.aux1;
  const int nt = (int)blockDim.x, tid = (int)threadIdx.x;      // nt: a power of two <= 1024
  double t0[NQ], t1[NQ];
#pragma unroll
  for (int q = 0; q < NQ; ++q) t0[q] = t1[q] = (double)Pat::rr_identity(q);
  i64 i = tid;
  for (; i + nt < P; i += 2 * nt) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const float a = ws[(i64)q * P + i], b = ws[(i64)q * P + i + nt];
      t0[q] = Pat::rr_merge(q, t0[q], (double)a);
      t1[q] = Pat::rr_merge(q, t1[q], (double)b);
    }
  }
  for (; i < P; i += nt) {
#pragma unroll
    for (int q = 0; q < NQ; ++q) t0[q] = Pat::rr_merge(q, t0[q], (double)ws[(i64)q * P + i]);
  }
#pragma unroll
  for (int q = 0; q < NQ; ++q) red[q][tid] = Pat::rr_merge(q, t0[q], t1[q]);
  __syncthreads();
  for (int s = nt >> 1; s > 0; s >>= 1) {
    if (tid < s) {
#pragma unroll
      for (int q = 0; q < NQ; ++q) red[q][tid] = Pat::rr_merge(q, red[q][tid], red[q][tid + s]);
    }
    __syncthreads();
  }
  if (tid == 0) {
    float v[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) v[q] = (float)red[q][0];
    Pat::rowred_store(A, v);
  }
}

// Second launch of a row reduce with sums over the rows: adds up the P rows of partial sums of
// every summed output, in a fixed order (the result does not depend on timing) and in fp64
// (partial sums in fp32 each cover the rows of one block only).  A block takes 16 columns; its 256
// lanes are 16 columns x 16 lanes that each walk every 16th partial row of all sums together, sixteen
// loads in flight, the ones past the last row from a lane's last row instead (a tail of single loads is a chain of trips
// to memory); the lanes of a column meet by lane exchanges, then in LDS.
// Bound by those trips.  Whole calls, us, four loads in flight a lane and sum and a tail of single ones / this: LayerNorm
// backward (two sums) 32768 x 1024 (767 partial rows) 47.3 / 45.7, 65536 x 128 24.6 / 22.9, 2000 x 768 (250) 13.8 / 13.0, 100 x 1024
// 8.6 / 8.2; GELU backward 3000 x 2048 11.5 / 11.5, 8192 x 16384 (16) 135.4 / 135.4, 136.6 in batches.  512 lanes, 32 to a column, with eight loads: 44.8,
// 22.2, 12.8, but 9.0 and 11.9 for the small ones.  All loads clamped, not the last batch alone: 100 x 1024 9.0, 3000 x 2048
// 12.2.  With branches around the loads they came one by one: 64.5.
constexpr int kColsumCols = 16;
template <class Pat, class PART>
DISC_DEV void colsum_add_up(const typename Pat::Args& A) {
  constexpr int NQ = Pat::NCOLSUM, CL = kColsumCols;
  __shared__ double red[NQ][4][CL];
  const int cl = (int)threadIdx.x % CL, pl = (int)threadIdx.x / CL;
  constexpr int PL = 256 / CL;
  const i64 inner = A.inner, P = A.aux0;
  const PART* ws = reinterpret_cast<const PART*>(A.ws0);
  for (i64 c0 = (i64)blockIdx.x * CL; c0 < inner; c0 += (i64)gridDim.x * CL) {
    const i64 col = c0 + cl;
    constexpr int U = NQ >= 2 ? 8 : 16, UT = U / 2;    // partial rows in flight per lane and sum; ... behind the whole batches
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    if (col < inner) {
      const i64 plane = P * inner, step = PL * inner;
      const PART* src = ws + col + pl * inner;
      int n = pl < P ? (int)((P - pl + PL - 1) / PL) : 0;   // this lane's partial rows
      for (; n >= U; n -= U) {
        PART x[NQ][U];
#pragma unroll
        for (int u = 0; u < U; ++u, src += step)
#pragma unroll
          for (int q = 0; q < NQ; ++q) x[q][u] = src[q * plane];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int u = 0; u < U; ++u) acc[q] += (double)x[q][u];
      }
      if (P <= 2 * PL) {                          // one or two rows for every lane
        for (; n > 0; --n, src += step)
#pragma unroll
          for (int q = 0; q < NQ; ++q) acc[q] += (double)src[q * plane];
      }
      for (; n > 0; n -= UT) {
        PART x[NQ][UT];
#pragma unroll
        for (int u = 0; u < UT; ++u) {
#pragma unroll
          for (int q = 0; q < NQ; ++q) x[q][u] = src[q * plane];
          src += u + 1 < n ? step : 0;
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
          for (int u = 0; u < UT; ++u) acc[q] += u < n ? (double)x[q][u] : 0.0;
      }
    }
#pragma unroll
    for (int q = 0; q < NQ; ++q) {                // the four lanes of a column in a wavefront, then the wavefronts
      acc[q] += lane_xchg<16>(acc[q]);
      acc[q] += lane_xchg<32>(acc[q]);
      if (((int)threadIdx.x & 63) < CL) red[q][threadIdx.x >> 6][cl] = acc[q];
    }
    __syncthreads();
    if (pl == 0 && col < inner) {
      float v[NQ];
#pragma unroll
      for (int q = 0; q < NQ; ++q) {
        double t = 0.0;
#pragma unroll
        for (int k = 0; k < 4; ++k) t += red[q][k][cl];
        v[q] = (float)t;
      }
      Pat::colsum_store(A, col, v);
    }
    __syncthreads();
  }
}
// A.aux2: the partial rows are fp64 (row_cols_body)
template <class Pat>
DISC_DEV void colsum_finish_body(const typename Pat::Args& A) {
  if constexpr (Pat::ROW_COLS) {
    if (A.aux2) return colsum_add_up<Pat, double>(A);
  }
  colsum_add_up<Pat, float>(A);
}

// =======================================================================================
// A transpose on its own (not a fusion): out[b][p][q] = in[b][q][p], any element type.  A block
// moves square tiles through LDS so that both the reads (along p, the operand's innermost axis)
// and the writes (along q) are contiguous.  Every global access is 16 bytes wide (8 two-byte
// elements), and a tile row is 256 bytes of the operand -- two whole cache lines per row on both
// sides: 128 x 128 tiles for one- and two-byte elements, 64 x 64 for wider ones (with 64 x 64
// tiles and one element per lane, two-byte elements moved 128 bytes per row and reached 2.5 TB/s
// where four-byte elements reached 4.3).  A lane issues all its loads of a tile before the first
// LDS write.  The LDS row pitch is an odd number of dwords, so the column-wise element reads of
// the second half spread over the banks.
// =======================================================================================
// Which tile is the t-th: its batch entry, and its first row and column in the result.  Where tiles of one result row
// end inside cache lines, the two parts of a line should meet in one L2: `lists` gives every XCD (block t runs
// on t mod 8) a contiguous eighth of the tiles, result columns first over kTransposeNear tile rows at a time, whose operand rows lie
// side by side.  Otherwise consecutive blocks walk a diagonal of the tile grid: with a power-of-two row pitch
// the tiles of one tile row (or column) would otherwise queue up on the same memory channels.
// us, diagonal / lists, a tile to a block: bf16 6000 x 4097 24.4 / 22.4, 9000 x 9000 95.0 / 76.5, 3001 x 5000 16.9 / 12.2, 701 x 30000
// 23.4 / 17.8; f32 12001 x 8003 243 / 187.  (1 / 3 / 8 tile rows at a time: 6000 x 7000 41.7 / - / 41.7, 41.0 with 4; 30000
// x 500 15.1 / 15.0 / 13.3, 13.3 with 4.)  The host asks for lists below 2^29 tiles: kTransposeNear rows of them fit 32 bits.
constexpr u32 kTransposeNear = 4;
DISC_DEV i64 transpose_place(i64 t, i64 batch, i64 tiles_p, i64 tiles_q, int TP, int TQ, bool lists, i64& p0, i64& q0) {
  const i64 per_batch = tiles_p * tiles_q;
  i64 b, tq, tp;
  if (batch * per_batch < (1LL << 31)) {         // (64-bit divisions take 0.3 us each in front of the first load)
    const u32 pb = (u32)per_batch, Tp = (u32)tiles_p, Tq = (u32)tiles_q;
    u32 k = (u32)t, n, p, q;
    if (lists) {
      const u32 all = (u32)batch * pb, x = k & 7, extra = all & 7;
      k = x * (all >> 3) + (x < extra ? x : extra) + (k >> 3);
    }
    n = batch > 1 ? k / pb : 0;
    k -= n * pb;
    if (lists) {
      const u32 g = k / (kTransposeNear * Tq), in = k - g * (kTransposeNear * Tq), left = Tp - g * kTransposeNear;
      q = left >= kTransposeNear ? in / kTransposeNear : in / left;
      p = g * kTransposeNear + in - q * (left >= kTransposeNear ? kTransposeNear : left);
    } else {
      q = k / Tp;
      p = k - q * Tp + q;
      if (p >= Tp) p %= Tp;
    }
    b = __builtin_amdgcn_readfirstlane((int)n);
    tq = __builtin_amdgcn_readfirstlane((int)q);
    tp = __builtin_amdgcn_readfirstlane((int)p);
  } else {
    b = t / per_batch;
    const i64 r = t - b * per_batch;
    tq = r / tiles_p;
    tp = r - tq * tiles_p + tq;
    if (tp >= tiles_p) tp %= tiles_p;
  }
  p0 = tp * TP;
  q0 = tq * TQ;
  return b;
}
// Two-byte elements: tiles of TP result rows x TQ result columns.  A lane loads the same eight elements of two operand
// rows, packs those that will be neighbours into dwords and writes these, so that the other half reads whole
// 16-byte pieces: ten LDS accesses per 16 elements in place of 32.  The dword of row pair r and column c lies at
// r ^ (c / 8 << 2): the accesses that a wavefront makes side by side fall on all banks.
// Bound by memory, and by how evenly the tiles spread over its channels; bf16, us, single elements through LDS / packed,
// 128 x 128 / packed, 128 x 64: 1000 x 1000 7.0 / 6.9 / 4.6, 4000 x 4001 16.1 / 16.1 / 14.2, 30000 x 500 19.2 / 16.0 / 14.4, 6000 x
// 4097 with a softmax behind it 40.7 / 40.2 / 39.3; 8192 x 8192 62 / 62 / 67.7, 5000 x 9000 52.7 / - / 62.7, 16384 x 8192 121 / -
// / 144.  (64 x 128: 42.1 and 65.4, 64 x 64: 42.6 and 56.6 at 6000 x 4097 and 8192 x 8192.)
template <int TP, int TQ, class T>
DISC_DEV void ktranspose2_body(const T* __restrict__ in, T* __restrict__ out, i64 batch, i64 P, i64 Q, bool lists) {
  static_assert(sizeof(T) == 2 && TP == 128 && (TQ == 64 || TQ == 128), "two-byte elements");
  constexpr int VP = TP / 8, VQ = TQ / 8, PQ = TQ / 2;
  constexpr int NP = PQ * VP / 256, NR = TP * VQ / 256;      // pairs of 16-byte loads, and stores, of a lane
  typedef u32 u32x4 __attribute__((ext_vector_type(4)));
  __shared__ __attribute__((aligned(16))) u32 tile[TP * PQ];
  const i64 tiles_p = (P + TP - 1) / TP, tiles_q = (Q + TQ - 1) / TQ;
  const i64 ntiles = batch * tiles_p * tiles_q;
  const int v = (int)threadIdx.x % VP, g = (int)threadIdx.x / VP, vq = (int)threadIdx.x % VQ, c0 = (int)threadIdx.x / VQ;
  for (i64 t = blockIdx.x; t < ntiles; t += gridDim.x) {
    i64 p0, q0;
    const i64 b = transpose_place(t, batch, tiles_p, tiles_q, TP, TQ, lists, p0, q0);
    const T* src = in + b * P * Q;
    T* dst = out + b * P * Q;
    Vec<T, 8> x[NP][2];
#pragma unroll
    for (int k = 0; k < NP; ++k)
#pragma unroll
      for (int h = 0; h < 2; ++h) {               // row q of the operand, elements p ...
        const i64 q = q0 + 2 * (g + 256 / VP * k) + h, p = p0 + v * 8;
        if (q < Q) {
          if (p + 8 <= P) {
            x[k][h].v = *reinterpret_cast<const typename Vec<T, 8>::unaligned_t*>(src + q * P + p);
          } else {
            x[k][h].clear();
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (p + e < P) x[k][h].set(e, src[q * P + p + e]);
          }
        }
      }
#pragma unroll
    for (int k = 0; k < NP; ++k) {
      const u32x4 lo = __builtin_bit_cast(u32x4, x[k][0].v), hi = __builtin_bit_cast(u32x4, x[k][1].v);
      u32* at = tile + v * 8 * PQ + ((g + 256 / VP * k) ^ ((v << 2) & (PQ - 1)));
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        at[(2 * w) * PQ] = __builtin_amdgcn_perm(hi[w], lo[w], 0x05040100);
        at[(2 * w + 1) * PQ] = __builtin_amdgcn_perm(hi[w], lo[w], 0x07060302);
      }
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NR; ++k) {                // row p of the result, elements q ...
      const int c = c0 + 256 / VQ * k;
      const i64 p = p0 + c, q = q0 + vq * 8;
      Vec<T, 8> o;
      o.v = __builtin_bit_cast(typename Vec<T, 8>::vec_t,
                               *reinterpret_cast<const u32x4*>(tile + c * PQ + ((vq << 2) ^ (((c >> 3) << 2) & (PQ - 1)))));
      if (p < P) {
        if (q + 8 <= Q) {
          *reinterpret_cast<typename Vec<T, 8>::unaligned_t*>(dst + p * Q + q) = o.v;
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (q + e < Q) dst[p * Q + q + e] = o.get(e);
        }
      }
    }
    __syncthreads();
  }
}

template <class T>
DISC_DEV void ktranspose_body(const T* __restrict__ in, T* __restrict__ out, i64 batch, i64 P, i64 Q, bool lists) {
  constexpr int VE = 16 / (int)sizeof(T);                    // elements per 16-byte access
  constexpr int TS = sizeof(T) <= 2 ? 128 : 64;
  constexpr int PAD = sizeof(T) >= 4 ? 1 : 4 / (int)sizeof(T);
  constexpr int VPR = TS / VE;                               // 16-byte pieces per tile row
  constexpr int NVEC = TS * VPR / 256;                       // pieces per lane and tile
  __shared__ __attribute__((aligned(16))) T tile[TS][TS + PAD];
  const i64 tiles_p = (P + TS - 1) / TS, tiles_q = (Q + TS - 1) / TS;
  const i64 ntiles = batch * tiles_p * tiles_q;
  for (i64 t = blockIdx.x; t < ntiles; t += gridDim.x) {
    i64 p0, q0;
    const i64 b = transpose_place(t, batch, tiles_p, tiles_q, TS, TS, lists, p0, q0);
    const T* src = in + b * P * Q;
    T* dst = out + b * P * Q;
    Vec<T, VE> piece[NVEC];
#pragma unroll
    for (int k = 0; k < NVEC; ++k) {              // row q0 + row of the operand, elements p0 + v * VE ...
      const int idx = (int)threadIdx.x + k * 256;
      const int row = idx / VPR, v = idx % VPR;
      const i64 q = q0 + row, p = p0 + v * VE;
      piece[k].clear();
      if (q < Q) {
        if (p + VE <= P) {
          piece[k].v = *reinterpret_cast<const typename Vec<T, VE>::unaligned_t*>(src + q * P + p);
        } else {
#pragma unroll
          for (int e = 0; e < VE; ++e)
            if (p + e < P) piece[k].set(e, src[q * P + p + e]);
        }
      }
    }
#pragma unroll
    for (int k = 0; k < NVEC; ++k) {
      const int idx = (int)threadIdx.x + k * 256;
      const int row = idx / VPR, v = idx % VPR;
#pragma unroll
      for (int e = 0; e < VE; ++e) tile[row][v * VE + e] = piece[k].get(e);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < NVEC; ++k) {              // row p0 + row of the result, elements q0 + v * VE ...
      const int idx = (int)threadIdx.x + k * 256;
      const int row = idx / VPR, v = idx % VPR;
      const i64 p = p0 + row, q = q0 + v * VE;
      Vec<T, VE> o;
      o.clear();
#pragma unroll
      for (int e = 0; e < VE; ++e) o.set(e, tile[v * VE + e][row]);
      if (p < P) {
        if (q + VE <= Q) {
          *reinterpret_cast<typename Vec<T, VE>::unaligned_t*>(dst + p * Q + q) = o.v;
        } else {
#pragma unroll
          for (int e = 0; e < VE; ++e)
            if (q + e < Q) dst[p * Q + q + e] = o.get(e);
        }
      }
    }
    __syncthreads();
  }
}

// A row reduce whose one full-size operand comes in transposed: instead of a transpose kernel, a buffer and
// the row kernel, a block takes rpb rows of the result -- a strip of rpb columns of the operand
// [batch][inner][A.aux0] -- and turns them on the way into its registers.  Slot j of all its lanes is a piece of G * V
// operand rows: one 16-byte access per lane, all pieces at once, written to LDS by element and read back by row.
// The row stays in registers as loaded through all phases and the epilogue, as in the streaming version (values
// kept between the phases would take twice what is there).  The strips that share cache lines of the
// operand are dealt to one XCD.
// (A lane adds up to 16 slots where the row kernels have three: in one chain weighted sums of 1014 values a row were 1.5e-7
// off, 1.0e-7 in two kernels.)
// What bounds it: a strip of 16 or 32 bytes a row costs a cache line per access, and load, arithmetic and
// stores of a block follow one another, so a CU needs several strips.  Two strips after one another in a block, the
// second one loaded behind the first one's arithmetic, were no faster (8192 x 8192 99.9 us, 93.7 without).
template <class Pat, int P, int V, int NV, class SP>
DISC_DEV void row_xpose_phases(const typename Pat::Args& A, typename Pat::RowCtx& rc, typename Pat::template Slot<V> (&slot)[NV],
                               int lane, int G, int inner) {
  if constexpr (P < Pat::NPHASE) {
    constexpr bool split = Pat::SUM_PHASES >> P & 1;        // two slots to a chain of additions, whose sums meet
    typename Pat::template Acc<P> acc, part;
    Pat::template acc_init<P>(acc);
    asm volatile("" : "+v"(lane));           // (columns are cheaper to compute again than to keep)
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int col = (j * G + lane) * V;
      typename Pat::template Keep<V> kp;
      if (split && j % 2 == 0) Pat::template acc_init<P>(part);
      if (col < inner)
        Pat::template phase<P, V, false>(A, split ? part : acc, as_loaded<Pat, V>(slot[j]), kp, SP::upto(inner - col < V ? inner - col : V), col, rc);
      if (split && j % 2 == 1) Pat::template acc_merge<P>(acc, part);
    }
    group_allreduce<Pat, P>(acc, G);
    Pat::template row_after<P>(A, rc, acc);
    row_xpose_phases<Pat, P + 1, V, NV, SP>(A, rc, slot, lane, G, inner);
  }
}
// A.aux0 = rows of a batch entry, A.aux1 = strips of one, A.aux2 = strips in all, A.aux3 = strips per XCD;
// rp.flags = log2 of the 16-byte accesses of an operand row.  SP: EvenSpan where inner is a multiple of V.
template <class Pat, int V, int NV, class SP>
DISC_DEV void row_xpose_body(const typename Pat::Args& A, const RowPlan& rp) {
  typedef typename Pat::XpT T;
  static_assert(V * sizeof(T) == 16, "one 16-byte access per lane and piece");
  constexpr int PAD = V;                                      // (rows of the tile on other banks, reads aligned)
  __shared__ __attribute__((aligned(16))) T tile[2][1024 * V + 64 * PAD];
  const int strip = (int)(blockIdx.x & 7) * (int)A.aux3 + (int)(blockIdx.x >> 3);      // (the grid is a multiple of 8)
  if (strip >= (int)A.aux2) return;
  const i64 Q = A.aux0;
  const int P = (int)A.inner, G = rp.G, rpb = rp.rpb;
  // (the last strip of a batch entry starts where it ends with the last row; the host sees to Q >= rpb)
  const i64 batch = A.aux1 == A.aux2 ? 0 : (i64)((u32)strip / (u32)A.aux1);
  const i64 q0 = (strip - batch * A.aux1) * rpb, first = q0 + rpb <= Q ? q0 : Q - rpb;
  const int pitch = G * V + PAD;
  const int tp = (int)threadIdx.x >> rp.flags, tq = ((int)threadIdx.x & ((1 << rp.flags) - 1)) * V;
  const int lane = (int)threadIdx.x & (G - 1), grp = (int)threadIdx.x >> rp.log2G;
  typename Pat::template Slot<V> slot[NV];                    // (first the pieces, then, from LDS, the slots)
  {
    const T* src = Pat::xp_src(A) + batch * P * Q + first;
    const unsigned mine = (unsigned)tp * (unsigned)Q + (unsigned)tq;      // (fits in bytes: the host sees to it)
#pragma unroll
    for (int j = 0; j < NV; ++j)
      if (j * G * V + tp < P)
        Pat::template xp_slot<V>(slot[j]).v = *reinterpret_cast<const typename Vec<T, V>::unaligned_t*>(at(src + (i64)(j * G * V) * Q, mine));
    asm volatile("" ::: "memory");                            // all loads before the first piece is turned
  }
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    if (j * G * V < P) {
      T* t = tile[j & 1];
      Vec<T, V>& x = Pat::template xp_slot<V>(slot[j]);
#pragma unroll
      for (int e = 0; e < V; ++e) t[(tq + e) * pitch + tp] = x.get(e);
      __syncthreads();
      x.v = *reinterpret_cast<const typename Vec<T, V>::vec_t*>(t + grp * pitch + lane * V);
    }
  }
  const bool active = first + grp >= q0;                      // (its first rows are the strip's before it)
  const i64 row = batch * Q + first + grp;
  typename Pat::RowCtx rc;
  Pat::row_begin(A, row, rc);
  rc.sl = nullptr;
  row_xpose_phases<Pat, 0, V, NV, SP>(A, rc, slot, lane, G, P);
  int l = lane;
  asm volatile("" : "+v"(l));
#pragma unroll
  for (int j = 0; j < NV; ++j) {
    const int col = (j * G + l) * V;
    if (col < P) {
      const SP sp = SP::upto(P - col < V ? P - col : V);
      typename Pat::template OutSlot<V> o;
      typename Pat::template Keep<V> kp;
      Pat::template epilogue<V, false>(A, rc, as_loaded<Pat, V>(slot[j]), kp, col, sp, o);
      if (active) Pat::template store<V>(A, rc, (unsigned)col, sp, o);
    }
  }
  if (active && l == 0) Pat::row_store(A, row, rc);
}

// =======================================================================================
// Input fusion with a column reduction as root (reduce over an outer axis).  Canonical
// space [outer, mid, inner], `mid` reduced.  Three stages, no atomics, so results are
// bit-identical from run to run:
//   1. col_partial: the reduced axis is cut into chunks; a block owns one chunk of one column
//      tile.  Lanes run along `inner` (coalesced, V elements each), the block's row-lanes
//      stride over the rows of the chunk with four rows in flight; every lane keeps V column
//      accumulators (fp64 for fp32 sums).  The row-lanes of a column are combined through an
//      LDS transpose in fixed order and one partial per (chunk, column) goes to the workspace.
//   2. col_finish:  per column, partials are merged in fixed order; values and outputs that
//      no longer have the reduced axis (sum, mean, ...) are produced here.
//   3. the epilogue is a loop fusion (kloop_body) that reads the reduce results as column
//      vectors -- the tensor is read a second time, from Infinity Cache when it fits.
// =======================================================================================
struct ColPlan {
  int GC;          // lanes along inner per block, power of two <= 64
  int log2GC;
  int nchunk;      // chunks of the reduced axis
  int lists;       // order of the blocks, see col_place
  i64 chunk_rows;  // rows per chunk
  i64 outer;
  i64 epi_rows;    // two-launch version: rows of the reduced axis per block of the second launch
};

// V column accumulators of one lane over rows [m0 + ty, m1) with stride TY of outer slice o,
// four rows in flight
template <class Pat, int V>
DISC_DEV void col_accumulate(const typename Pat::Args& A, i64 o, i64 col, int nvalid, i64 m0, i64 m1, int ty, int TY,
                             typename Pat::template Acc<0> (&acc)[V]) {
#pragma unroll
  for (int e = 0; e < V; ++e) Pat::template acc_init<0>(acc[e]);
  if (nvalid <= 0) return;
  i64 m = m0 + ty;
  for (; m + 3 * TY < m1; m += 4 * TY) {
    typename Pat::template Slot<V> s[4];
    typename Pat::RowCtx rc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      Pat::row_begin(A, o * A.mid + m + u * TY, rc[u]);
      Pat::template load<V>(A, rc[u], col, Span::upto(nvalid), s[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (e < nvalid) Pat::template accum<0, V>(A, acc[e], s[u], e, (int)(m + u * TY), rc[u]);
  }
  for (; m < m1; m += TY) {
    typename Pat::template Slot<V> s;
    typename Pat::RowCtx rc;
    Pat::row_begin(A, o * A.mid + m, rc);
    Pat::template load<V>(A, rc, col, Span::upto(nvalid), s);
#pragma unroll
    for (int e = 0; e < V; ++e)
      if (e < nvalid) Pat::template accum<0, V>(A, acc[e], s, e, (int)m, rc);
  }
}

// Exchange with the lane whose number differs in bit S (a true xor exchange, unlike lane_xchg whose
// middle steps assume that earlier steps have run): DPP quad permutes, the swizzle unit for 4 and 8,
// the permlane swaps for 16 and 32.
template <int S>
DISC_DEV u32 lane_xor_u32(u32 v) {
  if constexpr (S == 1 || S == 2 || S == 16 || S == 32) return lane_xchg_u32<S>(v);
  else return (u32)__builtin_amdgcn_ds_swizzle((int)v, (S << 10) | 0x1f);   // bit mode: and 0x1f, or 0, xor S
}
template <int S, class T>
DISC_DEV T lane_xor_pod(const T& v) {
  static_assert(sizeof(T) % 4 == 0, "accumulators are made of 4- and 8-byte fields");
  u32 w[sizeof(T) / 4];
  __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
  for (int i = 0; i < (int)(sizeof(T) / 4); ++i) w[i] = lane_xor_u32<S>(w[i]);
  T r;
  __builtin_memcpy(&r, w, sizeof(T));
  return r;
}
template <class Pat, int S, int V>
DISC_DEV void col_lane_step(typename Pat::template Acc<0> (&acc)[V]) {
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const typename Pat::template Acc<0> o = lane_xor_pod<S>(acc[e]);
    Pat::template acc_merge<0>(acc[e], o);
  }
}

// The row-lanes of a block each hold accumulators of the same GC * V columns (thread = ty * GC + tx).
// Combines them column by column in a fixed order and leaves the block's result in EVERY lane:
// the lanes of a wavefront that hold the same columns meet through xor exchanges over the lane
// distances GC .. 32 (both partners compute the same commutative merge, so they agree bit for bit),
// then the wavefronts meet through one LDS cell per wavefront and column.  (One lane per column
// walking all row-lanes' cells in LDS, as before, cost up to 2 us per block with 128 row-lanes.)
// `lds` holds 4 * 64 * V accumulators; ends with a barrier, so the caller may reuse it at once.
// IDENTITY: from the identity on, one merge more and a few registers less.
template <class Pat, int V, bool IDENTITY = false>
DISC_DEV void col_block_merge(typename Pat::template Acc<0> (&acc)[V], typename Pat::template Acc<0>* lds, int GC, int tx) {
  int g = GC;
  asm volatile("" : "+s"(g));
  if (g <= 1) col_lane_step<Pat, 1, V>(acc);
  if (g <= 2) col_lane_step<Pat, 2, V>(acc);
  if (g <= 4) col_lane_step<Pat, 4, V>(acc);
  if (g <= 8) col_lane_step<Pat, 8, V>(acc);
  if (g <= 16) col_lane_step<Pat, 16, V>(acc);
  if (g <= 32) col_lane_step<Pat, 32, V>(acc);
  const int wave = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, nw = (int)blockDim.x >> 6;
  const int gw = GC < 64 ? GC : 64;          // columns-lanes per wavefront
  if (lane < gw) {
#pragma unroll
    for (int e = 0; e < V; ++e) lds[(wave * gw + lane) * V + e] = acc[e];
  }
  __syncthreads();
  // (A multiple of four wavefronts, their cells read side by side: one dependent LDS read after the other, a
  // strip of 1024 threads took 7.4 us instead of 6.4 and every call of two launches 1 us more.)
  // (Positions take registers that the waves in flight miss, and are read one by one: maximum with position, 2 x 13 x
  // 48740, 19.8 / 16.4 us.)
  constexpr int N = Pat::HAS_POSITION ? 1 : 4;
  auto cells = [&](int w, auto first) {
    typename Pat::template Acc<0> x[N][V];
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int e = 0; e < V; ++e) x[k][e] = lds[((w + k) * gw + tx) * V + e];
    if constexpr (first.value) {
#pragma unroll
      for (int e = 0; e < V; ++e) acc[e] = x[0][e];
    }
#pragma unroll
    for (int k = first.value; k < N; ++k)
#pragma unroll
      for (int e = 0; e < V; ++e) Pat::template acc_merge<0>(acc[e], x[k][e]);
  };
  if constexpr (IDENTITY) {
#pragma unroll
    for (int e = 0; e < V; ++e) Pat::template acc_init<0>(acc[e]);
  } else {
    cells(0, IntC<1>{});
  }
  for (int w = IDENTITY ? 0 : N; w < nw; w += N) cells(w, IntC<0>{});
  __syncthreads();
}

// Column tile and row range (chunk, in the first launch) of a block.  `lists`: every XCD (blocks i mod 8) takes a contiguous
// eighth of the tiles, all tiles of a row range before the next one: where the pieces of a row do not end on cache
// lines, their neighbours have the other part of a line, and meet in one L2 (dealt out one by one to the XCDs, a
// line was fetched and written in two).  fp32 centring, us, one by one / lists: 65536 x 700 187 / 140, 65536 x 333 114.6 / 68.2,
// 30000 x 1000 78.5 / 68.1, 10000 x 301 19.7 / 14.2; pieces of whole lines, 20000 x 1024 40.2 / 44.6.
// In the second launch (BACK) an XCD takes the same rows as in the first one, the last ones first: what it read last is the
// likeliest to be still in its L2, or in the memory-side cache (ranges from the end,
// XCDs the other way round: 4000 x 1000 15.7 us, 14.2 like this, 4000 x 300 10.5 / 9.5, 65536 x 333 72.3 / 70.5).
template <bool BACK>
DISC_DEV void col_place(bool lists, i64& tile, i64& range) {
  tile = blockIdx.x;
  range = BACK ? gridDim.y - 1 - blockIdx.y : blockIdx.y;
  if (lists) {                                  // (the host sees to fewer than 2^31 blocks)
    const u32 at = blockIdx.y * gridDim.x + blockIdx.x, n = gridDim.x * gridDim.y, x = at & 7, extra = n & 7;
    const u32 first = x * (n >> 3) + (x < extra ? x : extra), last = first + (n >> 3) - (x < extra ? 0 : 1);
    const u32 k = BACK ? last - (at >> 3) : first + (at >> 3), q = k / gridDim.x;
    range = __builtin_amdgcn_readfirstlane((int)q);
    tile = __builtin_amdgcn_readfirstlane((int)(k - q * gridDim.x));
  }
}

template <class Pat, int V>
DISC_DEV void col_partial_body(const typename Pat::Args& A, const ColPlan& cp) {
  typedef typename Pat::template Acc<0> AccT;
  __shared__ AccT lds[256 * V];
  i64 tile, chunk;
  col_place<false>(cp.lists != 0, tile, chunk);
  const int tx = threadIdx.x & (cp.GC - 1);
  const int ty = threadIdx.x >> cp.log2GC;
  const int TY = blockDim.x >> cp.log2GC;
  const i64 col = (tile * cp.GC + tx) * V;
  const i64 rem = A.inner - col;
  const int nvalid = rem <= 0 ? 0 : (rem < (i64)V ? (int)rem : V);
  const i64 m0 = chunk * cp.chunk_rows;
  const i64 m1 = m0 + cp.chunk_rows < A.mid ? m0 + cp.chunk_rows : A.mid;
  for (i64 o = blockIdx.z; o < cp.outer; o += gridDim.z) {
    AccT acc[V];
    col_accumulate<Pat, V>(A, o, col, nvalid, m0, m1, ty, TY, acc);
    col_block_merge<Pat, V>(acc, lds, cp.GC, tx);
    if (ty == 0) {
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (e < nvalid) Pat::acc_st(A, (o * cp.nchunk + chunk) * A.inner + col + e, acc[e]);
    }
  }
}

// The rows [m0, m1) of outer slice o, a block's share of them, through the epilogue: `base` holds
// the reduce results of the lane's columns (the same for every row), the operands are loaded into
// copies of it, four rows in flight per lane.
template <class Pat, class PatE, int V, int NT>
DISC_DEV void col_rows_epilogue(const typename Pat::Args& A, const typename PatE::template Slot<V>& base, i64 o, i64 col,
                                Span sp, i64 m0, i64 m1, int ty, int TY) {
  i64 m = m0 + ty;
  for (; m + 3 * TY < m1; m += 4 * TY) {
    typename PatE::template Slot<V> s[4];
    typename PatE::RowCtx rc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      s[u] = base;
      PatE::row_begin(A, o * A.mid + m + u * TY, rc[u]);
      PatE::template load_x<V, NT>(A, rc[u], col, sp, s[u]);
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      typename PatE::template OutSlot<V> out;
      typename PatE::template Keep<V> kp;
      PatE::template epilogue<V, false>(A, rc[u], s[u], kp, col, sp, out);
      PatE::template store<V, NT>(A, rc[u], col, sp, out);
    }
  }
  for (; m < m1; m += TY) {
    typename PatE::template Slot<V> s1 = base;
    typename PatE::RowCtx rc;
    PatE::row_begin(A, o * A.mid + m, rc);
    PatE::template load_x<V, NT>(A, rc, col, sp, s1);
    typename PatE::template OutSlot<V> out;
    typename PatE::template Keep<V> kp;
    PatE::template epilogue<V, false>(A, rc, s1, kp, col, sp, out);
    PatE::template store<V, NT>(A, rc, col, sp, out);
  }
}

// A strip whose rows all fit the lanes' registers, NR rows a lane: loaded once, all of it in flight, summed,
// merged and taken through the epilogue from there.  Bound by latency, one trip to memory, the merge and the
// stores: 700 x 1024 fp32 7.2 us with two passes of four rows in flight, 6.0 like this, 4.0-4.7 for an empty call.
template <class Pat, class PatE, int V, int NR>
DISC_DEV void col_strip_hold(const typename Pat::Args& A, const ColPlan& cp, typename Pat::template Acc<0>* lds, i64 o, i64 col,
                             int nvalid, int tx, int ty, int TY) {
  typedef typename Pat::template Acc<0> AccT;
  const int mid = (int)A.mid;
  typename Pat::template Slot<V> s[NR];
  const Span sp = Span::upto(nvalid);
  if (nvalid > 0) {
#pragma unroll
    for (int u = 0; u < NR; ++u) {
      const int m = ty + u * TY;
      if (m < mid) {
        typename Pat::RowCtx rc;
        Pat::row_begin(A, o * A.mid + m, rc);
        Pat::template load<V>(A, rc, col, sp, s[u]);
      }
    }
  }
  asm volatile("" ::: "memory");
  AccT acc[V];
#pragma unroll
  for (int e = 0; e < V; ++e) Pat::template acc_init<0>(acc[e]);
  if (nvalid > 0) {
#pragma unroll
    for (int u = 0; u < NR; ++u) {
      const int m = ty + u * TY;
      if (m < mid) {
        typename Pat::RowCtx rc;
        Pat::row_begin(A, o * A.mid + m, rc);
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (e < nvalid) Pat::template accum<0, V>(A, acc[e], s[u], e, m, rc);
      }
    }
  }
  col_block_merge<Pat, V, true>(acc, lds, cp.GC, tx);
  if (nvalid > 0) {
    typename PatE::template Slot<V> base;
    PatE::template clear_red<V>(base);
#pragma unroll
    for (int e = 0; e < V; ++e)
      if (e < nvalid) PatE::template finish_elem<V>(A, o, col + e, acc[e], base, e, ty == 0);
#pragma unroll
    for (int u = 0; u < NR; ++u) {
      const int m = ty + u * TY;
      if (m < mid) {
        typename PatE::RowCtx rc;
        PatE::row_begin(A, o * A.mid + m, rc);
        typename PatE::template Slot<V> x = base;
        PatE::template take<V>(x, s[u]);
        typename PatE::template OutSlot<V> out;
        typename PatE::template Keep<V> kp;
        PatE::template epilogue<V, false>(A, rc, x, kp, col, sp, out);
        PatE::template store<V, 0>(A, rc, col, sp, out);
      }
    }
  }
}

template <class Pat, class PatE, int V, int NR>
DISC_DEV void col_strip_held_body(const typename Pat::Args& A, const ColPlan& cp) {
  __shared__ typename Pat::template Acc<0> lds[256 * V];   // (blocks above 256 threads have at most 16 lanes along the columns)
  const int tx = threadIdx.x & (cp.GC - 1);
  const int ty = threadIdx.x >> cp.log2GC;
  const i64 col = ((i64)blockIdx.x * cp.GC + tx) * V;
  const i64 rem = A.inner - col;
  const int nvalid = rem <= 0 ? 0 : (rem < (i64)V ? (int)rem : V);
  for (i64 o = blockIdx.y; o < cp.outer; o += gridDim.y)
    col_strip_hold<Pat, PatE, V, NR>(A, cp, lds, o, col, nvalid, tx, ty, (int)(blockDim.x >> cp.log2GC));
}

// Single-launch version for small problems, where every further launch costs more than the work
// (a kernel that makes one round trip to memory takes 5-6 us on this part whatever it moves): a
// block owns a strip of GC * V columns and ALL rows of it.  It reduces the strip, every lane ends up
// with the results of its own columns in registers (col_block_merge), the lanes of the first row
// write the outputs that lost the reduced axis, and -- when the pattern has per-element outputs --
// the block walks its strip a second time for the epilogue, reading the tensor from cache.  Nothing
// goes through memory between the two passes.  PatE = void: no epilogue; the reduce results go to
// the workspace planes as in the three-launch version.
template <class Pat, class PatE, int V>
DISC_DEV void col_strip_body(const typename Pat::Args& A, const ColPlan& cp) {
  typedef typename Pat::template Acc<0> AccT;
  __shared__ AccT lds[256 * V];
  const int tx = threadIdx.x & (cp.GC - 1);
  const int ty = threadIdx.x >> cp.log2GC;
  const int TY = blockDim.x >> cp.log2GC;
  const i64 col = ((i64)blockIdx.x * cp.GC + tx) * V;
  const i64 rem = A.inner - col;
  const int nvalid = rem <= 0 ? 0 : (rem < (i64)V ? (int)rem : V);
  for (i64 o = blockIdx.y; o < cp.outer; o += gridDim.y) {
    AccT acc[V];
    col_accumulate<Pat, V>(A, o, col, nvalid, 0, A.mid, ty, TY, acc);
    col_block_merge<Pat, V>(acc, lds, cp.GC, tx);
    if constexpr (__is_same(PatE, void)) {
      if (ty == 0) {
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (e < nvalid) Pat::col_finish(A, o, col + e, acc[e]);
      }
    } else {
      if (nvalid > 0) {
        typename PatE::template Slot<V> base;
        PatE::template clear_red<V>(base);
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (e < nvalid) PatE::template finish_elem<V>(A, o, col + e, acc[e], base, e, ty == 0);
        col_rows_epilogue<Pat, PatE, V, 0>(A, base, o, col, Span::upto(nvalid), 0, A.mid, ty, TY);
      }
    }
  }
}

// Second of three launches: per column, the partials of all chunks merged in a fixed order.  A
// block takes 16 columns; its 256 lanes are 16 columns x 16 lanes that each walk every 16th chunk
// with four loads in flight, and the 16 lane results of a column meet in LDS.  (One lane per
// column walking the chunks one dependent load at a time, on inner / 64 blocks, took 18 us for
// 256 chunks x 1024 columns.)
template <class Pat>
DISC_DEV void col_finish_body(const typename Pat::Args& A, const ColPlan& cp) {
  typedef typename Pat::template Acc<0> AccT;
  constexpr int CL = 16, PL = 16;
  __shared__ AccT lds[PL][CL + 1];
  const int cl = (int)threadIdx.x % CL, pl = (int)threadIdx.x / CL;
  const i64 c = (i64)blockIdx.x * CL + cl;
  for (i64 o = blockIdx.y; o < cp.outer; o += gridDim.y) {
    AccT acc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) Pat::template acc_init<0>(acc[u]);
    if (c < A.inner) {
      const i64 base = o * cp.nchunk * A.inner + c;
      int j = pl;
      for (; j + 3 * PL < cp.nchunk; j += 4 * PL) {
        AccT t[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) Pat::acc_ld(A, base + (i64)(j + u * PL) * A.inner, t[u]);
#pragma unroll
        for (int u = 0; u < 4; ++u) Pat::template acc_merge<0>(acc[u], t[u]);
      }
      for (; j < cp.nchunk; j += PL) {
        AccT t;
        Pat::acc_ld(A, base + (i64)j * A.inner, t);
        Pat::template acc_merge<0>(acc[0], t);
      }
    }
#pragma unroll
    for (int u = 1; u < 4; ++u) Pat::template acc_merge<0>(acc[0], acc[u]);
    lds[pl][cl] = acc[0];
    __syncthreads();
    if (pl == 0 && c < A.inner) {
      AccT tot = lds[0][cl];
      for (int k = 1; k < PL; ++k) Pat::template acc_merge<0>(tot, lds[k][cl]);
      Pat::col_finish(A, o, c, tot);
    }
    __syncthreads();
  }
}

// Two-launch version: the second launch both finishes and applies the epilogue.  A block owns a
// column tile (the same GC * V columns as in the partial pass) and a range of rows.  It first merges
// the few chunk partials of its own columns (every block of a column tile repeats this small piece
// of work, in the same fixed order, so all of them hold the same results; the block of the first
// row range also writes the outputs that lost the reduced axis), keeps the reduce results in
// registers -- they are the same for every row -- and then streams its rows through the epilogue.
// No finish launch, no reduce-result planes in memory, no per-slot loads of them.
// The row ranges are handed out in reverse: the first blocks to start take the rows that the
// partial pass read last and that are most likely still in the memory-side cache.
// NT: bit 0 = non-temporal loads of the full-size operands, bit 1 = non-temporal stores.
template <class Pat, class PatE, int V, int NT>
DISC_DEV void col_epi2_body(const typename Pat::Args& A, const ColPlan& cp) {
  typedef typename Pat::template Acc<0> AccT;
  __shared__ AccT lds[256 * V];
  i64 tile, rb;
  col_place<true>(cp.lists != 0, tile, rb);
  const int tx = threadIdx.x & (cp.GC - 1);
  const int ty = threadIdx.x >> cp.log2GC;
  const int TY = blockDim.x >> cp.log2GC;
  const i64 col = (tile * cp.GC + tx) * V;
  const i64 rem = A.inner - col;
  const int nvalid = rem <= 0 ? 0 : (rem < (i64)V ? (int)rem : V);
  const i64 m0 = rb * cp.epi_rows;
  const i64 m1 = m0 + cp.epi_rows < A.mid ? m0 + cp.epi_rows : A.mid;
  for (i64 o = blockIdx.z; o < cp.outer; o += gridDim.z) {
    AccT acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) Pat::template acc_init<0>(acc[e]);
    if (nvalid > 0) {
      for (int j = ty; j < cp.nchunk; j += TY) {
        AccT t[V];
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (e < nvalid) Pat::acc_ld(A, (o * cp.nchunk + j) * A.inner + col + e, t[e]);
#pragma unroll
        for (int e = 0; e < V; ++e)
          if (e < nvalid) Pat::template acc_merge<0>(acc[e], t[e]);
      }
    }
    col_block_merge<Pat, V>(acc, lds, cp.GC, tx);
    if (nvalid > 0) {
      typename PatE::template Slot<V> base;
      PatE::template clear_red<V>(base);
#pragma unroll
      for (int e = 0; e < V; ++e)
        if (e < nvalid) PatE::template finish_elem<V>(A, o, col + e, acc[e], base, e, rb == 0 && ty == 0);
      col_rows_epilogue<Pat, PatE, V, NT>(A, base, o, col, Span::upto(nvalid), m0, m1, ty, TY);
    }
  }
}

// =======================================================================================
// Outputs whose size depends on the data (compaction by a predicate computed in the pattern; Unique
// of a sorted tensor is the case keep[i] = x[i] != x[i-1]).  Rank-1 values of length N = A.inner.
// A tile is 4 wavefronts x COMPACT_SLOTS slots x 64 lanes x V elements; a wavefront's part of it is
// contiguous and its slots are striped over the lanes, so every load and every rank store is one
// contiguous stretch per wavefront.  A slot's kept elements are one word of flags; what the lanes in
// front keep comes from one scan over the wavefront for two slots, and what a part keeps meets in LDS,
// so that it leaves as contiguous stores whatever the share that is kept.
// The output order is the input order; nothing is read back by the host:
//   1. compact_count:   evaluates the fused chain and counts what is kept; the counts go to the workspace.
//   2. compact_scan:    (short inputs only: a tile to a block) one block turns the counts into
//                       exclusive offsets, in a fixed order, and stores the total -- the
//                       data-dependent size -- in the COMPACT_COUNT outputs.
//   3. compact_scatter: evaluates the chain again (the inputs are read twice; nothing but the counts is kept between the
//                       launches) and stores the kept values and the ranks.  Without the scan launch every
//                       block adds up the counts in front of its own (four for each of at most 1024 blocks), and
//                       the last one stores the total.
//   Large inputs: compact_clear and compact_chain, which reads them once.
// =======================================================================================
constexpr int kCompactWaves = 4;          // wavefronts per block
// (slots per lane: Pat::COMPACT_SLOTS)
// The lane's number, not known to be the same from tile to tile: what is derived from it is cheap to
// derive again, and carried through the loop over the tiles it doubled the registers of the kernels.
DISC_DEV int opaque_lane() {
  int lane = (int)threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  return lane;
}

// The calling lane's slots of a wavefront's part of a tile.  `w0` = first element of the part (a scalar: the lanes add
// 32-bit offsets).  WHOLE: the part lies inside the tensor, so no slot is ragged and every load is one wide access; only
// slot 0 can be the tensor's first one.
template <bool WHOLE, class Pat, int V, int U>
DISC_DEV void compact_load(const typename Pat::Args& A, i64 w0, typename Pat::template Slot<V> (&slot)[U]) {
  const int lane = opaque_lane();
  typename Pat::RowCtx rc;
  Pat::row_begin3(A, 0, 0, w0, rc);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const unsigned at = (unsigned)((u * 64 + lane) * V);
    if constexpr (WHOLE) {
      if (u == 0) Pat::template load<V>(A, rc, at, EvenSpan::upto(V), slot[u]);
      else Pat::template load<V>(A, rc, at, InnerSpan::upto(V), slot[u]);
    } else {
      const i64 rem = A.inner - (w0 + at);
      if (rem > 0) Pat::template load<V>(A, rc, at, Span::upto(rem < (i64)V ? (int)rem : V), slot[u]);
    }
  }
}
// Their values, and one word of kept flags per slot (bit e = element e).
template <bool WHOLE, class Pat, int V, int U>
DISC_DEV void compact_eval(const typename Pat::Args& A, i64 w0, const typename Pat::template Slot<V> (&slot)[U],
                           typename Pat::template OutSlot<V> (&o)[U], u32 (&kb)[U]) {
  const int lane = opaque_lane();
  typename Pat::RowCtx rc;
  Pat::row_begin3(A, 0, 0, w0, rc);
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const i64 col = w0 + (u * 64 + lane) * V, rem = A.inner - col;
    const int n = WHOLE ? V : rem <= 0 ? 0 : (rem < (i64)V ? (int)rem : V);
    u32 bits = 0;
    if (n > 0) {
      typename Pat::template Keep<V> kp;
      typename Pat::template Slot<V> x = slot[u];
      Pat::template compact_prev<V>(x);
      if constexpr (!WHOLE) Pat::template epilogue<V, false>(A, rc, x, kp, col, Span::upto(n), o[u]);
      else if (u == 0) Pat::template epilogue<V, false>(A, rc, x, kp, col, EvenSpan::upto(n), o[u]);
      else Pat::template epilogue<V, false>(A, rc, x, kp, col, InnerSpan::upto(n), o[u]);
#pragma unroll
      for (int e = 0; e < V; ++e) bits |= (e < n && o[u].keep[e]) ? 1u << e : 0u;
    }
    kb[u] = bits;
  }
}
// Inclusive sum over the lanes of a wavefront, all of them active: four steps within rows of 16 lanes, then the last
// lane of a row to the row behind it and of a half to the other.
DISC_DEV u32 wave_scan(u32 x) {
  x += (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xf, 0xf, false);   // row_shr:1
  x += (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x112, 0xf, 0xf, false);
  x += (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x114, 0xf, 0xf, false);
  x += (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x118, 0xf, 0xf, false);
  x += (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x142, 0xa, 0xf, false);   // row_bcast:15, rows 1 and 3
  x += (u32)__builtin_amdgcn_update_dpp(0, (int)x, 0x143, 0xc, 0xf, false);   // row_bcast:31, rows 2 and 3
  return x;
}

// Where the kept elements of a part go: what the lanes in front keep of the same slot, two slots to a word, and what
// the wavefront keeps of each.
template <int U>
struct CompactRanks {
  u32 front[U / 2], all[U / 2];
  DISC_DEV int count(const u32 (&kb)[U]) {
    int kept = 0;
#pragma unroll
    for (int h = 0; h < U / 2; ++h) {
      const u32 own = (u32)__builtin_popcount(kb[2 * h]) | (u32)__builtin_popcount(kb[2 * h + 1]) << 16;
      const u32 upto = wave_scan(own);
      front[h] = upto - own;
      all[h] = (u32)__builtin_amdgcn_readlane((int)upto, 63);
      kept += (int)(all[h] & 0xffff) + (int)(all[h] >> 16);
    }
    return kept;
  }
  // kept by the wavefront in slots up to u
  DISC_DEV int upto(int u) const {
    int kept = 0;
#pragma unroll
    for (int k = 0; k < U; ++k) kept += k < u ? (int)(k % 2 ? all[k / 2] >> 16 : all[k / 2] & 0xffff) : 0;
    return kept;
  }
  // kept in front of the lane's slots, in this part; returns what the part keeps
  DISC_DEV int before(int (&b)[U]) const {
    static_assert(U % 2 == 0, "two slots to a word");
    int kept = 0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      b[u] = kept + (int)(u % 2 ? front[u / 2] >> 16 : front[u / 2] & 0xffff);
      kept += (int)(u % 2 ? all[u / 2] >> 16 : all[u / 2] & 0xffff);
    }
    return kept;
  }
};

// Stores the ranks of a wavefront's part of a tile; `pos` = number of elements kept in front of it.
template <bool WHOLE, bool NT, class Pat, int V, int U>
DISC_DEV void compact_store_ranks(const typename Pat::Args& A, i64 w0, const u32 (&kb)[U], const int (&before)[U], i64 pos) {
  if constexpr (Pat::HAS_RANK) {
    const int lane = opaque_lane();
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const unsigned at = (unsigned)((u * 64 + lane) * V);
      i64 rank[V];
      int r = before[u] - 1;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        r += (int)((kb[u] >> e) & 1);
        rank[e] = pos + r;
      }
      const i64 rem = A.inner - (w0 + at);
      if constexpr (WHOLE) Pat::template rank_store<V, NT>(A, w0, at, rank, EvenSpan::upto(V));
      else if (rem > 0) Pat::template rank_store<V, NT>(A, w0, at, rank, Span::upto(rem < (i64)V ? (int)rem : V));
    }
  }
}
// The kept values too; returns `pos` with the part's own added.  `stage`: (64 * V * COMPACT_STRETCH + 64) * COMPACT_BYTES
// bytes of LDS of the wavefront's own.
template <bool WHOLE, bool NT, class Pat, int V, int U>
DISC_DEV i64 compact_emit(const typename Pat::Args& A, i64 w0, const typename Pat::template OutSlot<V> (&o)[U],
                          const u32 (&kb)[U], const CompactRanks<U>& ranks, i64 pos, char* stage) {
  int before[U];
  const int kept = ranks.before(before);
  compact_store_ranks<WHOLE, NT, Pat, V, U>(A, w0, kb, before, pos);
  Pat::template compact_put<V, NT, U>(A, o, kb, ranks, before, pos, stage);
  return pos + kept;
}

// A tile's part of a wavefront, first the count and later the stores (short inputs).
template <bool NT, class Pat, int V, int U>
struct CompactPart {
  typename Pat::template OutSlot<V> o[U];
  u32 kb[U];
  CompactRanks<U> ranks;
  i64 w0;
  bool whole;
  DISC_DEV int count(const typename Pat::Args& A, i64 tile) {
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    w0 = (tile * kCompactWaves + wave) * (64 * U * V);
    whole = w0 + 64 * U * V <= A.inner;
    typename Pat::template Slot<V> slot[U];
    if (whole) {
      compact_load<true, Pat, V, U>(A, w0, slot);
      compact_eval<true, Pat, V, U>(A, w0, slot, o, kb);
    } else {
      compact_load<false, Pat, V, U>(A, w0, slot);
      compact_eval<false, Pat, V, U>(A, w0, slot, o, kb);
    }
    return ranks.count(kb);
  }
  DISC_DEV void store(const typename Pat::Args& A, i64 pos, char* stage) {
    if (whole) compact_emit<true, NT, Pat, V, U>(A, w0, o, kb, ranks, pos, stage);
    else compact_emit<false, NT, Pat, V, U>(A, w0, o, kb, ranks, pos, stage);
  }
};
DISC_DEV i64 wave_scalar(i64 x) {
  return ((i64)__builtin_amdgcn_readfirstlane((int)(x >> 32)) << 32) | (u32)__builtin_amdgcn_readfirstlane((int)x);
}

// LDS written by lanes of a wavefront and read by other lanes of the same one: the accesses stay in
// program order (one wavefront's LDS operations complete in order)
DISC_DEV void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The kept elements of a wavefront's part, collected in LDS and stored as one contiguous stretch at dst + pos, by
// pieces of 64 elements that start where dst does: one piece per part is written by two parts, not one per slot.
// (Stored straight from the lanes, a kept element here and there, every store instruction covers the same few cache
// lines once more.)  S slots at a time: all four, or as many as 8 KB of a wavefront hold (8-byte values of two-byte operands took 68 KB of
// a block; the registers leave two blocks on a CU either way, 33555445 of them 80.7 us / 80.8, 300007 8.7 / 8.5).
template <int V, bool NT, int U, int S, class T, class GET>
DISC_DEV void compact_put_elems(T* __restrict__ dst, i64 pos, const u32 (&kb)[U], const CompactRanks<U>& ranks, const int (&before)[U], char* stage, GET get) {
  T* q = reinterpret_cast<T*>(stage);
  const int lane = (int)threadIdx.x & 63;
#pragma unroll
  for (int s = 0; s < U; s += S) {
    const int first = ranks.upto(s), kept = ranks.upto(s + S) - first;
    const int h = (int)(pos + first) & 63;
    wave_lds_sync();
#pragma unroll
    for (int u = s; u < s + S; ++u) {
      int r = h + before[u] - first;
#pragma unroll
      for (int e = 0; e < V; ++e) {
        if ((kb[u] >> e) & 1) q[r++] = get(u, e);
      }
    }
    wave_lds_sync();
    T* to = dst + (pos + first - h);
    for (int i = lane; i < h + kept; i += 64) {
      if (i >= h) {
        if constexpr (NT) __builtin_nontemporal_store(q[i], to + i);
        else to[i] = q[i];
      }
    }
  }
}

// The two halves of it, for values that wait in LDS until their place is known.
template <int V, int U, class T, class GET>
DISC_DEV void compact_hold_elems(const u32 (&kb)[U], const int (&before)[U], char* stage, GET get) {
  T* q = reinterpret_cast<T*>(stage);
  wave_lds_sync();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    int r = before[u];
#pragma unroll
    for (int e = 0; e < V; ++e) {
      if ((kb[u] >> e) & 1) q[r++] = get(u, e);
    }
  }
}
template <bool NT, class T>
DISC_DEV void compact_flush_elems(T* __restrict__ dst, i64 pos, int kept, const char* stage) {
  const T* q = reinterpret_cast<const T*>(stage);
  const int lane = (int)threadIdx.x & 63;
  const int h = (int)pos & 63;
  wave_lds_sync();
  T* to = dst + pos;
  for (int i = lane - h; i < kept; i += 64) {
    if (i >= 0) {
      if constexpr (NT) __builtin_nontemporal_store(q[i], to + i);
      else to[i] = q[i];
    }
  }
}

// Longer inputs: the parts of a launch dealt out to its wavefronts in contiguous runs of A.aux1 or, the first A.aux3
// of them, one more; f(part, its slots) for the whole ones, the next one loaded before the current one is used.  Returns
// the part behind the run's whole ones.  (Contiguous, because the kept values of neighbouring parts share a line: dealt out
// one by one, sorted i32 keys, 10^7 25.4 us against 24.1, 2^21 10.5 / 8.7.)
template <class Pat, int V, int U, class F>
DISC_DEV i64 compact_run(const typename Pat::Args& A, i64 p, i64 end, typename Pat::template Slot<V> (&slot)[U], F f) {
  for (; p < end; ++p) {
    typename Pat::template Slot<V> next[U];
    if (p + 1 < end) compact_load<true, Pat, V, U>(A, (p + 1) * (64 * U * V), next);
    asm volatile("" ::: "memory");          // these loads before what is done with the current part
    f(p, slot);
#pragma unroll
    for (int u = 0; u < U; ++u) slot[u] = next[u];
  }
  return p;
}
struct CompactRange {
  i64 first, last;                          // the wavefront's whole parts
  bool ragged;                              // the last part of the tensor is not whole, and the wavefront's
};
template <class Pat, int V, int U>
DISC_DEV CompactRange compact_range(const typename Pat::Args& A) {
  const i64 w = (i64)blockIdx.x * kCompactWaves + __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const i64 whole = A.inner / (64 * U * V);
  CompactRange r;
  r.first = w * A.aux1 + (w < A.aux3 ? w : A.aux3);
  const i64 end = r.first + A.aux1 + (w < A.aux3 ? 1 : 0);
  r.ragged = whole >= r.first && whole < end && whole * (64 * U * V) < A.inner;
  r.last = end < whole ? end : whole;
  return r;
}

// A.aux2 = 0: A.aux0 tiles, one to a block, whose counts go to the workspace as 8 bytes each; otherwise A.aux0
// blocks, a run of parts and four bytes to a wavefront.
template <class Pat, int V>
DISC_DEV void compact_count_body(const typename Pat::Args& A) {
  constexpr int U = Pat::COMPACT_SLOTS;
  const int wave = (int)threadIdx.x >> 6;
  if (A.aux2) {
    const CompactRange r = compact_range<Pat, V, U>(A);
    typename Pat::template Slot<V> slot[U];
    int cnt = 0;
    if (r.first < r.last) compact_load<true, Pat, V, U>(A, r.first * (64 * U * V), slot);
    compact_run<Pat, V, U>(A, r.first, r.last, slot, [&](i64 p, const typename Pat::template Slot<V> (&s)[U]) {
      typename Pat::template OutSlot<V> o[U];
      u32 kb[U];
      compact_eval<true, Pat, V, U>(A, p * (64 * U * V), s, o, kb);
      CompactRanks<U> ranks;
      cnt += ranks.count(kb);
    });
    if (r.ragged) {
      const i64 w0 = A.inner / (64 * U * V) * (64 * U * V);
      typename Pat::template OutSlot<V> o[U];
      u32 kb[U];
      compact_load<false, Pat, V, U>(A, w0, slot);
      compact_eval<false, Pat, V, U>(A, w0, slot, o, kb);
      CompactRanks<U> ranks;
      cnt += ranks.count(kb);
    }
    if (((int)threadIdx.x & 63) == 0) reinterpret_cast<int*>(A.ws0)[(i64)blockIdx.x * kCompactWaves + wave] = cnt;
    return;
  }
  __shared__ i64 wsum[kCompactWaves];
  for (i64 c = blockIdx.x; c < A.aux0; c += gridDim.x) {
    CompactPart<false, Pat, V, U> part;
    const int cnt = part.count(A, c);
    if (((int)threadIdx.x & 63) == 0) wsum[wave] = cnt;
    __syncthreads();
    if (threadIdx.x == 0) reinterpret_cast<i64*>(A.ws0)[c] = wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
  }
}

// one block of 1024 threads: exclusive scan of the A.aux0 block counts, in place
template <class Pat>
DISC_DEV void compact_scan_body(const typename Pat::Args& A) {
  __shared__ i64 part[1024];
  i64* counts = reinterpret_cast<i64*>(A.ws0);
  const i64 nb = A.aux0;
  const int nt = (int)blockDim.x, tid = (int)threadIdx.x;
  const i64 per = (nb + nt - 1) / nt;
  const i64 lo = (i64)tid * per, hi = lo + per < nb ? lo + per : nb;
  i64 sum = 0;
  for (i64 i = lo; i < hi; ++i) sum += counts[i];
  part[tid] = sum;
  __syncthreads();
  for (int d = 1; d < nt; d <<= 1) {          // inclusive scan of the per-thread sums
    const i64 t = tid >= d ? part[tid - d] : 0;
    __syncthreads();
    part[tid] += t;
    __syncthreads();
  }
  i64 run = part[tid] - sum;                   // exclusive prefix of this thread's stretch
  for (i64 i = lo; i < hi; ++i) {
    const i64 c = counts[i];
    counts[i] = run;
    run += c;
  }
  if (tid == nt - 1) Pat::count_store(A, part[nt - 1]);
}

// sum of x over the 256 threads of a block, in every thread
DISC_DEV i64 compact_block_sum(i64 x, i64 (&cell)[kCompactWaves]) {
  x += lane_xchg<1>(x);
  x += lane_xchg<2>(x);
  x += lane_xchg<4>(x);
  x += lane_xchg<8>(x);
  x += lane_xchg<16>(x);
  x += lane_xchg<32>(x);
  if (((int)threadIdx.x & 63) == 0) cell[threadIdx.x >> 6] = x;
  __syncthreads();
  x = cell[0] + cell[1] + cell[2] + cell[3];
  __syncthreads();
  return x;
}

// A.aux2: see compact_count_body.  NT: non-temporal stores, for launches whose results do not fit the memory-side cache
// anyway.  With plain stores the results of one call sit there dirty, and the count launch of the next call, which only
// reads, first has to push them out to memory.  Bound by latency up to some 10^6 elements and by memory above; sorted i32
// keys, a quarter distinct, a slot's kept values at a time, blocks of whole tiles and a second wide load for the element in
// front / as it is: 300007 8.4 us / 8.0, 2 x 10^6 9.2 / 8.6, 6 x 10^6 15.7 / 13.2, 20007 (three launches) 11.8 / 11.3.
template <class Pat, int V, bool NT = false>
DISC_DEV void compact_scatter_body(const typename Pat::Args& A) {
  constexpr int U = Pat::COMPACT_SLOTS;
  __shared__ i64 cell[kCompactWaves];
  __shared__ int wsum[kCompactWaves];
  __shared__ __attribute__((aligned(16))) char stage[kCompactWaves][(64 * V * Pat::COMPACT_STRETCH + 64) * Pat::COMPACT_BYTES + 16];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  if (A.aux2) {
    const CompactRange r = compact_range<Pat, V, U>(A);
    typename Pat::template Slot<V> slot[U];
    if (r.first < r.last) compact_load<true, Pat, V, U>(A, r.first * (64 * U * V), slot);
    typedef int int4v __attribute__((ext_vector_type(4)));
    const int4v* counts = reinterpret_cast<const int4v*>(A.ws0);
    i64 x = 0;
    for (int i = (int)threadIdx.x; i < (int)blockIdx.x; i += 256) x += (i64)counts[i][0] + counts[i][1] + counts[i][2] + counts[i][3];
    const int4v own = counts[blockIdx.x];
    i64 pos = compact_block_sum(x, cell);
#pragma unroll
    for (int w = 0; w < kCompactWaves; ++w) pos += w < wave ? own[w] : 0;
    pos = wave_scalar(pos);
    compact_run<Pat, V, U>(A, r.first, r.last, slot, [&](i64 p, const typename Pat::template Slot<V> (&s)[U]) {
      typename Pat::template OutSlot<V> o[U];
      u32 kb[U];
      compact_eval<true, Pat, V, U>(A, p * (64 * U * V), s, o, kb);
      CompactRanks<U> ranks;
      ranks.count(kb);
      pos = compact_emit<true, NT, Pat, V, U>(A, p * (64 * U * V), o, kb, ranks, pos, stage[wave]);
    });
    if (r.ragged) {
      const i64 w0 = A.inner / (64 * U * V) * (64 * U * V);
      typename Pat::template OutSlot<V> o[U];
      u32 kb[U];
      compact_load<false, Pat, V, U>(A, w0, slot);
      compact_eval<false, Pat, V, U>(A, w0, slot, o, kb);
      CompactRanks<U> ranks;
      ranks.count(kb);
      pos = compact_emit<false, NT, Pat, V, U>(A, w0, o, kb, ranks, pos, stage[wave]);
    }
    if (blockIdx.x == gridDim.x - 1 && (int)threadIdx.x == 64 * (kCompactWaves - 1)) Pat::count_store(A, pos);
    return;
  }
  const i64* offsets = reinterpret_cast<const i64*>(A.ws0);
  for (i64 c = blockIdx.x; c < A.aux0; c += gridDim.x) {
    const i64 pos = wave_scalar(offsets[c]);
    CompactPart<NT, Pat, V, U> part;
    const int cnt = part.count(A, c);
    if (((int)threadIdx.x & 63) == 0) wsum[wave] = cnt;
    __syncthreads();
    int before = 0;
#pragma unroll
    for (int w = 0; w < kCompactWaves; ++w) before += w < wave ? wsum[w] : 0;
    part.store(A, pos + __builtin_amdgcn_readfirstlane(before), stage[wave]);
    __syncthreads();
  }
}

// Large inputs in one pass: A.aux0 tiles dealt out to the blocks one by one (gridDim.x <= 1024, all resident), a part of a
// tile to a wavefront.  A block publishes what a tile keeps, plus one, in a cell of the workspace (zero before the launch) two
// iterations before it stores that tile, and the place of a tile is that of the block's tile before it plus the cells
// in between, one per block: no chain of look-backs, one exchange per iteration, with a whole iteration and more
// between publishing and use.  Until then the tile's flags are a word per lane and its kept values wait in LDS.
// The result does not depend on a wait: a cell that has not come after A.aux2 looks -- its block may not be resident -- is
// counted by the wavefront that misses it, from the inputs, and published for the others: one at a time, each wavefront
// another one, and all are looked at again after it.  A cell is one
// 4-byte word, written and read whole at device scope; nothing else passes between blocks.
// Bound by memory: 2^25 sorted i32 keys, a quarter distinct, 302 MB in 56 us (5.4 TB/s; a plain copy of as much moves
// 5.7) + 4.4 to clear the cells; two launches that read them twice 78.7 us.  2^25 i64 121 / 92, 1.2 x 10^7 i32 29.9 / 21.1.
// Published one iteration ahead, the looks ended up behind the stores of the iteration before: 67.5.  (Two blocks a CU
// 75, three 60.9, four 60.4; numbers in between load the CUs unevenly and the fuller ones set the pace, 3.5 to a
// CU 79; non-temporal loads 61.0.)
// A.aux3: the kept values non-temporal too (the ranks are in any case): from some 150 MiB of operands and results on (i32, plain / so:
// 12 x 10^6 21.1 / 23.0, 16 x 10^6 25.3 / 28.0, 22 x 10^6 38.9 / 37.9; i64 12 x 10^6 37.1 / 34.5); ranks plain as well 28.4 at 12 x 10^6.
template <class Pat, int V, int U>
DISC_DEV int compact_recount(const typename Pat::Args& A, i64 tile) {
  int cnt = 0;
#pragma unroll 1
  for (int k = 0; k < kCompactWaves * U; ++k) {               // (a slot at a time: few registers beside those in use)
    const i64 w0 = (tile * (kCompactWaves * U) + k) * (64 * V);
    typename Pat::template Slot<V> s[1];
    typename Pat::template OutSlot<V> o[1];
    u32 kb[1];
    compact_load<false, Pat, V, 1>(A, w0, s);
    compact_eval<false, Pat, V, 1>(A, w0, s, o, kb);
    cnt += __builtin_amdgcn_readlane((int)wave_scan((u32)__builtin_popcount(kb[0])), 63);
  }
  return cnt;
}
template <class Pat, int V>
DISC_DEV void compact_chain_body(const typename Pat::Args& A) {
  constexpr int U = Pat::COMPACT_SLOTS, E = 64 * U * V, C = 4;       // C cells of a window to a lane
  static_assert(U * V <= 32, "the kept flags of a part in one word");
  __shared__ __attribute__((aligned(16))) char stage[2][kCompactWaves][E * Pat::COMPACT_ALL_BYTES + 16];
  __shared__ int kept[2][kCompactWaves], gap[2][kCompactWaves];
  __shared__ u32 arrived[2];
  u32* cells = reinterpret_cast<u32*>(A.ws0);
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = (int)threadIdx.x & 63;
  if (threadIdx.x < 2) arrived[threadIdx.x] = 0;
  __syncthreads();
  auto first = [&](i64 t) { return (t * kCompactWaves + wave) * (i64)E; };
  // a part of the block's tile t whose place is not known yet
  struct Waiting {
    u32 flags;
    CompactRanks<U> ranks;
    int before;                             // what the wavefronts in front keep of the tile
  };
  Waiting now, next, eval;                  // of tiles t, t + grid, t + 2 grid
  typename Pat::template Slot<V> slot[U];
  u32 win[C];
  // the window of a tile: cells [lo, lo + n)
  i64 lo = 0;
  int n = 0;
  auto look = [&](int c) {
    return c * 256 + (int)threadIdx.x < n ? __hip_atomic_load(cells + lo + c * 256 + (int)threadIdx.x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 1u;
  };
  const i64 G = gridDim.x;
  i64 t = blockIdx.x - 2 * G, run = 0;      // (negative: no tile yet)
  i64 patience = A.aux2;                    // looks at a window before a cell is counted here; few after one that came to that
  if (first(blockIdx.x) + E <= A.inner) compact_load<true, Pat, V, U>(A, first(blockIdx.x), slot);
  for (int buf = 0;; buf ^= 1, t += G) {
    // two tiles ahead: count, publish, load the one behind it
    const i64 t2 = t + 2 * G, w2 = first(t2);
    typename Pat::template OutSlot<V> o[U];
    u32 kb[U];
    if (t2 < A.aux0) {
      if (w2 + E <= A.inner) {
        compact_eval<true, Pat, V, U>(A, w2, slot, o, kb);
      } else {
        compact_load<false, Pat, V, U>(A, w2, slot);
        compact_eval<false, Pat, V, U>(A, w2, slot, o, kb);
      }
      const int cnt = eval.ranks.count(kb);
      if (lane == 0) {
        kept[buf][wave] = cnt;
        // (a tile has less than 2^24 elements: its count and the wavefronts that have added theirs in one word)
        const u32 before = __hip_atomic_fetch_add(&arrived[buf], (1u << 24) + (u32)cnt, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (before >> 24 == kCompactWaves - 1) {
          __hip_atomic_store(cells + t2, (before & 0xffffff) + (u32)cnt + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          arrived[buf] = 0;
        }
      }
      eval.flags = 0;
#pragma unroll
      for (int u = 0; u < U; ++u) eval.flags |= kb[u] << (u * V);
      if (first(t2 + G) + E <= A.inner) compact_load<true, Pat, V, U>(A, first(t2 + G), slot);
    }
    // this tile's window
    if (t >= 0) {
      bool counted = false;
      for (i64 looks = 0;; ++looks) {
        u64 gone[C], any = 0;
#pragma unroll
        for (int c = 0; c < C; ++c) any |= gone[c] = __builtin_amdgcn_ballot_w64(win[c] == 0);
        if (any == 0) break;
        if (looks < patience) {
          __builtin_amdgcn_s_sleep(2);
        } else {
          // one of the wavefront's missing cells, another one in every block, which then finds those that the others have counted
          counted = true;
          const int turn = (int)(blockIdx.x * 2654435761u >> 26);
          int cell = -1;
#pragma unroll
          for (int k = C - 1; k >= 0; --k) {
            const int c = (k + (int)blockIdx.x) & (C - 1);
            u64 m = gone[0];
#pragma unroll
            for (int i = 1; i < C; ++i) m = c == i ? gone[i] : m;
            m = m >> turn | m << (-turn & 63);
            if (m != 0) cell = c * 64 + (((int)__builtin_ctzll(m) + turn) & 63);
          }
          const i64 tile = lo + (cell >> 6) * 256 + wave * 64 + (cell & 63);
          const u32 got = (u32)compact_recount<Pat, V, U>(A, tile) + 1;
          if (lane == (cell & 63)) __hip_atomic_store(cells + tile, got, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
          for (int c = 0; c < C; ++c)
            if (c == cell >> 6 && lane == (cell & 63)) win[c] = got;
        }
#pragma unroll
        for (int c = 0; c < C; ++c)
          if (win[c] == 0) win[c] = look(c);
      }
      patience = !counted ? A.aux2 : A.aux2 < 8 ? A.aux2 : 8;
      u32 sum = 0;
#pragma unroll
      for (int c = 0; c < C; ++c) sum += win[c] - 1;
      sum = wave_scan(sum);
      if (lane == 63) gap[buf][wave] = (int)sum;
    }
    __syncthreads();
    if (t2 < A.aux0) {
      int ahead = 0;
#pragma unroll
      for (int w = 0; w < kCompactWaves; ++w) ahead += w < wave ? kept[buf][w] : 0;
      eval.before = __builtin_amdgcn_readfirstlane(ahead);
    }
    if (t + G >= 0 && t + G < A.aux0) {
      lo = t >= 0 ? t : 0;
      n = t >= 0 ? (int)G : (int)blockIdx.x;
#pragma unroll
      for (int c = 0; c < C; ++c) win[c] = look(c);
      asm volatile("" ::: "memory");        // (looked at in the next iteration: before the stores)
    }
    if (t >= 0) {
      int all = 0;
#pragma unroll
      for (int w = 0; w < kCompactWaves; ++w) all += gap[buf][w];
      run += __builtin_amdgcn_readfirstlane(all);
      const i64 at = wave_scalar(run + now.before), w0 = first(t);
      int before[U];
      const int cnt = now.ranks.before(before);
      u32 kb0[U];
#pragma unroll
      for (int u = 0; u < U; ++u) kb0[u] = (now.flags >> (u * V)) & ((1u << V) - 1);
      if (w0 + E <= A.inner) compact_store_ranks<true, true, Pat, V, U>(A, w0, kb0, before, at);
      else compact_store_ranks<false, true, Pat, V, U>(A, w0, kb0, before, at);
      if (A.aux3) Pat::template compact_flush<true>(A, cnt, at, stage[buf][wave]);
      else Pat::template compact_flush<false>(A, cnt, at, stage[buf][wave]);
      if (t == A.aux0 - 1 && wave == kCompactWaves - 1 && lane == 0) Pat::count_store(A, at + cnt);
      if (t + G >= A.aux0) break;
    }
    if (t2 < A.aux0) {
      int before[U];
      eval.ranks.before(before);
      Pat::template compact_hold<V, U>(o, kb, before, stage[buf][wave]);
    }
    now = next;
    next = eval;
  }
}
template <class Pat>
DISC_DEV void compact_clear_body(const typename Pat::Args& A) {
  const i64 i = (i64)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < A.aux0) reinterpret_cast<u32*>(A.ws0)[i] = 0;
}

}  // namespace disc
