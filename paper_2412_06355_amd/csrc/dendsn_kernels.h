// DendSN layer scan kernels for gfx950 (CDNA4, wave64).
//
// One kernel per direction.  A neuron's B branches (P = B KC compartments) are
// held by L adjacent lanes of one wavefront, BL = B / L whole branches per lane,
// so one time step of X for a wave is one contiguous, fully coalesced stretch of
// [T, N, P] memory (or, in the channel-major layout, KC BL accesses that are each
// contiguous across the wave).  The dendritic states stay in registers across
// the time loop; the only cross-lane traffic is the branch-to-soma sum Z,
// reduced with DPP inside the L-lane group, and every lane of the group then
// runs the soma redundantly (no broadcast).
//
// A block owns a tile of positions of one sample (see TileMode) and loops over a
// group of batch items, so per-channel parameters are loaded once per lane and
// parameter-gradient partials are summed in registers across those items.
//
// The forward kernel and the backward kernel's recompute of the forward call
// the same inline step functions, so (compiled with -ffp-contract=off, explicit
// fmaf and the raw v_exp_f32) they reproduce bit-identical states and spikes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dendsn_plan.h"

namespace dendsn {

typedef uint16_t bf16_t;  // bf16 storage

// Kernel variant V: bit 0 = Mexican-hat activation (else identity), bit 1 =
// residual dendrite (Z also receives the mean synaptic input of the neuron),
// bits 2-3 = log2 of the compartments per branch KC (1, 2 or 4), bit 4 =
// channel-major X / grad_x ([T, batch, C, P, S]: a neuron's compartments S
// elements apart), bit 6 = Stateless Dendrite (a compartment's state is its
// input of the step: no leak, no dendritic state across steps or checkpoints,
// no adjoint recurrence and no alpha gradient).  A lane holds BL branches,
// i.e. E = BL * KC compartments of its neuron.
template <int V> constexpr bool kMH = (V & 1) != 0;
template <int V> constexpr bool kRes = (V & 2) != 0;
template <int V> constexpr int kKC = 1 << ((V >> 2) & 3);
template <int V> constexpr bool kCM = (V & 16) != 0;
template <int V> constexpr int kSG = (V >> 5) & 1;  // backward only: dendsn_sg surrogate
template <int V> constexpr bool kSL = (V & 64) != 0;
// Forward over bf16 rows without the residual dendrite: the branch gate is applied
// while the raw rows are widened (the residual sums every compartment's input,
// gated or not).  Measured: forward 2-2.5 % faster; the backward kept its
// per-step select (there the change was neutral to 1.4 % slower).
template <typename IO, int V> constexpr bool kGateIn = sizeof(IO) == 2 && !kRes<V>;
// The branch sum takes a lane's branches in fused pairs (one multiply and one
// fused multiply-add per pair) when a lane holds at least two.  Every split of
// a neuron that the two directions and the two layouts use holds whole pairs in
// a lane whenever one of them does, except with four compartments per branch
// (the channel-major backward then holds one branch per lane, its forward two),
// which keeps the plain tree: the branch sum stays one tree over the fused
// leaves, and the directions and layouts agree bit for bit.
template <int V, int BL> constexpr bool kFuse = BL >= 2 && kKC<V> < 4;

// -(1/2) log2(e): exp(-u^2/2) = exp2(u^2 * kNegHalfLog2e)
constexpr float kNegHalfLog2e = -0.721347520444481703680f;
constexpr float kLog2e = 1.442695040888963407360f;
constexpr float kPi = 3.141592653589793238463f;

// ---------------------------------------------------------------------------
// Storage conversions
// ---------------------------------------------------------------------------
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Two floats -> two bf16 in one dword, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  f32x2_t f = {a, b};
  bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(uint32_t, h);
}
__device__ __forceinline__ bf16_t to_bf16(float a) {
  return __builtin_bit_cast(bf16_t, static_cast<__bf16>(a));
}

// Streaming loads are non-temporal: X, grad_spikes and checkpoints are read
// once per pass, so they should not displace anything in the caches.  A lane
// row of more than 16 bytes takes several loads that each touch every cache
// line of the wave's stretch; those use the default policy, so that the later
// loads of a row find the lines the first brought in (non-temporal, a copy of
// 40-byte lane pieces ran at 1.9 TB/s against 4.6-4.9 with the default policy).
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));

// The policy is a template parameter: as a runtime flag, callers of one
// instance with both values let the compiler merge its two loads of the same
// address into one plain load, which dropped the non-temporal hint for every
// caller (the fp32 CIFAR forward, 16-byte rows, ran 14 % slower once a wide
// fp32 mapping shared its 16-byte load instance).
template <bool kCached, typename T>
__device__ __forceinline__ T stream_load(const T* p);

template <int BL>
__device__ __forceinline__ void store_vec(float* __restrict__ p, const float (&v)[BL]) {
  if constexpr (BL % 4 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 4; ++i)
      reinterpret_cast<float4*>(p)[i] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
  } else if constexpr (BL % 2 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 2; ++i) reinterpret_cast<float2*>(p)[i] = make_float2(v[2 * i], v[2 * i + 1]);
  } else {
#pragma unroll
    for (int i = 0; i < BL; ++i) p[i] = v[i];
  }
}

// Address = wave-uniform base (scalar registers) + 32-bit per-lane byte offset.
template <typename P>
__device__ __forceinline__ P* at(P* base, uint32_t off) {
  return reinterpret_cast<P*>(reinterpret_cast<char*>(base) + off);
}
template <typename P>
__device__ __forceinline__ const P* at(const P* base, uint32_t off) {
  return reinterpret_cast<const P*>(reinterpret_cast<const char*>(base) + off);
}


// ---------------------------------------------------------------------------
// Streamed rows through buffer resources: the row base is wave-uniform (scalar
// registers, the resource), the lane's part a 32-bit offset, and a further
// uniform part rides in the instruction's scalar offset, so no per-lane 64-bit
// address arithmetic is spent on the backward's X, grad_spikes and grad_x rows.  Accesses
// are non-temporal (each byte is touched once per pass).
// ---------------------------------------------------------------------------
typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr int kAuxNT = 2;  // cache policy: non-temporal (streaming)
// s_waitcnt vmcnt(0), other counters untouched: every vector memory access of
// the wave has completed.
constexpr int kWaitVmem = 0x0F70;


__device__ __forceinline__ rsrc_t make_rsrc(const void* base) {
  // raw buffer, byte range 4 GiB - 1 (every lane offset is a uint32 below it)
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, -1, 0x00020000);
}

// A raw buffer of `bytes` bytes: loads at or past the end return 0 without
// touching memory (bytes = 0 makes every load a zero).
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, int(bytes), 0x00020000);
}

// A wave-uniform value the compiler cannot prove uniform (a select on loop
// state inside the lanes' active region) made explicit: as part of a buffer
// resource it would otherwise be fed to the load through a per-lane loop over
// distinct values, whose first wait drains every request in flight.  The empty
// asm keeps the value in a scalar register: without it a select was folded
// through the readfirstlane back into a vector register.
__device__ __forceinline__ uint32_t uniform_u32(uint32_t v) {
  uint32_t r = __builtin_amdgcn_readfirstlane(v);
#ifdef __HIP_DEVICE_COMPILE__
  asm("" : "+s"(r));
#endif
  return r;
}

template <typename P>
__device__ __forceinline__ const P* uniform_ptr(const P* p) {  // the same for a base address
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint64_t lo = uniform_u32(uint32_t(u)), hi = uniform_u32(uint32_t(u >> 32));
  return reinterpret_cast<const P*>(hi << 32 | lo);
}

// A lane's BL adjacent floats (checkpointed states), cached as in bload_raw.
template <int BL>
__device__ __forceinline__ void bload_vec(rsrc_t r, uint32_t off, float (&v)[BL]) {
  constexpr int kAuxNT = BL * 4 > 16 ? 0 : dendsn::kAuxNT;
  if constexpr (BL % 4 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 4; ++i) {
      const u32x4_t q = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16u * i, 0, kAuxNT);
      v[4 * i] = __uint_as_float(q.x); v[4 * i + 1] = __uint_as_float(q.y);
      v[4 * i + 2] = __uint_as_float(q.z); v[4 * i + 3] = __uint_as_float(q.w);
    }
  } else if constexpr (BL % 2 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 2; ++i) {
      const u32x2_t q = __builtin_amdgcn_raw_buffer_load_b64(r, off + 8u * i, 0, kAuxNT);
      v[2 * i] = __uint_as_float(q.x); v[2 * i + 1] = __uint_as_float(q.y);
    }
  } else {
#pragma unroll
    for (int i = 0; i < BL; ++i) v[i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off + 4u * i, 0, kAuxNT));
  }
}

template <int BL, int AUX = kAuxNT>
__device__ __forceinline__ void bstore_vec(rsrc_t r, uint32_t off, const float (&v)[BL], float*) {
  if constexpr (BL % 4 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 4; ++i) {
      const u32x4_t q = {__float_as_uint(v[4 * i]), __float_as_uint(v[4 * i + 1]), __float_as_uint(v[4 * i + 2]),
                         __float_as_uint(v[4 * i + 3])};
      __builtin_amdgcn_raw_buffer_store_b128(q, r, off + 16u * i, 0, AUX);
    }
  } else if constexpr (BL % 2 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 2; ++i) {
      const u32x2_t q = {__float_as_uint(v[2 * i]), __float_as_uint(v[2 * i + 1])};
      __builtin_amdgcn_raw_buffer_store_b64(q, r, off + 8u * i, 0, AUX);
    }
  } else {
#pragma unroll
    for (int i = 0; i < BL; ++i) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v[i]), r, off + 4u * i, 0, AUX);
  }
}

template <int BL, int AUX = kAuxNT>
__device__ __forceinline__ void bstore_vec(rsrc_t r, uint32_t off, const float (&v)[BL], bf16_t*) {
  if constexpr (BL % 8 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 8; ++i) {
      const u32x4_t q = {pack_bf16x2(v[8 * i + 0], v[8 * i + 1]), pack_bf16x2(v[8 * i + 2], v[8 * i + 3]),
                         pack_bf16x2(v[8 * i + 4], v[8 * i + 5]), pack_bf16x2(v[8 * i + 6], v[8 * i + 7])};
      __builtin_amdgcn_raw_buffer_store_b128(q, r, off + 16u * i, 0, AUX);
    }
  } else if constexpr (BL % 4 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 4; ++i) {
      const u32x2_t q = {pack_bf16x2(v[4 * i + 0], v[4 * i + 1]), pack_bf16x2(v[4 * i + 2], v[4 * i + 3])};
      __builtin_amdgcn_raw_buffer_store_b64(q, r, off + 8u * i, 0, AUX);
    }
  } else if constexpr (BL % 2 == 0) {
#pragma unroll
    for (int i = 0; i < BL / 2; ++i)
      __builtin_amdgcn_raw_buffer_store_b32(pack_bf16x2(v[2 * i], v[2 * i + 1]), r, off + 4u * i, 0, AUX);
  } else {
#pragma unroll
    for (int i = 0; i < BL; ++i) __builtin_amdgcn_raw_buffer_store_b16(to_bf16(v[i]), r, off + 2u * i, 0, AUX);
  }
}

__device__ __forceinline__ void bstore_one(rsrc_t r, uint32_t off, uint32_t soff, float v, float*) {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), r, off, soff, kAuxNT);
}
__device__ __forceinline__ void bstore_one(rsrc_t r, uint32_t off, uint32_t soff, float v, bf16_t*) {
  __builtin_amdgcn_raw_buffer_store_b16(to_bf16(v), r, off, soff, kAuxNT);
}

// A lane's E compartments of grad_x in the row starting at `row`: adjacent (a
// vector access at the lane offset) or, in the channel-major layout, es bytes apart
// (one access each, the uniform i * es in the scalar offset; the lanes of a wave
// hold adjacent positions, so each access is contiguous across the wave).
template <int E, bool CM, typename IO>
__device__ __forceinline__ void store_gx(IO* row, uint32_t off, uint32_t es, const float (&v)[E]) {
  const rsrc_t r = make_rsrc(row);
  if constexpr (CM) {
#pragma unroll
    for (int i = 0; i < E; ++i) bstore_one(r, off, uint32_t(i) * es, v[i], row);
  } else {
    // Non-temporal up to 16 bytes a lane.  A longer row is several stores, each
    // writing every line it touches in pieces; as streaming stores the pieces
    // reached HBM separately (the ten-compartment fp32 rows wrote 32 % more
    // than grad_x, 1 % slower), so those go through L2 as default stores.
    // (Shorter multi-store rows, e.g. 12-byte bf16 ones, ran 1.7 % slower so.)
    constexpr bool streaming = E * sizeof(IO) <= 16;
    bstore_vec<E, streaming ? kAuxNT : 0>(r, off, v, row);
  }
}

// grad_x of one step, staged (see load_pieces): the lane's raw dwords go to the
// wave's LDS buffer and leave as whole 16-byte pieces, consecutive lanes on
// consecutive pieces (non-temporal: whole lines).
template <typename IO, int E>
__device__ __forceinline__ void store_gx_staged(IO* row, uint32_t span, const float (&v)[E], uint32_t* stage) {
  constexpr int W = sizeof(IO) == 4 ? E : E / 2;
  static_assert(sizeof(IO) == 4 || E % 2 == 0, "staged bf16 rows hold element pairs");
  const uint32_t lane = __lane_id();
#pragma unroll
  for (int j = 0; j < W; ++j)
    stage[lane * W + j] = sizeof(IO) == 4 ? __float_as_uint(v[j]) : pack_bf16x2(v[2 * j], v[2 * j + 1 < E ? 2 * j + 1 : 0]);
  __builtin_amdgcn_wave_barrier();
  const rsrc_t r = make_rsrc(row);
#pragma unroll
  for (int i = 0; i < (64 * W + 255) / 256; ++i) {
    const uint32_t d = (uint32_t(i) * 64 + lane) * 4;
    if (i < 64 * W / 256 || lane < (64 * W % 256) / 4)  // whole rounds, then the partial one
      __builtin_amdgcn_raw_buffer_store_b128(*reinterpret_cast<const u32x4_t*>(stage + d), r, span + d * 4, 0, kAuxNT);
  }
  __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Rows in raw form: the dwords the loads return (fp32 elements, bf16 element
// pairs, or one bf16 element in the low half), converted to float where they
// are used, so that the wait for a prefetched row falls at its first use and not
// right after its load.
// ---------------------------------------------------------------------------
template <typename IO, int E, bool CM>
constexpr int kRawW = (sizeof(IO) == 2 && !CM && E % 2 == 0) ? E / 2 : E;  // dwords per row

// Global (address) loads, as the forward issues them (non-temporal, except for
// lane rows of more than 16 bytes, as in bload_raw).
template <bool kCached, typename T>
__device__ __forceinline__ T stream_load(const T* p) {
  if constexpr (kCached) return *p;
  else return __builtin_nontemporal_load(p);
}

template <typename IO, int E, bool CM, int W>
__device__ __forceinline__ void load_raw(const IO* row, uint32_t off, uint32_t es, uint32_t (&w)[W]) {
  constexpr bool dwords = sizeof(IO) == 4 || (!CM && W * 2 == E);  // contiguous whole dwords
  constexpr bool wide = !CM && W * 4 > 16;
  if constexpr (CM) {
#pragma unroll
    for (int i = 0; i < W; ++i) {
      const IO* q = at(row, off + uint32_t(i) * es);
      if constexpr (sizeof(IO) == 4) w[i] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t*>(q));
      else w[i] = uint32_t(__builtin_nontemporal_load(reinterpret_cast<const uint16_t*>(q)));
    }
  } else if constexpr (dwords && W % 4 == 0) {
    const u32x4_t* q = reinterpret_cast<const u32x4_t*>(at(row, off));
#pragma unroll
    for (int i = 0; i < W / 4; ++i) {
      const u32x4_t v = stream_load<wide>(q + i);
      w[4 * i] = v.x; w[4 * i + 1] = v.y; w[4 * i + 2] = v.z; w[4 * i + 3] = v.w;
    }
  } else if constexpr (dwords && W % 2 == 0) {
    const u32x2_t* q = reinterpret_cast<const u32x2_t*>(at(row, off));
#pragma unroll
    for (int i = 0; i < W / 2; ++i) {
      const u32x2_t v = stream_load<wide>(q + i);
      w[2 * i] = v.x; w[2 * i + 1] = v.y;
    }
  } else if constexpr (dwords) {
    const uint32_t* q = reinterpret_cast<const uint32_t*>(at(row, off));
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = stream_load<wide>(q + i);
  } else {
    const uint16_t* q = reinterpret_cast<const uint16_t*>(at(row, off));
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = uint32_t(stream_load<wide>(q + i));
  }
}

// Buffer loads, as the backward issues them.  A lane row of more than 16 bytes
// takes several loads that each touch every cache line of the wave's row; those
// go through the caches with the default policy, so the later loads of a row
// find the lines the first one brought in.
template <typename IO, int E, bool CM, int W>
__device__ __forceinline__ void bload_raw(rsrc_t r, uint32_t off, uint32_t es, uint32_t (&w)[W]) {
  constexpr bool dwords = sizeof(IO) == 4 || (!CM && W * 2 == E);  // contiguous whole dwords
  constexpr int kAuxNT = (!CM && W * 4 > 16) ? 0 : dendsn::kAuxNT;
  if constexpr (CM) {
#pragma unroll
    for (int i = 0; i < W; ++i)
      w[i] = sizeof(IO) == 4 ? __builtin_amdgcn_raw_buffer_load_b32(r, off, uint32_t(i) * es, kAuxNT)
                             : uint32_t(__builtin_amdgcn_raw_buffer_load_b16(r, off, uint32_t(i) * es, kAuxNT));
  } else if constexpr (dwords && W % 4 == 0) {
#pragma unroll
    for (int i = 0; i < W / 4; ++i) {
      const u32x4_t q = __builtin_amdgcn_raw_buffer_load_b128(r, off + 16u * i, 0, kAuxNT);
      w[4 * i] = q.x; w[4 * i + 1] = q.y; w[4 * i + 2] = q.z; w[4 * i + 3] = q.w;
    }
  } else if constexpr (dwords && W % 2 == 0) {
#pragma unroll
    for (int i = 0; i < W / 2; ++i) {
      const u32x2_t q = __builtin_amdgcn_raw_buffer_load_b64(r, off + 8u * i, 0, kAuxNT);
      w[2 * i] = q.x; w[2 * i + 1] = q.y;
    }
  } else if constexpr (dwords) {
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = __builtin_amdgcn_raw_buffer_load_b32(r, off + 4u * i, 0, kAuxNT);
  } else {
#pragma unroll
    for (int i = 0; i < W; ++i) w[i] = uint32_t(__builtin_amdgcn_raw_buffer_load_b16(r, off + 2u * i, 0, kAuxNT));
  }
}

template <typename IO, int E, int W>
__device__ __forceinline__ void raw_to_float(const uint32_t (&w)[W], float (&v)[E]) {
  if constexpr (sizeof(IO) == 4) {
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = __uint_as_float(w[i]);
  } else if constexpr (W * 2 == E) {
#pragma unroll
    for (int i = 0; i < W; ++i) { v[2 * i] = bf16_lo(w[i]); v[2 * i + 1] = bf16_hi(w[i]); }
  } else {
#pragma unroll
    for (int i = 0; i < E; ++i) v[i] = bf16_lo(w[i]);
  }
}

// v_perm_b32 byte selectors (result byte k <- selector byte k: 0-3 pick a byte
// of the dword, 0x0c gives 0x00): the bf16 in the low or high half widened to
// fp32 (low 16 bits zero), or +0.
constexpr uint32_t kPermLo = 0x01000C0Cu;
constexpr uint32_t kPermHi = 0x03020C0Cu;
constexpr uint32_t kPermZero = 0x0C0C0C0Cu;

// raw_to_float for bf16 rows with the branch gate folded in: one v_perm per
// element widens it, or zeroes it on a gated-off branch (so a gated branch's
// compartments integrate exact zeros and stay at +0 whatever the input holds).
template <int E, int W>
__device__ __forceinline__ void raw_to_float_gated(const uint32_t (&w)[W], const uint32_t (&sel)[E], float (&v)[E]) {
#pragma unroll
  for (int i = 0; i < E; ++i) {
    const uint32_t d = w[W * 2 == E ? i / 2 : i];
    v[i] = __uint_as_float(__builtin_amdgcn_perm(d, d, sel[i]));
  }
}

template <typename IO>
__device__ __forceinline__ float raw_to_float(uint32_t w) {
  return sizeof(IO) == 4 ? __uint_as_float(w) : bf16_lo(w);
}

// ---------------------------------------------------------------------------
// Wide lane rows (more than 16 bytes of a row in one lane: the one-lane
// mappings of neurons with many compartments), staged.  Loaded lane by lane,
// each of a lane's several loads touches every cache line of the wave's
// stretch (a copy of 40-byte lane pieces ran 4.6-4.9 TB/s on MI355X against 5.7
// for 16-byte lanes, a read 5.9 against 6.3).  When the wave's 64 lanes hold one
// contiguous, 16-byte aligned stretch of 64 W dwords (every lane active), the
// wave moves the stretch as whole 16-byte pieces instead, consecutive lanes on
// consecutive pieces, and hands each lane its W dwords through a per-wave LDS
// buffer (ST = true below).
// ---------------------------------------------------------------------------
template <int W> constexpr int kPieces = (64 * W + 255) / 256;  // 16-byte pieces per lane
// Rows staged: a lane's row is more than 16 contiguous bytes that it keeps as
// whole dwords (fp32 elements or bf16 pairs; not the channel-major layout).
template <typename IO, int E, bool CM>
constexpr bool kWideRow = !CM && (sizeof(IO) == 4 || E % 2 == 0) && E * int(sizeof(IO)) > 16;
// dwords a lane keeps of one row: its W dwords, or its pieces when staged
template <int W, bool ST> constexpr int kSlotW = ST ? 4 * kPieces<W> : W;

// The pieces of the wave's stretch at byte `span` of `row` (non-temporal:
// whole lines); a piece past the stretch rereads the stretch's first.
// Round i of a stretch of 64 W dwords: lane l moves dwords 4 (64 i + l) ..
// + 3; every lane takes part in the first 64 W / 256 rounds, lanes below
// kTailLanes in the last, partial one.
template <int W> constexpr int kFullRounds = 64 * W / 256;
template <int W> constexpr uint32_t kTailLanes = (64 * W % 256) / 4;
template <int W>
__device__ __forceinline__ bool in_stretch(int i, uint32_t lane) {
  return i < kFullRounds<W> || lane < kTailLanes<W>;
}

template <typename IO, int W>
__device__ __forceinline__ void load_pieces(const IO* row, uint32_t span, uint32_t (&w)[4 * kPieces<W>]) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (int i = 0; i < kPieces<W>; ++i) {
    const uint32_t d = (uint32_t(i) * 64 + lane) * 4;
    const u32x4_t q = __builtin_nontemporal_load(
        reinterpret_cast<const u32x4_t*>(at(row, span + (in_stretch<W>(i, lane) ? d * 4 : 0u))));
    w[4 * i] = q.x; w[4 * i + 1] = q.y; w[4 * i + 2] = q.z; w[4 * i + 3] = q.w;
  }
}

// The same through a buffer resource (the backward's rows).
template <int W>
__device__ __forceinline__ void bload_pieces(rsrc_t r, uint32_t span, uint32_t (&w)[4 * kPieces<W>]) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (int i = 0; i < kPieces<W>; ++i) {
    const uint32_t d = (uint32_t(i) * 64 + lane) * 4;
    const u32x4_t q = __builtin_amdgcn_raw_buffer_load_b128(r, span + (in_stretch<W>(i, lane) ? d * 4 : 0u), 0, kAuxNT);
    w[4 * i] = q.x; w[4 * i + 1] = q.y; w[4 * i + 2] = q.z; w[4 * i + 3] = q.w;
  }
}

// The lane's W dwords out of the wave's pieces, through the wave's LDS buffer
// `stage` (64 W dwords).  LDS accesses of one wave complete in order.
template <int W>
__device__ __forceinline__ void pieces_to_lane(const uint32_t (&w)[4 * kPieces<W>], uint32_t* stage,
                                               uint32_t (&out)[W]) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (int i = 0; i < kPieces<W>; ++i) {
    const uint32_t d = (uint32_t(i) * 64 + lane) * 4;
    if (in_stretch<W>(i, lane)) *reinterpret_cast<u32x4_t*>(stage + d) = u32x4_t{w[4 * i], w[4 * i + 1], w[4 * i + 2], w[4 * i + 3]};
  }
  __builtin_amdgcn_wave_barrier();
#pragma unroll
  for (int j = 0; j < W; ++j) out[j] = stage[lane * W + j];
  __builtin_amdgcn_wave_barrier();
}

// A row slot (kSlotW dwords) as the lane's W raw dwords.
template <int W, bool ST>
__device__ __forceinline__ void slot_to_lane(const uint32_t (&slot)[kSlotW<W, ST>], uint32_t* stage, uint32_t (&out)[W]) {
  if constexpr (ST) {
    pieces_to_lane<W>(slot, stage, out);
  } else {
#pragma unroll
    for (int j = 0; j < W; ++j) out[j] = slot[j];
  }
}

// The same pieces moved by the memory unit straight into LDS (buffer loads
// with the LDS-DMA form): round i writes the 64 lanes' 16-byte pieces to dwords
// 256 i + 4 lane .. + 3 of `lds`, so the stretch's dword k lands at lds[k] and
// no register holds it in flight.  Lanes past the stretch in the last round
// request nothing, so a row's area is exactly its 64 W dwords.  The wave reads
// the area only after its vector memory counter has drained, and refills it
// only after its reads of it have completed (LDS reads and the DMA's LDS
// writes are not ordered otherwise).
template <int W> constexpr int kDmaDw = 64 * W;
typedef __attribute__((address_space(3))) void lds_void_t;
// s_waitcnt lgkmcnt(0), other counters untouched: every LDS access of the wave
// has completed.
constexpr int kWaitLds = 0xC07F;

// One round: the wave's 64 pieces at byte offsets `off` (per lane) into the 256
// dwords at `lds` (a plain function: the LDS-DMA builtin inside a template
// instantiated by the host compilation pass is rejected there).  Non-temporal,
// like every whole-line stream here (measured on MI355X, stateful P = 10
// backward: 375 -> 370 us alone, 388 -> 351 us back to back with the forward;
// with the default policy the X lines it leaves in the caches only served a
// forward of the same layer launched right after it, as no training step does).
__device__ __forceinline__ void dma_round(rsrc_t r, uint32_t off, uint32_t* lds) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void_t*)lds, 16, off, 0, 0, kAuxNT);
}

template <int W>
__device__ __forceinline__ void dma_pieces(rsrc_t r, uint32_t span, uint32_t* lds) {
  const uint32_t lane = __lane_id();
#pragma unroll
  for (int i = 0; i < kPieces<W>; ++i) {
    const uint32_t d = (uint32_t(i) * 64 + lane) * 4;
    if (in_stretch<W>(i, lane)) dma_round(r, span + d * 4, lds + i * 256);
  }
}

__device__ __forceinline__ void store_spike(float* p, bool s) { *p = s ? 1.0f : 0.0f; }
__device__ __forceinline__ void store_spike(bf16_t* p, bool s) { *p = s ? bf16_t(0x3f80) : bf16_t(0); }

// ---------------------------------------------------------------------------
// Cross-lane sum inside an L-lane group (L <= 16) with DPP.  Every lane of the
// group ends with the same bits: each level adds a pair of partial sums that
// both partners hold, and float addition is commutative.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}

template <int L>
__device__ __forceinline__ float group_sum(float v) {
  static_assert(L == 1 || L == 2 || L == 4 || L == 8 || L == 16, "L must be a power of two <= 16");
  if constexpr (L >= 2) v += dpp_f32<0xb1>(v);   // quad_perm(1,0,3,2): partner lane ^ 1
  if constexpr (L >= 4) v += dpp_f32<0x4e>(v);   // quad_perm(2,3,0,1): partner lane ^ 2
  if constexpr (L >= 8) v += dpp_f32<0x141>(v);  // row_half_mirror: lane i <-> 7 - i in each 8
  if constexpr (L >= 16) v += dpp_f32<0x140>(v); // row_mirror: lane i <-> 15 - i in each 16
  return v;
}

// Pairwise tree over a lane's BL partial products (left fold for odd counts).
template <int BL>
__device__ __forceinline__ float lane_sum(const float (&p)[BL]) {
  if constexpr (BL == 1) {
    return p[0];
  } else if constexpr (BL == 2) {
    return p[0] + p[1];
  } else if constexpr (BL == 4) {
    return (p[0] + p[1]) + (p[2] + p[3]);
  } else if constexpr (BL == 8) {
    return ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
  } else {
    float s = p[0];
#pragma unroll
    for (int i = 1; i < BL; ++i) s += p[i];
    return s;
  }
}

// ---------------------------------------------------------------------------
// Per-lane branch parameters of one channel.
// ---------------------------------------------------------------------------
template <int BL, int KC>
struct Branches {
  float k[BL];        // kappa * m  (0 for a gated-off branch)
  float xi[BL * KC];  // per compartment
  float rz[BL];       // 1 / zeta
  float krz[BL];      // kappa* / zeta
  bool on[BL];        // mask bit
  float rp;           // 1 / P, the residual term's weight of each compartment
  // bf16 raw rows: v_perm selector per compartment that widens its bf16 half of
  // the dword to fp32, or yields 0 on a gated-off branch (see raw_to_float_gated)
  uint32_t xsel[BL * KC];
};

// packed_pairs: bf16 rows held as element pairs per dword (kRawW == E / 2)
template <int BL, int KC>
__device__ __forceinline__ void load_branches(const ScanArgs& a, int64_t c, int sub, Branches<BL, KC>& br,
                                              bool packed_pairs = false) {
  const int64_t base = c * a.B + int64_t(sub) * BL;
  const int64_t base_i = c * a.P + int64_t(sub) * (BL * KC);
  // Every load is issued before any value is used (the null checks are uniform
  // branches around whole groups), so the lot costs one memory round trip.
  float kap[BL], zet[BL];
  uint32_t msk[BL];
#pragma unroll
  for (int j = 0; j < BL; ++j) kap[j] = a.kappa[base + j];
  if (a.zeta) {
#pragma unroll
    for (int j = 0; j < BL; ++j) zet[j] = a.zeta[base + j];
  } else {
#pragma unroll
    for (int j = 0; j < BL; ++j) zet[j] = 1.0f;
  }
  if (a.mask) {
#pragma unroll
    for (int j = 0; j < BL; ++j) msk[j] = a.mask[base + j];
  } else {
#pragma unroll
    for (int j = 0; j < BL; ++j) msk[j] = 1;
  }
  if (a.xi) {
#pragma unroll
    for (int i = 0; i < BL * KC; ++i) br.xi[i] = a.xi[base_i + i];
  } else {
#pragma unroll
    for (int i = 0; i < BL * KC; ++i) br.xi[i] = 0.0f;
  }
#pragma unroll
  for (int j = 0; j < BL; ++j) {
    const bool on = msk[j] != 0;
    br.on[j] = on;
    br.k[j] = on ? kap[j] : 0.0f;
    br.rz[j] = 1.0f / zet[j];
    br.krz[j] = br.k[j] * br.rz[j];
  }
  br.rp = a.rP;
#pragma unroll
  for (int i = 0; i < BL * KC; ++i)
    br.xsel[i] = !br.on[i / KC] ? kPermZero : (packed_pairs && (i & 1) ? kPermHi : kPermLo);
}

// Sum of squares of a branch's KC compartment offsets d = Vd - xi, in a fixed order.
template <int KC>
__device__ __forceinline__ float branch_sumsq(const float* vd, const float* xi) {
  float d = vd[0] - xi[0];
  float ss = d * d;
#pragma unroll
  for (int i = 1; i < KC; ++i) {
    d = vd[i] - xi[i];
    ss = fmaf(d, d, ss);
  }
  return ss;
}

// ---------------------------------------------------------------------------
// One forward step of the dendrite (leaky compartments, L2 aggregation over
// each branch's compartments, activation, weighted branch sum) and of the LIF
// soma.  A gated-off branch keeps a zero state (its input zeroed, or its state
// reset every step), so nothing it receives can reach the soma or its gradients.
// ---------------------------------------------------------------------------
// kGated: no select needed, because xv is already 0 on gated-off branches
// (their state then stays +0 by itself) or because every branch of the lane is
// on.  tfac / yfac (one compartment per branch, Mexican hat) receive each
// branch's signed (Vd - xi) / zeta and psi as rounded here, for the adjoint.
template <int BL, int L, int V, bool kGated = false>
__device__ __forceinline__ float dendrite_step(float (&vd)[BL * kKC<V>], const float (&xv)[BL * kKC<V>],
                                               const Branches<BL, kKC<V>>& br, float alpha,
                                               float* efac = nullptr, float* tfac = nullptr,
                                               float* yfac = nullptr) {
  constexpr int KC = kKC<V>;
  float part[BL];
#pragma unroll
  for (int j = 0; j < BL; ++j) {
#pragma unroll
    for (int i = j * KC; i < (j + 1) * KC; ++i) {
      const float v = kSL<V> ? xv[i] : fmaf(alpha, vd[i], xv[i]);
      vd[i] = (kGated || br.on[j]) ? v : 0.0f;
    }
    // KC = 1: the signed (Vd - xi)/zeta, u = |tt|; else u = ||Vd - xi|| / zeta >= 0
    float tt;
    if constexpr (KC == 1)
      tt = (vd[j] - br.xi[j]) * br.rz[j];
    else
      tt = __builtin_amdgcn_sqrtf(branch_sumsq<KC>(&vd[j * KC], &br.xi[j * KC])) * br.rz[j];
    float y;
    if constexpr (kMH<V>) {
      const float q = tt * tt;
      const float e = __builtin_amdgcn_exp2f(q * kNegHalfLog2e);
      if (efac) efac[j] = e;
      y = fmaf(-q, e, e);  // (1 - q) e
      if (tfac) tfac[j] = tt;
      if (yfac) yfac[j] = y;
    } else {
      y = KC == 1 ? fabsf(tt) : tt;
    }
    // branch pairs (2i, 2i+1) of a lane enter the sum as one fused leaf
    // kappa*_{2i+1} Y_{2i+1} + kappa*_{2i} Y_{2i}; an odd branch count folds left
    float pj = (kFuse<V, BL> && (BL % 2 == 0 ? (j & 1) : j > 0)) ? fmaf(br.k[j], y, part[j > 0 ? j - 1 : 0]) : br.k[j] * y;
    if constexpr (kRes<V>) {
#pragma unroll
      for (int i = j * KC; i < (j + 1) * KC; ++i) pj = fmaf(xv[i], br.rp, pj);  // every compartment feeds the residual
    }
    part[j] = pj;
  }
  if constexpr (kFuse<V, BL>) {
    if constexpr (BL % 2 == 0) {
      float leaf[BL / 2];
#pragma unroll
      for (int i = 0; i < BL / 2; ++i) leaf[i] = part[2 * i + 1];
      return group_sum<L>(lane_sum<BL / 2>(leaf));
    } else {
      return group_sum<L>(part[BL - 1]);
    }
  }
  return group_sum<L>(lane_sum<BL>(part));
}

__device__ __forceinline__ void soma_step(float& h, bool& s, float z, float beta, float vth) {
  h = s ? z : fmaf(beta, h, z);   // beta (1 - S[t-1]) H[t-1] + Z[t]
  s = h >= vth;                   // Theta(H - v_th), Theta(0) = 1
}

// Surrogate derivative of Theta at x = H - v_th, with a x log2(e) (or pi x)
// formed in one fused multiply-add from H; kind is a compile-time constant of
// each backward kernel (dendsn_sg).
__device__ __forceinline__ float surrogate(float h, float vth, int kind, float a) {
  if (kind == 1) {  // a sigma(a x) (1 - sigma(a x)) = a e / (1 + e)^2, e = exp(-|a x|), x = h - v_th
    const float ac = a * kLog2e;
    const float t = fmaf(h, ac, -ac * vth);  // a x log2(e)
    const float e = __builtin_amdgcn_exp2f(-fabsf(t));
    const float d = 1.0f + e;
    return a * e * __builtin_amdgcn_rcpf(d * d);
  }
  const float px = fmaf(h, kPi, -kPi * vth);  // pi x: 1 / (1 + pi^2 x^2)
  return __builtin_amdgcn_rcpf(fmaf(px, px, 1.0f));
}

// ---------------------------------------------------------------------------
// Where a thread sits: lane-in-neuron, position, batch way, group, channel.
// ---------------------------------------------------------------------------
struct Pos {
  int sub, p, way, g;
  int64_t c, m, tile;
  bool active;
};

template <int L>
__device__ __forceinline__ Pos locate(const ScanArgs& a) {
  Pos r;
  const int tid = threadIdx.x;
  r.sub = tid % L;
  const int q = tid / L;
  // nw > 1 (spatial tiles): each wave covers nw * 64 / L adjacent
  // positions, a lane taking slot q of each 64 / L stretch, so each of the nw
  // accesses per row is contiguous across the wave.
  constexpr int kSlots = 64 / L;
  r.p = a.nw > 1 ? (q / kSlots) * (a.nw * kSlots) + q % kSlots : q % a.pb;
  // Batch ways are whole waves (kFC: pb * L is 64 or 128) or a single way, so the way
  // index is wave-uniform; readfirstlane lets the compiler keep it scalar.
  r.way = __builtin_amdgcn_readfirstlane(q / a.pb);
  // Blocks are dealt to the 8 XCDs round-robin; with xk > 1 block b takes the
  // tile of b's slot in runs of xk consecutive tiles per XCD turn, so tiles
  // that share cache lines (and neighbouring DRAM pages) meet in one XCD's L2.
  int64_t blk = blockIdx.x;
  if (a.xk > 1) {
    const int64_t x = blk % 8, j = blk / 8;
    blk = (j / a.xk) * (8 * int64_t(a.xk)) + x * a.xk + j % a.xk;
  }
  r.tile = blk % a.ntiles;
  r.g = int(blk / a.ntiles);
  if (a.mode == kSpatial) {
    const int64_t c = r.tile / a.tpc;
    const int64_t s = (r.tile % a.tpc) * a.pb + r.p;
    r.c = c;
    r.active = s < a.S;
    r.m = c * a.S + s;
  } else {
    const int64_t c = r.tile * a.cpt + r.p / a.S;
    r.c = c;
    r.active = (r.p < int64_t(a.cpt) * a.S) && (c < a.C);
    r.m = c * a.S + r.p % a.S;
  }
  return r;
}

// ---------------------------------------------------------------------------
// Per-lane byte offsets of one neuron inside a sample's slice of a time row;
// every other part of an address is wave-uniform (scalar registers).
// ---------------------------------------------------------------------------
struct LaneOff {
  uint32_t x;   // X / grad_x element (I/O dtype)
  uint32_t c;   // checkpointed dendritic state (fp32)
  uint32_t s;   // spikes / grad_spikes (I/O dtype)
  uint32_t v;   // fp32 per-neuron rows (v_soma, grad_v_soma, checkpointed H)
  uint32_t xw;  // staged wide rows (see load_pieces): the wave's stretch in X / grad_x
};

template <typename IO, int E, bool CM>
__device__ __forceinline__ LaneOff lane_offsets(const ScanArgs& a, const Pos& pos) {
  LaneOff o;
  // channel-major: compartment i of position s = m - c S of channel c sits at
  // (c P + i) S + s; this lane's first compartment is i = sub E
  o.x = CM ? uint32_t((pos.m + pos.c * (a.P - 1) * a.S + int64_t(pos.sub) * E * a.S) * int64_t(sizeof(IO)))
           : uint32_t((pos.m * a.P + pos.sub * E) * int64_t(sizeof(IO)));
  o.c = uint32_t((pos.m * a.P + pos.sub * E) * 4);
  o.s = uint32_t(pos.m * int64_t(sizeof(IO)));
  o.v = uint32_t(pos.m * 4);
  return o;
}

// Batch items of one lane: bt = first, first + ways, ... < end (wave-uniform).
__device__ __forceinline__ int items_of(const ScanArgs& a, const Pos& pos, int64_t* first) {
  *first = int64_t(pos.g) * a.bpg + pos.way;
  const int64_t end = min(a.batch, int64_t(pos.g + 1) * a.bpg);
  return *first < end ? int((end - *first + a.ways - 1) / a.ways) : 0;
}

// A lane's walk over its neurons when it holds nw > 1 positions per batch item
// (neurons n, n + 64 / L, ... of the item, then the next item): the wave-uniform
// shifts of the [T, N] row index n and of the matching X element offset nx (n P,
// or in the channel-major layout the item's base plus the position shift).
struct Walk {
  int nw;
  int64_t dn, dnx, dn_item, dnx_item;
};

template <int L, bool CM>
__device__ __forceinline__ Walk make_walk(const ScanArgs& a, int64_t item_neurons) {
  Walk k;
  k.nw = a.nw > 1 ? a.nw : 1;
  k.dn = 64 / L;
  k.dnx = CM ? k.dn : k.dn * a.P;
  k.dn_item = item_neurons - (k.nw - 1) * k.dn;
  k.dnx_item = item_neurons * a.P - (k.nw - 1) * k.dnx;
  return k;
}

// ---------------------------------------------------------------------------
// Forward kernel.
//
// Each lane walks the rows X[t] of its neurons (one neuron per batch item) as
// one stream, in chunks of D rows, double-buffered: chunk c+1 is in flight
// while chunk c is computed.  A neuron's rows are padded to a multiple of D by
// re-reading its last row; padded steps compute but store nothing, and the
// state restarts at each neuron's first chunk.
// ---------------------------------------------------------------------------
template <typename IO, int BL, int D>
struct RowCursor {  // wave-uniform position of the next chunk to load
  const IO* base;   // X row 0 of the current neuron's batch item
  int w, t;         // position index inside the item (0 .. nw-1), first row of the chunk
};

template <bool CM, bool ST, typename IO, int BL, int D>
__device__ __forceinline__ void load_chunk(const ScanArgs& a, RowCursor<IO, BL, D>& cur, uint32_t ox, int T,
                                           int Tp, int64_t rowX, const Walk& wk,
                                           uint32_t (&buf)[D][kSlotW<kRawW<IO, BL, CM>, ST>]) {
#pragma unroll
  for (int k = 0; k < D; ++k) {
    // A padding step past T (its result is discarded): every lane reads the
    // start of row T - 1, one cache line per wave instead of a whole row
    // (staged: the first stretch of the row).
    const int tk = cur.t + k;
    const int t = min(tk, T - 1);
    if constexpr (ST)
      load_pieces<IO, kRawW<IO, BL, CM>>(cur.base + int64_t(t) * rowX, tk < T ? ox : 0u, buf[k]);
    else
      load_raw<IO, BL, CM>(cur.base + int64_t(t) * rowX, tk < T ? ox : 0u, a.xes, buf[k]);
  }
  cur.t += D;
  if (cur.t >= Tp) {
    cur.t = 0;
    const bool last = ++cur.w == wk.nw;
    if (last) cur.w = 0;
    cur.base += last ? wk.dnx_item : wk.dnx;
  }
}

// Running state of the neuron a lane is computing, and wave-uniform output
// pointers of its batch item (advanced step by step, never recomputed).
template <typename IO, int E>
struct FwdLane {
  float vd[E];
  float h;
  bool s;
  int t;          // step index of the chunk being computed (0 .. Tp-1)
  int w;          // position index inside the batch item (0 .. nw-1)
  int kc;         // steps until the next checkpoint
  IO* sp;         // spikes row t of this batch item
  float* vp;      // v_soma row t (or null)
  float* ckv;     // next checkpoint's dendritic-state block of this item (stateful dendrite)
  float* ckh;     // next checkpoint's H row of this item
};

template <typename IO, int E>
__device__ __forceinline__ void fwd_item_start(const FwdArgs& fa, int64_t n0, FwdLane<IO, E>& st) {
  const ScanArgs& a = fa.s;
  st.t = 0;
  st.kc = a.K;
  st.sp = static_cast<IO*>(fa.spikes) + n0;
  st.vp = fa.vsoma ? fa.vsoma + n0 : nullptr;
  st.ckv = fa.ckpt ? fa.ckpt + n0 * a.P : nullptr;
  st.ckh = fa.ckh ? fa.ckh + n0 : nullptr;
#pragma unroll
  for (int j = 0; j < E; ++j) st.vd[j] = 0.0f;
  st.h = 0.0f;
  st.s = false;
}

template <typename IO, int BL, int L, int V, int D, bool ST>
__device__ __forceinline__ void compute_chunk(const FwdArgs& fa, const LaneOff& lo, const Branches<BL, kKC<V>>& br,
                                              float alpha, bool lead, int T, int Tp, const Walk& wk,
                                              const uint32_t (&buf)[D][kSlotW<kRawW<IO, BL * kKC<V>, kCM<V>>, ST>],
                                              uint32_t* stage, FwdLane<IO, BL * kKC<V>>& st) {
  constexpr int E = BL * kKC<V>;
  constexpr int W = kRawW<IO, E, kCM<V>>;
  const ScanArgs& a = fa.s;
#pragma unroll
  for (int k = 0; k < D; ++k) {
    const int t = st.t + k;
    float xk[E];
    uint32_t raw[W];
    slot_to_lane<W, ST>(buf[k], stage, raw);
    if constexpr (kGateIn<IO, V>) raw_to_float_gated(raw, br.xsel, xk);
    else raw_to_float<IO, E>(raw, xk);
    const float z = dendrite_step<BL, L, V, kGateIn<IO, V>>(st.vd, xk, br, alpha);
    soma_step(st.h, st.s, z, a.beta, a.vth);
    if (t < T) {  // padded steps store nothing
      if (lead) {
        store_spike(at(st.sp, lo.s), st.s);
        if (st.vp) *at(st.vp, lo.v) = st.h;
      }
      if (--st.kc == 0) {
        st.kc = a.K;
        if (st.ckh && t + 1 < T) {
          if constexpr (!kSL<V>) {  // the Stateless Dendrite has no state to keep
            store_vec<E>(at(st.ckv, lo.c), st.vd);
            st.ckv += a.N * a.P;
          }
          if (lead) *at(st.ckh, lo.v) = st.h;
          st.ckh += a.N;
        }
      }
      st.sp += a.N;
      if (st.vp) st.vp += a.N;
    }
  }
  st.t += D;
  if (st.t >= Tp) {  // next neuron of this lane: next position of the item, or the next item
    const bool last = ++st.w == wk.nw;
    if (last) st.w = 0;
    const int64_t n0 = (st.sp - static_cast<IO*>(fa.spikes)) - int64_t(T) * a.N + (last ? wk.dn_item : wk.dn);
    fwd_item_start<IO, E>(fa, n0, st);
  }
}

// ---------------------------------------------------------------------------
// Forward fast path: T a multiple of D (no padding steps), no v_soma output and
// checkpoints, if any, only at chunk ends (K a multiple of D; the kernel takes
// it without interior checkpoints).  A step's bookkeeping is then the spike
// store alone: a row's address is the previous row's plus one row stride, and
// the checkpoint and next-neuron decisions are taken once per chunk.  A SIMD issues at most one scalar instruction per
// vector instruction slot, so the general path's per-step address arithmetic
// and conditions (more scalar than vector instructions per step) held the
// kernel back.
// ---------------------------------------------------------------------------
template <typename IO, int BL, int L, int V, int D, bool ST>
__device__ __forceinline__ void fwd_fast(const FwdArgs& fa, const LaneOff& lo, const Branches<BL, kKC<V>>& br,
                                         float alpha, bool lead, int64_t bt0, int nk, const Walk& wk,
                                         uint32_t* stage) {
  constexpr int E = BL * kKC<V>;
  constexpr int W = kRawW<IO, E, kCM<V>>;
  constexpr int SW = kSlotW<W, ST>;
  const ScanArgs& a = fa.s;
  const int T = int(a.T), K = a.K;
  const int64_t rowX = a.N * a.P;
  const int nchunks = nk * wk.nw * (T / D);
  if (nchunks <= 0) return;
  // load cursor (wave-uniform): the next chunk's first row, the row 0 of that
  // chunk's neuron, its step and position index
  const IO* lrow = static_cast<const IO*>(a.x) + bt0 * a.M * a.P;
  const IO* lbase = lrow;
  int lt = 0, lw = 0;
  auto load = [&](uint32_t (&buf)[D][SW]) {
    const IO* r = lrow;
#pragma unroll
    for (int k = 0; k < D; ++k) {
      if constexpr (ST) load_pieces<IO, W>(r, lo.x, buf[k]);
      else load_raw<IO, E, kCM<V>>(r, lo.x, a.xes, buf[k]);
      r += rowX;
    }
    lt += D;
    if (lt == T) {
      lt = 0;
      const bool last = ++lw == wk.nw;
      if (last) lw = 0;
      lbase += last ? wk.dnx_item : wk.dnx;
      r = lbase;
    }
    lrow = r;
  };
  // the neuron being computed: state, step, position, output rows (uniform)
  IO* const spk = static_cast<IO*>(fa.spikes);
  int64_t n0 = bt0 * a.M;
  IO* sp = spk + n0;
  float* ckv = fa.ckpt ? fa.ckpt + n0 * a.P : nullptr;
  float* ckh = fa.ckh ? fa.ckh + n0 : nullptr;
  float vd[E];
#pragma unroll
  for (int j = 0; j < E; ++j) vd[j] = 0.0f;
  float h = 0.0f;
  bool s = false;
  int ct = 0, cw = 0, kc = K;
  auto compute = [&](const uint32_t (&buf)[D][SW]) {
#pragma unroll
    for (int k = 0; k < D; ++k) {
      float xk[E];
      uint32_t raw[W];
      slot_to_lane<W, ST>(buf[k], stage, raw);
      if constexpr (kGateIn<IO, V>) raw_to_float_gated(raw, br.xsel, xk);
      else raw_to_float<IO, E>(raw, xk);
      const float z = dendrite_step<BL, L, V, kGateIn<IO, V>>(vd, xk, br, alpha);
      soma_step(h, s, z, a.beta, a.vth);
      if (lead) store_spike(at(sp, lo.s), s);
      sp += a.N;
    }
    ct += D;
    kc -= D;
    if (kc == 0) {  // a checkpoint after this chunk's last step (none after the last step)
      kc = K;
      if (ckh && ct < T) {
        if constexpr (!kSL<V>) {
          store_vec<E>(at(ckv, lo.c), vd);
          ckv += a.N * a.P;
        }
        if (lead) *at(ckh, lo.v) = h;
        ckh += a.N;
      }
    }
    if (ct == T) {  // next neuron of this lane: next position of the item, or the next item
      ct = 0;
      kc = K;
      const bool last = ++cw == wk.nw;
      if (last) cw = 0;
      n0 += last ? wk.dn_item : wk.dn;
      sp = spk + n0;
      ckv = fa.ckpt ? fa.ckpt + n0 * a.P : nullptr;
      ckh = fa.ckh ? fa.ckh + n0 : nullptr;
#pragma unroll
      for (int j = 0; j < E; ++j) vd[j] = 0.0f;
      h = 0.0f;
      s = false;
    }
  };
  uint32_t bufA[D][SW], bufB[D][SW];
  load(bufA);
  // Every later wait is then counted from loads issued inside the loop, which
  // are unconditional (the last one or two chunks run after it).
  __builtin_amdgcn_s_waitcnt(kWaitVmem);
  int c = 0;
  for (; c + 2 < nchunks; c += 2) {
    load(bufB);
    compute(bufA);
    load(bufA);
    compute(bufB);
  }
  if (c + 1 < nchunks) {
    load(bufB);
    compute(bufA);
    compute(bufB);
  } else {
    compute(bufA);
  }
}

// The forward of the lane's neurons (ST: wide rows staged, see load_pieces;
// lo.x is then the wave's stretch, the same for every lane).
template <typename IO, int BL, int L, int V, int D, bool ST>
__device__ __forceinline__ void fwd_run(const FwdArgs& fa, const LaneOff& lo, const Branches<BL, kKC<V>>& br,
                                        float alpha, bool lead, int64_t bt0, int nk, uint32_t* stage) {
  constexpr int E = BL * kKC<V>;
  constexpr int SW = kSlotW<kRawW<IO, E, kCM<V>>, ST>;
  const ScanArgs& a = fa.s;
  const int T = int(a.T);
  const int Tp = (T + D - 1) / D * D;
  const int64_t rowX = a.N * a.P;
  const Walk wk = make_walk<L, kCM<V>>(a, int64_t(a.ways) * a.M);
  // (with interior checkpoints, e.g. the T = 64 layer with K = 8, the general
  // path measured 2 % faster: those long sequences are bound by memory latency)
  if (T % D == 0 && !fa.vsoma && a.nck == 0) {
    fwd_fast<IO, BL, L, V, D, ST>(fa, lo, br, alpha, lead, bt0, nk, wk, stage);
    return;
  }
  const int nchunks = nk * wk.nw * (Tp / D);

  RowCursor<IO, E, D> cur;
  cur.base = static_cast<const IO*>(a.x) + bt0 * a.M * a.P;
  cur.w = 0;
  cur.t = 0;
  FwdLane<IO, E> st;
  st.w = 0;
  fwd_item_start<IO, E>(fa, bt0 * a.M, st);

  if (nchunks <= 0) return;
  uint32_t bufA[D][SW], bufB[D][SW];
  load_chunk<kCM<V>, ST>(a, cur, lo.x, T, Tp, rowX, wk, bufA);
  // Every later wait is then counted from loads issued inside the loop, which
  // are unconditional (the last one or two chunks run after it).
  __builtin_amdgcn_s_waitcnt(kWaitVmem);
  int c = 0;
  for (; c + 2 < nchunks; c += 2) {
    load_chunk<kCM<V>, ST>(a, cur, lo.x, T, Tp, rowX, wk, bufB);
    compute_chunk<IO, BL, L, V, D, ST>(fa, lo, br, alpha, lead, T, Tp, wk, bufA, stage, st);
    load_chunk<kCM<V>, ST>(a, cur, lo.x, T, Tp, rowX, wk, bufA);
    compute_chunk<IO, BL, L, V, D, ST>(fa, lo, br, alpha, lead, T, Tp, wk, bufB, stage, st);
  }
  if (c + 1 < nchunks) {
    load_chunk<kCM<V>, ST>(a, cur, lo.x, T, Tp, rowX, wk, bufB);
    compute_chunk<IO, BL, L, V, D, ST>(fa, lo, br, alpha, lead, T, Tp, wk, bufA, stage, st);
    compute_chunk<IO, BL, L, V, D, ST>(fa, lo, br, alpha, lead, T, Tp, wk, bufB, stage, st);
  } else {
    compute_chunk<IO, BL, L, V, D, ST>(fa, lo, br, alpha, lead, T, Tp, wk, bufA, stage, st);
  }
}

// Whether a wave may stage its wide rows: every lane active (checked by the
// caller), the layer's per-sample slice a multiple of 16 bytes (the host's
// flag: then every row and item keeps the alignment of the first), and the
// wave's first stretch 16-byte aligned.  lo.x of lane 0 is the stretch's start.
template <typename IO>
__device__ __forceinline__ bool stage_rows(const ScanArgs& a, uint32_t span0, int64_t bt0) {
  const uintptr_t p = reinterpret_cast<uintptr_t>(static_cast<const IO*>(a.x) + bt0 * a.M * a.P) + span0;
  return a.stg && (p & 15) == 0;
}

template <typename IO, int BL, int L, int V>
__global__ void __launch_bounds__(kThreads) dendsn_fwd_kernel(FwdArgs fa) {
  constexpr int D = 4;  // rows per chunk; two chunks in flight per lane
  if (fa.s.beta_p) fa.s.beta = fa.s.beta_p[0];  // learnable (PLIF) decay
  const ScanArgs& a = fa.s;
  const Pos pos = locate<L>(a);
  constexpr int E = BL * kKC<V>;
  constexpr int W = kRawW<IO, E, kCM<V>>;
  constexpr bool kWide = kWideRow<IO, E, kCM<V>>;
  const bool full = kWide && __all(pos.active);
  if (!pos.active) return;  // whole L-lane groups leave together
  Branches<BL, kKC<V>> br;
  load_branches<BL, kKC<V>>(a, pos.c, pos.sub, br, W * 2 == E);
  const float alpha = a.alpha ? a.alpha[0] : 0.0f;
  LaneOff lo = lane_offsets<IO, E, kCM<V>>(a, pos);
  const bool lead = pos.sub == 0;
  int64_t bt0;
  const int nk = items_of(a, pos, &bt0);
  if constexpr (kWide) {
    __shared__ uint32_t stage[kThreads / 64][64 * W];
    const uint32_t span = __builtin_amdgcn_readfirstlane(lo.x);
    if (full && stage_rows<IO>(a, span, bt0)) {
      lo.x = span;
      fwd_run<IO, BL, L, V, D, true>(fa, lo, br, alpha, lead, bt0, nk, stage[threadIdx.x >> 6]);
      return;
    }
  }
  fwd_run<IO, BL, L, V, D, false>(fa, lo, br, alpha, lead, bt0, nk, nullptr);
}

// ---------------------------------------------------------------------------
// Backward kernel.  For each neuron, the segments between checkpoints are
// visited from last to first.  A segment is cut into chunks of compile-time
// length KS (the first may be shorter), each a visit of the memory pipeline
// (BwdPath): a chunk starts from the checkpoint, or from a state of the same
// segment kept in LDS, recomputes its own steps while stashing the dendritic
// state and H in registers, then runs the adjoint recurrences backwards through
// them.
// ---------------------------------------------------------------------------
template <int BL, int E>
struct Accum {
  float k[BL], xi[E], z[BL];
  float a;   // g_alpha terms of this lane's branches
  float b;   // g_beta terms of this lane's neuron (counted by its first lane only)
};

// Groups of several batch items (Plan::fold): after each item the lane's sums join
// float64 sums in LDS and start again, so a lane's fp32 chain stays one item long
// whatever the group holds.  The order of the values: g_kappa, g_xi, g_zeta of the
// lane as in Accum, then g_alpha and g_beta.
template <int BL, int E>
constexpr int kFoldValues = 2 * BL + E + 2;

__device__ __forceinline__ double* fold_sums(const BwdArgs& ba) {
  extern __shared__ __align__(16) float slots[];
  return reinterpret_cast<double*>(slots + ba.fold_at);
}

template <int BL, int E>
__device__ __forceinline__ void fold_item(const BwdArgs& ba, Accum<BL, E>& acc) {
  if (!ba.fold) return;
  double* d = fold_sums(ba) + threadIdx.x;
  auto join = [&](int i, float& v) {
    d[i * kThreads] += double(v);
    v = 0.0f;
  };
#pragma unroll
  for (int j = 0; j < BL; ++j) join(j, acc.k[j]);
#pragma unroll
  for (int i = 0; i < E; ++i) join(BL + i, acc.xi[i]);
#pragma unroll
  for (int j = 0; j < BL; ++j) join(BL + E + j, acc.z[j]);
  join(2 * BL + E, acc.a);
  join(2 * BL + E + 1, acc.b);
}

template <typename IO, int E>
struct BwdLane {  // adjoint state carried backwards through time, and pointers
  float dh_next;
  float lam[E];
  uint32_t* stage;   // the wave's LDS buffer for staged wide rows (see load_pieces)
};

// A chunk's rows in raw form (see load_raw).  The single-chunk pipeline
// carries the next neuron's rows this way: a conversion issued next to the
// loads would make the wave wait for them at once instead of while the current
// neuron's adjoint pass runs.
template <typename IO, int E, int CS, bool CM, bool ST = false>
struct ChunkRaw {
  uint32_t x[CS][kSlotW<kRawW<IO, E, CM>, ST>];
  uint32_t gs[CS];
  float gv[CS];
};

// Requests CS rows from x / g / gv (the row of the chunk's first step) on; the
// row addresses advance by one stride at a time, two scalar additions per row.
// PART: only the first cs rows exist (cs is wave-uniform); the others are read
// through buffers of no bytes, so they cost no memory traffic and the number of
// requests, which the waits are counted by, stays the same.  GV = false:
// grad_v_soma is known absent; else gvbytes = 0 says that it is (one uniform
// branch: requests through empty buffers cost a masked bf16 layer of twelve steps,
// K = 4, 5 %).  rev = false: X alone.
// PAIRED: grad_spikes row by row with X (one-chunk neurons of four steps: 0.5-1 %
// faster); else behind all X rows, which the recompute waits for first (bf16
// ten-step layer 826 -> 752 us, 64 steps with K = 8: 236 -> 227 us).
template <typename IO, int E, int CS, bool CM, bool GV = true, bool ST = false, bool PART = false, bool PAIRED = false>
__device__ __forceinline__ void load_chunk_raw(const ScanArgs& a, const LaneOff& lo, const IO* x, const IO* g,
                                               const float* gv, uint32_t gvbytes, ChunkRaw<IO, E, CS, CM, ST>& in,
                                               int cs = CS, bool rev = true) {
  const int64_t rowX = a.N * a.P;
  auto bytes = [&](int k, bool want, uint32_t n) { return PART ? uniform_u32(want && k < cs ? n : 0u) : n; };
  auto load_gs = [&](int k) {
    const rsrc_t rg = make_rsrc(g, bytes(k, rev, 0xFFFFFFFFu));
    in.gs[k] = sizeof(IO) == 4 ? __builtin_amdgcn_raw_buffer_load_b32(rg, lo.s, 0, kAuxNT)
                               : uint32_t(__builtin_amdgcn_raw_buffer_load_b16(rg, lo.s, 0, kAuxNT));
    g += a.N;
  };
#pragma unroll
  for (int k = 0; k < CS; ++k) {
    const rsrc_t rx = make_rsrc(x, bytes(k, true, 0xFFFFFFFFu));
    if constexpr (ST) bload_pieces<kRawW<IO, E, CM>>(rx, lo.xw, in.x[k]);
    else bload_raw<IO, E, CM>(rx, lo.x, a.xes, in.x[k]);
    x += rowX;
    if (PAIRED) load_gs(k);
  }
  if (!PAIRED) {
#pragma unroll
    for (int k = 0; k < CS; ++k) load_gs(k);
  }
  if (GV && gvbytes) {
#pragma unroll
    for (int k = 0; k < CS; ++k) {
      in.gv[k] = __uint_as_float(
          __builtin_amdgcn_raw_buffer_load_b32(make_rsrc(gv, bytes(k, rev, gvbytes)), lo.v, 0, kAuxNT));
      gv += a.N;
    }
  } else {
#pragma unroll
    for (int k = 0; k < CS; ++k) in.gv[k] = 0.0f;
  }
}

// Registers a chunk's recompute leaves for its adjoint pass: the dendritic
// state before and at each step, H at each step and, for the Mexican hat, the
// exp(-u^2/2) factor of each step.
template <int BL, int CS, int V, bool TY = true>
struct Stash {
  float v[CS + 1][BL * kKC<V>];
  float e[kMH<V> ? CS : 1][BL];
  // one compartment per branch with the Mexican hat: the signed (Vd - xi) / zeta
  // and psi of each step, as the recompute rounded them (kTY; else the adjoint
  // forms both again, with the same operations)
  static constexpr bool kTY = TY && kMH<V> && kKC<V> == 1;
  float t[kTY ? CS : 1][BL];
  float y[kTY ? CS : 1][BL];
  float h[CS];
  float hd0;  // (1 - S) H before the chunk's first step: the decayed term beta multiplies
};

// Re-runs the chunk's forward steps exactly as the forward kernel did (the same
// inline step function, so the same bits).  NG: every branch of the lane is on
// (no gate select; with every branch on the select is the identity).  PART: only
// the first cs steps are run (cs is wave-uniform).
template <int BL, int L, int V, int CS, bool NG = false, bool PART = false, bool TY = true>
__device__ __forceinline__ void recompute_chunk(const ScanArgs& a, const Branches<BL, kKC<V>>& br, float alpha,
                                                const float (&v0)[BL * kKC<V>], float h0, bool s0,
                                                const float (&x)[CS][BL * kKC<V>], Stash<BL, CS, V, TY>& st,
                                                int cs = CS) {
  constexpr int E = BL * kKC<V>;
#pragma unroll
  for (int j = 0; j < E; ++j) st.v[0][j] = v0[j];
  st.hd0 = s0 ? 0.0f : h0;
  float h = h0;
  bool s = s0;
#pragma unroll
  for (int k = 0; k < CS; ++k) {
#pragma unroll
    for (int j = 0; j < E; ++j) st.v[k + 1][j] = st.v[k][j];
    if (PART && k >= cs) continue;
    constexpr bool ty = Stash<BL, CS, V, TY>::kTY;
    const float z = dendrite_step<BL, L, V, NG>(st.v[k + 1], x[k], br, alpha, kMH<V> ? st.e[kMH<V> ? k : 0] : nullptr,
                                            ty ? st.t[ty ? k : 0] : nullptr, ty ? st.y[ty ? k : 0] : nullptr);
    soma_step(h, s, z, a.beta, a.vth);
    st.h[k] = h;
  }
}

// The adjoint recurrences through one chunk, last step first; writes grad_x
// (gx: its row of the chunk's first step) and accumulates the parameter gradients.  PART: only the first cs steps of
// the chunk are real (cs is wave-uniform; the others are padding and skipped).
template <typename IO, int BL, int L, int V, int CS, bool PART = false, bool ST = false, bool TY = true>
__device__ __forceinline__ void reverse_chunk(const BwdArgs& ba, const LaneOff& lo, const Branches<BL, kKC<V>>& br,
                                              float alpha, float beta_r, IO* gx, const Stash<BL, CS, V, TY>& st,
                                              const float (&gs)[CS], const float (&gvr)[CS],
                                              BwdLane<IO, BL * kKC<V>>& bl, Accum<BL, BL * kKC<V>>& acc,
                                              int cs = CS) {
  constexpr int KC = kKC<V>, E = BL * KC;
  const ScanArgs& a = ba.s;
  const int64_t rowX = a.N * a.P;
  const float beta = a.beta, vth = a.vth;
  gx += (CS - 1) * rowX;  // grad_x row of step k, walking down
#pragma unroll
  for (int k = CS - 1; k >= 0; gx -= rowX, --k) {
    if (PART && k >= cs) continue;
    const float hk = st.h[k];
    const bool sk = hk >= vth;
    const float sgv = surrogate(hk, vth, kSG<V>, ba.sg_scale);
    const float dS = fmaf(-beta_r * hk, bl.dh_next, gs[k]);  // beta_r = 0: reset detached
    float dh = fmaf(sgv, dS, gvr[k]);
    dh = sk ? dh : fmaf(beta, bl.dh_next, dh);
    // H[t] = beta (1 - S[t-1]) H[t-1] + Z[t]: learnable-beta (PLIF) gradient
    const float hd = k > 0 ? (st.h[k > 0 ? k - 1 : 0] >= vth ? 0.0f : st.h[k > 0 ? k - 1 : 0]) : st.hd0;
    acc.b = fmaf(dh, hd, acc.b);
    float gxo[E];
#pragma unroll
    for (int j = 0; j < BL; ++j) {
      if constexpr (KC == 1) {
        constexpr bool ty = Stash<BL, CS, V, TY>::kTY;
        const float tt = ty ? st.t[ty ? k : 0][j] : (st.v[k + 1][j] - br.xi[j]) * br.rz[j];
        const float dhk = dh * br.krz[j];
        float y, r;  // psi(u), and r = kappa* dH psi'(u) sgn(Vd - xi) / zeta
        if constexpr (kMH<V>) {
          const float e = st.e[k][j];
          y = ty ? st.y[ty ? k : 0][j] : fmaf(-(tt * tt), e, e);
          r = (tt * fmaf(2.0f, e, y)) * -dhk;          // psi'(u) sgn = tt (q - 3) e = -tt (y + 2 e)
        } else {
          y = fabsf(tt);
          r = tt > 0.0f ? dhk : (tt < 0.0f ? -dhk : 0.0f);
        }
        bl.lam[j] = kSL<V> ? r : fmaf(alpha, bl.lam[j], r);
        gxo[j] = kRes<V> ? fmaf(dh, br.rp, bl.lam[j]) : bl.lam[j];
        acc.k[j] = fmaf(dh, y, acc.k[j]);
        acc.xi[j] -= r;
        acc.z[j] = fmaf(-r, tt, acc.z[j]);
        if constexpr (!kSL<V>) acc.a = fmaf(bl.lam[j], st.v[k][j], acc.a);
      } else {
        // u = ||d|| rz with d = Vd - xi over the branch's compartments;
        // du/dVd_i = rz d_i / ||d|| (0 at ||d|| = 0), du/dzeta = -u rz.
        const float nrm = __builtin_amdgcn_sqrtf(branch_sumsq<KC>(&st.v[k + 1][j * KC], &br.xi[j * KC]));
        const float u = nrm * br.rz[j];
        const float dhk = dh * br.krz[j];          // kappa* dH / zeta
        float y, w, gzu;  // psi(u), the factor of d_i in dL/dVd_i, and psi'(u) u
        if constexpr (kMH<V>) {
          const float q = u * u;
          const float e = st.e[kMH<V> ? k : 0][j];
          y = fmaf(-q, e, e);                        // (1 - q) e, rounded as in the forward
          const float qe = fmaf(-3.0f, e, q * e);    // psi'(u) / u = (q - 3) e
          w = dhk * (qe * br.rz[j]);                 // kappa* dH psi'(u) rz / ||d||
          gzu = qe * q;
        } else {
          y = u;
          w = nrm > 0.0f ? dhk * __builtin_amdgcn_rcpf(nrm) : 0.0f;
          gzu = u;
        }
#pragma unroll
        for (int i = j * KC; i < (j + 1) * KC; ++i) {
          const float r = w * (st.v[k + 1][i] - br.xi[i]);
          bl.lam[i] = kSL<V> ? r : fmaf(alpha, bl.lam[i], r);
          gxo[i] = kRes<V> ? fmaf(dh, br.rp, bl.lam[i]) : bl.lam[i];
          acc.xi[i] -= r;
          if constexpr (!kSL<V>) acc.a = fmaf(bl.lam[i], st.v[k][i], acc.a);
        }
        acc.k[j] = fmaf(dh, y, acc.k[j]);
        acc.z[j] = fmaf(-dhk, gzu, acc.z[j]);     // -kappa* dH psi'(u) u / zeta
      }
    }
    if constexpr (ST) store_gx_staged<IO, E>(gx, lo.xw, gxo, bl.stage);
    else store_gx<E, kCM<V>>(gx, lo.x, a.xes, gxo);
    bl.dh_next = dh;
  }
}

// The short-sequence case: T <= KS, so every neuron is one chunk that starts
// from the zero state (PART: T < KS, or known at run time only).  Software-
// pipelined over the lane's neurons: the next neuron's rows are requested as
// soon as this neuron's rows are widened to float, so they stream in during its
// recompute and adjoint pass.  FAST: no branch of the wave is gated off (no
// gate select, see recompute_chunk) and no grad_v_soma is given (no loads of it).
template <typename IO, int BL, int L, int V, int KS, bool FAST = false, bool ST = false, bool PART = false>
__device__ __forceinline__ void single_chunk_items(const BwdArgs& ba, const LaneOff& lo,
                                                   const Branches<BL, kKC<V>>& br, float alpha, int64_t bt0,
                                                   int nk, Accum<BL, BL * kKC<V>>& acc, uint32_t* stage) {
  constexpr int E = BL * kKC<V>;
  const ScanArgs& a = ba.s;
  const float beta_r = ba.detach ? 0.0f : a.beta;
  // The lane's nw positions of each item in turn, then the next item (Walk).
  const Walk wk = make_walk<L, kCM<V>>(a, int64_t(a.ways) * a.M);
  const int nvis = wk.nw * nk;
  const int cs = PART ? int(a.T) : KS;
  int64_t n0 = bt0 * a.M, nx0 = bt0 * a.M * a.P;
  const IO* x = static_cast<const IO*>(a.x);
  const IO* g = static_cast<const IO*>(ba.gspk);
  if (nvis <= 0) return;
  constexpr int W = kRawW<IO, E, kCM<V>>;
  ChunkRaw<IO, E, KS, kCM<V>, ST> cur;
  load_chunk_raw<IO, E, KS, kCM<V>, !FAST, ST, PART, !PART>(a, lo, x + nx0, g + n0, ba.gvz + n0, ba.gvn, cur, cs);
  // Every later wait is then counted from loads issued inside the loop, whose
  // next-neuron loads are unconditional (the last neuron runs after it).
  __builtin_amdgcn_s_waitcnt(kWaitVmem);
  int w = 0;
  auto item = [&](const ChunkRaw<IO, E, KS, kCM<V>, ST>& in, bool more, ChunkRaw<IO, E, KS, kCM<V>, ST>& nxt) {
    BwdLane<IO, E> bl;
    bl.stage = stage;
    bl.dh_next = 0.0f;
    IO* const gx = static_cast<IO*>(ba.gx) + nx0;
    float xin[KS][E], gsv[KS], zero[E];
#pragma unroll
    for (int j = 0; j < E; ++j) { bl.lam[j] = 0.0f; zero[j] = 0.0f; }
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      uint32_t raw[W];
      slot_to_lane<W, ST>(in.x[k], stage, raw);
      raw_to_float<IO, E>(raw, xin[k]);
      gsv[k] = raw_to_float<IO>(in.gs[k]);
    }
    float gvv[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) gvv[k] = FAST ? 0.0f : in.gv[k];
    if (more) {
      const bool last_w = ++w == wk.nw;
      if (last_w) w = 0;
      n0 += last_w ? wk.dn_item : wk.dn;
      nx0 += last_w ? wk.dnx_item : wk.dnx;
      load_chunk_raw<IO, E, KS, kCM<V>, !FAST, ST, PART, !PART>(a, lo, x + nx0, g + n0, ba.gvz + n0, ba.gvn, nxt, cs);
    }
    // Keeps the requests at this point: left to itself the scheduler sank them
    // below most of the recompute (bf16 layers' backward 2-6 % slower).
    __builtin_amdgcn_sched_barrier(0);
    // chunks of 8 steps leave no registers for psi (a third wave per SIMD instead)
    Stash<BL, KS, V, (KS <= 4)> st;
    recompute_chunk<BL, L, V, KS, FAST, PART>(a, br, alpha, zero, 0.0f, false, xin, st, cs);
    reverse_chunk<IO, BL, L, V, KS, PART, ST>(ba, lo, br, alpha, beta_r, gx, st, gsv, gvv, bl, acc, cs);
    fold_item<BL, E>(ba, acc);
  };
  for (int i = 0; i + 1 < nvis; ++i) {
    ChunkRaw<IO, E, KS, kCM<V>, ST> nxt;
    item(cur, true, nxt);
    cur = nxt;
  }
  item(cur, false, cur);
}

// Every other sequence: segments of K steps between checkpoints, visited from
// last to first.  A segment of at most KS steps is one visit of the memory
// pipeline (SEG); a longer one is cut into chunks of KS steps with the remainder
// first.  The next visit's rows are requested before this visit computes, so they
// stream in meanwhile.  A segment of several chunks is first run forward up to its
// last chunk (advance visits, X rows only), each chunk's starting state going to
// the lane's LDS slots; then every chunk, last to first, is recomputed from its
// slot and reversed.  With every start kept (bsh = 0) X is read at most twice;
// where the slots hold every (1 << bsh)-th start, a chunk between two advances
// again from the slot below it, about 1 + (2^bsh + 1) / 2 reads in all, and as
// bsh grows with T / KS, very long segments without checkpoints stay quadratic in
// T.  (Re-running each chunk from the segment's start with no load in flight,
// T = 64 bf16: 3070 us against 594.)  Rows past a short chunk's end go through
// buffers of no bytes and are skipped by the adjoint pass.
template <typename IO, int E, int CS, bool CM, bool ST, bool SL>
struct VisitRaw {
  ChunkRaw<IO, E, CS, CM, ST> in;
  float v0[SL ? 1 : E];  // checkpointed compartment states before the segment
  float h0;              // and somatic potential (0 for the first segment)
};

// Wave-uniform place in the visit order: neuron (its [T, N] index and X offset),
// segment, position index, the chunk being run and the chunk that its run leads
// to (equal where the chunk is reversed, else the visit only advances).
struct VisitAt {
  int64_t n0, nx0;
  int seg, w, i, j;
  int c0, cs;   // first step and length of chunk i
  bool first;   // the visit starts its run (its state comes from a checkpoint or a slot)
  bool last;    // the segment's last chunk is being reversed
  bool pre;     // the run starts at chunk 1: the visit itself steps through chunk 0
};

// Two-chunk segments whose first chunk is this short are not given an advance
// visit: the visit of the second chunk reads those rows itself (one more visit of
// KS requested rows cost more than the wait: five steps of bf16, 784 positions,
// 128 channels, B = 1 55.1 against 98.9 us, ten compartments 288 against 389).
constexpr int kPreSteps = 2;

// Chunk i of segment seg: i = 0 holds the remainder.
template <int KS>
__device__ __forceinline__ void place_chunk(const ScanArgs& a, VisitAt& c) {
  const int t0 = c.seg * a.K, len = min(a.K, int(a.T) - t0);
  const int rem = len - ((len - 1) / KS) * KS;  // 1 .. KS steps in chunk 0
  c.c0 = c.i > 0 ? t0 + rem + (c.i - 1) * KS : t0;
  c.cs = c.i > 0 ? KS : rem;
}
// The start of a segment's first run, to its last chunk.  PRE: see kPreSteps.
template <int KS, bool SEG, bool PRE>
__device__ __forceinline__ void enter_segment(const ScanArgs& a, VisitAt& c) {
  if constexpr (SEG) {
    c.c0 = c.seg * a.K;
    c.cs = min(a.K, int(a.T) - c.c0);
  } else {
    const int len = min(a.K, int(a.T) - c.seg * a.K);
    c.j = (len - 1) / KS;
    c.pre = PRE && c.j == 1 && len - KS <= kPreSteps;
    c.i = c.pre ? 1 : 0;
    c.first = c.last = true;
    place_chunk<KS>(a, c);
  }
}
// The next visit; true where it is another neuron's first.  SEG: every segment is
// one chunk.
template <int KS, bool SEG, bool PRE = true>
__device__ __forceinline__ bool next_visit(const ScanArgs& a, const Walk& wk, int nseg, VisitAt& c) {
  if (!SEG && c.j > 0) {
    if (c.i < c.j) {  // on towards chunk j
      ++c.i;
      c.first = false;
      place_chunk<KS>(a, c);
      return false;
    }
    --c.j;  // the chunk below, from the slot at or below it
    c.i = (c.j >> a.bsh) << a.bsh;
    c.first = true;
    c.last = c.pre = false;
    place_chunk<KS>(a, c);
    return false;
  }
  const bool neuron = c.seg == 0;
  if (neuron) {
    c.seg = nseg;
    const bool last_w = ++c.w == wk.nw;
    if (last_w) c.w = 0;
    c.n0 += last_w ? wk.dn_item : wk.dn;
    c.nx0 += last_w ? wk.dnx_item : wk.dnx;
  }
  --c.seg;
  enter_segment<KS, SEG, PRE>(a, c);
  return neuron;
}

// The next visit's rows are requested before this visit computes; where a
// stateful fp32 lane's stash fills the registers, after it (64 steps, K = 8:
// 236 -> 227 us; ten compartments spilled with rows in flight).
template <typename IO, int V>
constexpr bool kEarlyVisit = sizeof(IO) == 2 || kSL<V>;

// Whether the recompute skips the padding steps of a short chunk (a branch a
// step) or runs them too, with the steps of a chunk scheduled together.  Running
// them is faster (Stateless bf16, twelve steps, K = 4: 10-15 %; a masked layer 5 %)
// as long as the registers last: wide lanes spilled (fourteen compartments fp32
// 380 -> 720 us, ten stateful bf16 345 -> 394), and so did the multi-chunk visits
// of the stateful dendrite (24 steps bf16: 141 -> 155 us) and the channel-major
// eight-step ones with the Mexican hat (183 -> 202).
template <int E, int V, int KS, bool SEG>
constexpr bool kSkipPad = E >= 12 || (SEG ? E >= 10 && kMH<V> && !kSL<V> : !kSL<V> || (kCM<V> && KS == 8 && kMH<V>));

// more = false: past the last visit, everything through buffers of no bytes
// (early requests are unconditional, see the waits below).  EXACT: a segment is
// KS steps.
template <typename IO, int BL, int L, int V, int KS, bool GV, bool ST, bool SEG, bool EXACT>
__device__ __forceinline__ void load_visit(const BwdArgs& ba, const LaneOff& lo, const VisitAt& c, bool more,
                                           VisitRaw<IO, BL * kKC<V>, KS, kCM<V>, ST, kSL<V>>& r) {
  constexpr int E = BL * kKC<V>;
  const ScanArgs& a = ba.s;
  // The state checkpointed before the segment, where a run starts from it (else a
  // buffer of no bytes: zeros, as for the first segment).
  const bool ck = more && c.seg > 0 && (SEG || c.i == 0 || c.pre);
  const int64_t at_ck = ck ? int64_t(c.seg - 1) * a.N + c.n0 : 0;
  const uint32_t nb = uniform_u32(ck ? 0xFFFFFFFFu : 0u);
  if constexpr (!kSL<V>)
    bload_vec<E>(make_rsrc(uniform_ptr(ba.ckpt + at_ck * a.P), nb), lo.c, r.v0);
  r.h0 = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(make_rsrc(uniform_ptr(ba.ckh + at_ck), nb), lo.v, 0, kAuxNT));
  const int64_t row = int64_t(c.c0) * a.N;
  load_chunk_raw<IO, E, KS, kCM<V>, GV, ST, true>(a, lo, static_cast<const IO*>(a.x) + c.nx0 + row * a.P,
                                                  static_cast<const IO*>(ba.gspk) + c.n0 + row,
                                                  ba.gvz + c.n0 + row, ba.gvn, r.in, !more ? 0 : (EXACT ? KS : c.cs),
                                                  SEG || c.i == c.j);
}

template <typename IO, int BL, int L, int V, int KS, bool FAST, bool ST, bool SEG, bool EXACT>
__device__ __forceinline__ void visit_items(const BwdArgs& ba, const LaneOff& lo, const Branches<BL, kKC<V>>& br,
                                            float alpha, int64_t bt0, int nk, Accum<BL, BL * kKC<V>>& acc,
                                            uint32_t* stage, float* bnd) {
  static_assert(SEG || !EXACT, "exact segments are one chunk each");
  constexpr int E = BL * kKC<V>;
  constexpr int W = kRawW<IO, E, kCM<V>>;
  constexpr int SE = kSL<V> ? 0 : E;  // compartment states kept per slot
  constexpr bool kEarly = kEarlyVisit<IO, V>;
  constexpr bool kSkip = !EXACT && kSkipPad<E, V, KS, SEG>;
  using Raw = VisitRaw<IO, E, KS, kCM<V>, ST, kSL<V>>;
  const ScanArgs& a = ba.s;
  const float beta_r = ba.detach ? 0.0f : a.beta;
  const int nseg = (int(a.T) + a.K - 1) / a.K;
  const Walk wk = make_walk<L, kCM<V>>(a, int64_t(a.ways) * a.M);
  int todo = wk.nw * nk;  // neurons whose last visit is still to be requested
  if (todo <= 0) return;
  const int bsh = a.bsh;
  bnd += threadIdx.x;
  VisitAt ld{bt0 * a.M, bt0 * a.M * a.P, nseg - 1, 0, 0, 0, 0, 0, true, true, false};
  enter_segment<KS, SEG, true>(a, ld);
  VisitAt cp = ld;
  Raw cur;
  load_visit<IO, BL, L, V, KS, !FAST, ST, SEG, EXACT>(ba, lo, ld, true, cur);
  todo -= next_visit<KS, SEG>(a, wk, nseg, ld) ? 1 : 0;
  // Every later wait is then counted from loads issued inside the loop, which
  // are unconditional (past the last visit, rows of no bytes).
  __builtin_amdgcn_s_waitcnt(kWaitVmem);
  BwdLane<IO, E> bl;
  bl.dh_next = 0.0f;
  bl.stage = stage;
  float v[E], h = 0.0f;  // state before the visit's chunk
#pragma unroll
  for (int j = 0; j < E; ++j) bl.lam[j] = v[j] = 0.0f;
  bool s = false;
  auto visit = [&](const Raw& in, bool more, Raw& nxt) {
    if (SEG || cp.first) {
      if (SEG || cp.i == 0 || cp.pre) {
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = kSL<V> ? 0.0f : in.v0[kSL<V> ? 0 : j];
        h = in.h0;
        s = cp.seg > 0 && h >= a.vth;
      } else {
        const float* b = bnd + ((cp.i >> bsh) - 1) * ((SE + 1) * kThreads);
#pragma unroll
        for (int j = 0; j < SE; ++j) v[j] = b[j * kThreads];
        h = b[SE * kThreads];
        s = h >= a.vth;
      }
    }
    if (!SEG && cp.pre) {  // chunk 0, read here
      const IO* xr = static_cast<const IO*>(a.x) + cp.nx0 + int64_t(cp.seg) * a.K * (a.N * a.P);
#pragma unroll 1
      for (int t = cp.seg * a.K; t < cp.c0; ++t, xr += a.N * a.P) {
        uint32_t raw[W];
        float xv[E];
        bload_raw<IO, E, kCM<V>>(make_rsrc(xr), lo.x, a.xes, raw);
        raw_to_float<IO, E>(raw, xv);
        const float z = dendrite_step<BL, L, V, FAST>(v, xv, br, alpha);
        soma_step(h, s, z, a.beta, a.vth);
      }
    }
    float xin[KS][E], gsv[KS], gvv[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      uint32_t raw[W];
      slot_to_lane<W, ST>(in.in.x[k], stage, raw);
      raw_to_float<IO, E>(raw, xin[k]);
      gsv[k] = raw_to_float<IO>(in.in.gs[k]);
      gvv[k] = FAST ? 0.0f : in.in.gv[k];
    }
    auto request = [&] {
      load_visit<IO, BL, L, V, KS, !FAST, ST, SEG, EXACT>(ba, lo, ld, more, nxt);
      todo -= next_visit<KS, SEG>(a, wk, nseg, ld) ? 1 : 0;
    };
    if (kEarly) request();
    __builtin_amdgcn_sched_barrier(0);
    if (SEG || cp.i == cp.j) {
      if ((SEG || cp.last) && cp.seg == nseg - 1) {  // the neuron's last chunk: nothing after it
        bl.dh_next = 0.0f;
#pragma unroll
        for (int j = 0; j < E; ++j) bl.lam[j] = 0.0f;
      }
      IO* const gx = static_cast<IO*>(ba.gx) + cp.nx0 + int64_t(cp.c0) * (a.N * a.P);
      Stash<BL, KS, V, (KS <= 4 || sizeof(IO) == 4)> st;
      recompute_chunk<BL, L, V, KS, FAST, kSkip>(a, br, alpha, v, h, s, xin, st, cp.cs);
      reverse_chunk<IO, BL, L, V, KS, !EXACT, ST>(ba, lo, br, alpha, beta_r, gx, st, gsv, gvv, bl, acc, cp.cs);
      if (cp.seg == 0 && (SEG || cp.j == 0)) fold_item<BL, E>(ba, acc);  // the neuron's first step is done
    } else {
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        if (k >= cp.cs) continue;
        const float z = dendrite_step<BL, L, V, FAST>(v, xin[k], br, alpha);
        soma_step(h, s, z, a.beta, a.vth);
      }
      const int n = cp.i + 1;  // the chunk that starts here
      if (n < cp.j && (n >> bsh) << bsh == n) {  // (chunk j is next: its state is here)
        float* b = bnd + ((n >> bsh) - 1) * ((SE + 1) * kThreads);
#pragma unroll
        for (int j = 0; j < SE; ++j) b[j * kThreads] = v[j];
        b[SE * kThreads] = h;
      }
    }
    next_visit<KS, SEG>(a, wk, nseg, cp);
    if (!kEarly) __builtin_amdgcn_sched_barrier(0);
    if (!kEarly && more) request();
  };
  for (bool more = true; more;) {
    more = todo > 0;
    Raw nxt;
    visit(cur, more, nxt);
    cur = nxt;
  }
}

// The registers of a stateful wide visit in flight (its X rows and
// checkpointed state travel to LDS): grad_spikes, grad_v_soma and H before the
// segment.
template <int KS>
struct SegSmall {
  uint32_t gs[KS];
  float gv[KS];
  float h0;  // somatic potential before the segment (0 for the first)
};

// Requests visit c: X rows and, where a run starts from it, the checkpointed
// compartment state into `area` (rows past the chunk's end are not fetched), the
// rest into r.
template <typename IO, int BL, int V, int KS, bool FAST>
__device__ __forceinline__ void issue_wide_visit(const BwdArgs& ba, const LaneOff& lo, const VisitAt& c,
                                                 uint32_t* area, SegSmall<KS>& r) {
  constexpr int W = BL * kKC<V>;
  constexpr int RD = kDmaDw<W>;
  const ScanArgs& a = ba.s;
  const int64_t rowX = a.N * a.P;
  const IO* x = static_cast<const IO*>(a.x) + c.nx0;
  const IO* g = static_cast<const IO*>(ba.gspk) + c.n0;
  const bool rev = c.i == c.j;
#pragma unroll
  for (int k = 0; k < KS; ++k) {
    const bool real = k < c.cs;
    const int t = real ? c.c0 + k : c.c0;
    if (real) dma_pieces<W>(make_rsrc(x + int64_t(t) * rowX), lo.xw, area + k * RD);
    r.gs[k] = __builtin_amdgcn_raw_buffer_load_b32(
        make_rsrc(g + int64_t(t) * a.N, uniform_u32(real && rev ? 0xFFFFFFFFu : 0u)), lo.s, 0, kAuxNT);
    r.gv[k] = FAST ? 0.0f
                   : __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                         make_rsrc(ba.gvz + c.n0 + int64_t(t) * a.N, uniform_u32(real && rev ? ba.gvn : 0u)), lo.v, 0,
                         kAuxNT));
  }
  const bool ck = c.seg > 0 && c.i == 0;
  if (ck) dma_pieces<W>(make_rsrc(ba.ckpt + (int64_t(c.seg - 1) * a.N + c.n0) * a.P), lo.xw, area + KS * RD);
  const float* hp = uniform_ptr(ck ? ba.ckh + int64_t(c.seg - 1) * a.N + c.n0 : ba.gvz);
  r.h0 = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(make_rsrc(hp, uniform_u32(ck ? 0xFFFFFFFFu : 0u)),
                                                                lo.v, 0, kAuxNT));
}

// The stateful dendrite's wide fp32 lanes (a lane row of more than 16 bytes,
// e.g. ten compartments): pipelined over the lane's visits in visit_items'
// order, but the next visit's X rows and checkpointed compartment state travel
// by LDS DMA (dma_pieces) into the wave's LDS area, where they wait without
// registers: the stash of a wide stateful neuron leaves none for rows in flight.
// The small per-neuron rows (grad_spikes, grad_v_soma, the checkpointed H) ride
// in registers, and grad_x leaves as whole pieces through the wave's `stage`
// buffer (store_gx_staged).  The dendritic adjoint lam and dH cross chunk and
// segment boundaries in reverse time within one neuron and restart at its last
// chunk.  Rows past a short chunk's end are not fetched: the recompute runs over
// whatever the area holds there, and the adjoint pass skips those steps.
// MULTI: segments may hold several chunks.  Every run to a chunk then starts at
// the segment's start (no slots: the plan's bsh keeps none), its state in
// registers; with one chunk a segment (MULTI = false) none is carried.
template <typename IO, int BL, int L, int V, int KS, bool FAST, bool MULTI>
__device__ __forceinline__ void dma_visit_items(const BwdArgs& ba, const LaneOff& lo, const Branches<BL, kKC<V>>& br,
                                                float alpha, int64_t bt0, int nk, Accum<BL, BL * kKC<V>>& acc,
                                                uint32_t* area, uint32_t* stage) {
  constexpr int E = BL * kKC<V>;
  constexpr int W = E;               // fp32 rows: one dword per compartment
  constexpr int RD = kDmaDw<W>;      // LDS dwords per staged row
  static_assert(sizeof(IO) == 4 && !kSL<V> && !kCM<V>, "stateful wide fp32 lanes only");
  const ScanArgs& a = ba.s;
  const float beta_r = ba.detach ? 0.0f : a.beta;
  const int nseg = (int(a.T) + a.K - 1) / a.K;
  const Walk wk = make_walk<L, kCM<V>>(a, int64_t(a.ways) * a.M);
  int todo = wk.nw * nk;  // neurons whose last visit is still to be requested
  if (todo <= 0) return;
  VisitAt ld{bt0 * a.M, bt0 * a.M * a.P, nseg - 1, 0, 0, 0, 0, 0, true, true, false};
  enter_segment<KS, !MULTI, false>(a, ld);
  VisitAt cp = ld;
  SegSmall<KS> cur;
  issue_wide_visit<IO, BL, V, KS, FAST>(ba, lo, ld, area, cur);
  todo -= next_visit<KS, !MULTI, false>(a, wk, nseg, ld) ? 1 : 0;
  BwdLane<IO, E> bl;
  bl.stage = stage;
  bl.dh_next = 0.0f;
  const uint32_t lane = __lane_id();
  float v[E], h = 0.0f;  // state before the visit's chunk
#pragma unroll
  for (int j = 0; j < E; ++j) bl.lam[j] = v[j] = 0.0f;
  bool s = false;
  for (bool more = true; more;) {
    const bool rev = !MULTI || cp.i == cp.j;
    if (rev && cp.last && cp.seg == nseg - 1) {  // the neuron's last chunk: nothing after it
      bl.dh_next = 0.0f;
#pragma unroll
      for (int j = 0; j < E; ++j) bl.lam[j] = 0.0f;
    }
    // this visit's pieces are in the area once every vector memory access of
    // the wave has completed
    __builtin_amdgcn_s_waitcnt(kWaitVmem);
    asm volatile("" ::: "memory");
    float xin[KS][E];
#pragma unroll
    for (int k = 0; k < KS; ++k)
#pragma unroll
      for (int j = 0; j < E; ++j) xin[k][j] = __uint_as_float(area[k * RD + lane * W + j]);
    if (!MULTI || cp.first) {
      const bool from_ckpt = cp.seg > 0;
#pragma unroll
      for (int j = 0; j < E; ++j) {  // (read unconditionally; the first segment starts from 0)
        const float w = __uint_as_float(area[KS * RD + lane * W + j]);
        v[j] = from_ckpt ? w : 0.0f;
      }
      h = cur.h0;
      s = from_ckpt && h >= a.vth;
    }
    float gsv[KS], gvv[KS];
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      gsv[k] = __uint_as_float(cur.gs[k]);
      gvv[k] = cur.gv[k];
    }
    // the area is refilled only after these reads have completed
    __builtin_amdgcn_s_waitcnt(kWaitLds);
    asm volatile("" ::: "memory");
    more = todo > 0;
    if (more) {
      issue_wide_visit<IO, BL, V, KS, FAST>(ba, lo, ld, area, cur);
      todo -= next_visit<KS, !MULTI, false>(a, wk, nseg, ld) ? 1 : 0;
    }
    if (rev) {
      Stash<BL, KS, V> st;
      recompute_chunk<BL, L, V, KS, FAST>(a, br, alpha, v, h, s, xin, st);
      IO* const gx = static_cast<IO*>(ba.gx) + cp.nx0 + int64_t(cp.c0) * (a.N * a.P);
      reverse_chunk<IO, BL, L, V, KS, true, true>(ba, lo, br, alpha, beta_r, gx, st, gsv, gvv, bl, acc, cp.cs);
    } else {
#pragma unroll
      for (int k = 0; k < KS; ++k) {
        if (k >= cp.cs) continue;
        const float z = dendrite_step<BL, L, V, FAST>(v, xin[k], br, alpha);
        soma_step(h, s, z, a.beta, a.vth);
      }
    }
    next_visit<KS, !MULTI, false>(a, wk, nseg, cp);
  }
}

// Per channel the backward produces W = 2 B + P parameter gradients, in the
// order g_kappa [B], g_xi [P], g_zeta [B].  Partial slot p of output o of
// channel c lives output-major ([C W][slots], read by one wave per output) when
// there are many slots, slot-major ([slots][C W], one thread per output) when
// there are few.
__device__ __forceinline__ int64_t partial_index(const BwdArgs& ba, int64_t c, int o, int64_t p) {
  const int W = 2 * ba.s.B + ba.s.P;
  const int64_t g = c * W + o;
  return ba.wide ? g * ba.slots + p : p * (ba.s.C * W) + g;
}

// A lane has 2 BL + E accumulators, v = 0, 1, ...: g_kappa of its BL branches,
// g_xi of its E compartments, g_zeta of its branches.
// Channel output o (0 .. W-1) -> (lane-in-neuron sub, accumulator index v).
template <int BL, int E>
__device__ __forceinline__ void output_source(int o, int B, int P, int* sub, int* v) {
  if (o < B) {
    *sub = o / BL; *v = o % BL;
  } else if (o < B + P) {
    *sub = (o - B) / E; *v = BL + (o - B) % E;
  } else {
    *sub = (o - B - P) / BL; *v = BL + E + (o - B - P) % BL;
  }
}

// Block reduction of the folded float64 sums (spatial tiles), in a fixed order: 16
// lanes per output.  A partial leaves as two floats, its value and what rounding
// that left over, in two adjacent slots, so the sum over slots loses nothing.
template <int BL, int E, int L>
__device__ __forceinline__ void reduce_folded(const BwdArgs& ba, const Pos& pos) {
  const ScanArgs& a = ba.s;
  const int B = a.B, P = a.P, W = 2 * B + P;
  const double* d = fold_sums(ba);
  const int r = threadIdx.x & 15;
  __syncthreads();
  for (int o = threadIdx.x >> 4; o < W + 2; o += kThreads / 16) {
    int sub = 0, v = 2 * BL + E + (o - W), step = o == W ? 1 : L;  // g_alpha: every lane; g_beta: the neuron's first
    if (o < W) output_source<BL, E>(o, B, P, &sub, &v);
    double s = 0.0;
    for (int q = r * step; q < kThreads; q += 16 * step) s += d[v * kThreads + q + sub];
#pragma unroll
    for (int off = 8; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (r == 0) {
      const float hi = float(s);
      const float lo = __builtin_isinf(hi) ? 0.0f : float(s - double(hi));  // (an overflowed sum stays infinite)
      if (o < W) {
        const int64_t p = 2 * (int64_t(pos.g) * a.tpc + pos.tile % a.tpc);
        ba.wsP[partial_index(ba, pos.c, o, p)] = hi;
        ba.wsP[partial_index(ba, pos.c, o, p + 1)] = lo;
      } else {
        float* w = (o == W ? ba.wsA : ba.wsB) + 2 * (int64_t(pos.g) * a.ntiles + pos.tile);
        w[0] = hi;
        w[1] = lo;
      }
    }
  }
}

// Block reduction of the parameter-gradient partials, in a fixed order.
template <int BL, int E, int L>
__device__ __forceinline__ void reduce_partials(const BwdArgs& ba, const Pos& pos, Accum<BL, E>& acc) {
  const ScanArgs& a = ba.s;
  __shared__ float red[kThreads * E];
  __shared__ float reda[kThreads / 64];
  __shared__ float redb[kThreads / 64];
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int B = a.B, P = a.P, W = 2 * B + P;

  float va = acc.a, vb = acc.b;
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
    va += __shfl_xor(va, off);
    vb += __shfl_xor(vb, off);
  }
  if (lane == 0) {
    reda[wave] = va;
    redb[wave] = vb;
  }

  if (a.mode == kSpatial) {
    // One channel per block: sum lanes of equal sub within the wave, then waves.
    const int64_t c = pos.c;
    const int64_t jt = pos.tile % a.tpc;
    auto sum = [&](int v, float x) {
#pragma unroll
      for (int off = 32; off >= L; off >>= 1) x += __shfl_xor(x, off);
      if (lane < L) red[(v * 4 + wave) * L + lane] = x;
    };
#pragma unroll
    for (int j = 0; j < BL; ++j) sum(j, acc.k[j]);
#pragma unroll
    for (int i = 0; i < E; ++i) sum(BL + i, acc.xi[i]);
#pragma unroll
    for (int j = 0; j < BL; ++j) sum(BL + E + j, acc.z[j]);
    __syncthreads();
    for (int o = tid; o < W; o += kThreads) {
      int sub, v;
      output_source<BL, E>(o, B, P, &sub, &v);
      float sum = 0.0f;
      for (int w = 0; w < 4; ++w) sum += red[(v * 4 + w) * L + sub];
      ba.wsP[partial_index(ba, c, o, int64_t(pos.g) * a.tpc + jt)] = sum;
    }
  } else {
    // Whole channels per tile: sum the batch ways and the S positions of each
    // channel, one accumulator kind (kappa, xi, zeta) at a time.
    // o0, wq: the kind's first output and number of outputs per channel
    auto kind = [&](const auto& vals, int o0, int wq) {
      constexpr int nq = sizeof(vals) / sizeof(float);  // accumulators of this kind per lane
#pragma unroll
      for (int j = 0; j < nq; ++j) red[tid * E + j] = vals[j];
      __syncthreads();
      for (int o = tid; o < a.cpt * wq; o += kThreads) {
        const int slot = o / wq, ol = o % wq;
        const int64_t c = pos.tile * a.cpt + slot;
        if (c >= a.C) continue;
        const int sub = ol / nq, j = ol % nq;
        float sum = 0.0f;
        for (int w = 0; w < a.ways; ++w)
          for (int sp = 0; sp < a.S; ++sp) {
            const int thr = (w * a.pb + slot * int(a.S) + sp) * L + sub;
            sum += red[thr * E + j];
          }
        ba.wsP[partial_index(ba, c, o0 + ol, pos.g)] = sum;
      }
      __syncthreads();
    };
    kind(acc.k, 0, B);
    kind(acc.xi, B, P);
    kind(acc.z, B + P, B);
  }
  __syncthreads();
  if (tid == 0) {
    ba.wsA[int64_t(pos.g) * a.ntiles + pos.tile] = (reda[0] + reda[1]) + (reda[2] + reda[3]);
    ba.wsB[int64_t(pos.g) * a.ntiles + pos.tile] = (redb[0] + redb[1]) + (redb[2] + redb[3]);
  }
}

// Which pipeline a backward kernel runs: every neuron one chunk of exactly KS
// steps, one chunk of at most KS, visits over the chunks of segments, or over
// segments that are one chunk each, of at most or of exactly KS steps.
enum BwdPath { kOneChunk = 0, kPartChunk = 1, kVisits = 2, kSegments = 3, kExactSegments = 4 };

// The stateful dendrite's wide fp32 lanes move their rows by LDS DMA
// (dma_visit_items).
template <typename IO, int E, int V>
constexpr bool kWideSF = kWideRow<IO, E, kCM<V>> && !kSL<V> && sizeof(IO) == 4;

// The backward of the lane's neurons.  ST: wide rows staged (see load_pieces;
// lo.xw is the wave's stretch).
template <typename IO, int BL, int L, int V, int KS, int PATH, bool FAST, bool ST>
__device__ __forceinline__ void bwd_run(const BwdArgs& ba, const LaneOff& lo, const Branches<BL, kKC<V>>& br,
                                        float alpha, int64_t bt0, int nk, Accum<BL, BL * kKC<V>>& acc,
                                        uint32_t* stage, float* bnd) {
  if constexpr (PATH >= kVisits)
    visit_items<IO, BL, L, V, KS, FAST, ST, (PATH != kVisits), PATH == kExactSegments>(ba, lo, br, alpha, bt0, nk, acc,
                                                                                     stage, bnd);
  else
    single_chunk_items<IO, BL, L, V, KS, FAST, ST, PATH == kPartChunk>(ba, lo, br, alpha, bt0, nk, acc, stage);
}

// One pipeline a kernel, so that each has the registers it needs: with all of
// them in one kernel, the longest-lived one set the occupancy of every other.
// FAST (no mask and no grad_v_soma): no per-step gate select and no branch for grad_v_soma
// requests (bf16 ImageNet-stem layer: 434 -> 396 VALU instructions per neuron;
// bf16 backward 1-2 % faster without the empty loads).
// One chunk of up to eight steps gets a third wave per SIMD, seven to nine registers
// spilled where a lane holds four compartments: channel-major bf16 rows 157 -> 138 us
// (six steps), but compartments-innermost fp32 rows, sixteen branches, eight steps 70
// -> 74, so those keep two.
template <typename IO, int E, bool CM, int KS, int PATH, bool FAST>
constexpr int kBwdWaves = E * KS <= 8 ? 4
                          : E * KS <= 16 || (FAST && PATH == kPartChunk && (E <= 3 || (E == 4 && (sizeof(IO) == 2 || CM)))) ? 3 : 2;

template <typename IO, int BL, int L, int V, int KS, int PATH, bool FAST>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(kBwdWaves<IO, BL * kKC<V>, kCM<V>, KS, PATH, FAST>))) dendsn_bwd_kernel(BwdArgs ba) {
  constexpr int E = BL * kKC<V>;
  constexpr int W = kRawW<IO, E, kCM<V>>;
  // Staged wide rows (see load_pieces) for the Stateless Dendrite's pipelines:
  // the stateful dendrite's stash of a wide lane left no room for the pieces
  // (its staged short-sequence copy spilled in the loop).
  constexpr bool kWide = kWideRow<IO, E, kCM<V>> && kSL<V>;
  constexpr bool kDma = kWideSF<IO, E, V>;
  if (ba.s.beta_p) ba.s.beta = ba.s.beta_p[0];  // learnable (PLIF) decay
  const ScanArgs& a = ba.s;
  const Pos pos = locate<L>(a);
  const bool full = (kWide || kDma) && __all(pos.active);
  Accum<BL, E> acc;
#pragma unroll
  for (int j = 0; j < BL; ++j) acc.k[j] = acc.z[j] = 0.0f;
#pragma unroll
  for (int i = 0; i < E; ++i) acc.xi[i] = 0.0f;
  acc.a = 0.0f;
  acc.b = 0.0f;
  if (!kDma && ba.fold) {
#pragma unroll
    for (int i = 0; i < kFoldValues<BL, E>; ++i) fold_sums(ba)[i * kThreads + threadIdx.x] = 0.0;
  }
  if (pos.active) {
    Branches<BL, kKC<V>> br;
    load_branches<BL, kKC<V>>(a, pos.c, pos.sub, br);
    const float alpha = a.alpha ? a.alpha[0] : 0.0f;
    LaneOff lo = lane_offsets<IO, E, kCM<V>>(a, pos);
    int64_t bt0;
    const int nk = items_of(a, pos, &bt0);
    extern __shared__ __align__(16) float slots[];
    float* bnd = slots;  // chunk-start states of segments longer than KS (see visit_items)
    bool done = false;
    if constexpr (kWide) {
      __shared__ uint32_t stage[kThreads / 64][64 * W];
      lo.xw = __builtin_amdgcn_readfirstlane(lo.x);
      if (full && stage_rows<IO>(a, lo.xw, bt0)) {
        bwd_run<IO, BL, L, V, KS, PATH, FAST, true>(ba, lo, br, alpha, bt0, nk, acc, stage[threadIdx.x >> 6], bnd);
        done = true;
      }
    }
    if constexpr (kDma) {
      __shared__ uint32_t area[kThreads / 64][(KS + 1) * kDmaDw<W>];   // rows in flight
      __shared__ uint32_t stage_sf[kThreads / 64][64 * W];              // grad_x leaving
      // lane visits of long segments keep their slots in the area (5 E >= 4 (E + 1)
      // dwords a lane); the DMA visits keep none, so a block has one or the other
      bnd = reinterpret_cast<float*>(area);
      const uint32_t span = __builtin_amdgcn_readfirstlane(lo.x);
      if (full && a.K <= kDmaChunks * KS && stage_rows<IO>(a, span, bt0)) {
        lo.xw = span;
        dma_visit_items<IO, BL, L, V, KS, FAST, PATH == kVisits>(ba, lo, br, alpha, bt0, nk, acc,
                                                                 area[threadIdx.x >> 6], stage_sf[threadIdx.x >> 6]);
        done = true;
      }
    }
    if (!done) bwd_run<IO, BL, L, V, KS, PATH, FAST, false>(ba, lo, br, alpha, bt0, nk, acc, nullptr, bnd);
  }
  if (!kDma && ba.fold) {  // (block-uniform)
    reduce_folded<BL, E, L>(ba, pos);
    return;
  }
  if (pos.sub != 0) acc.b = 0.0f;  // the soma runs in every lane of a neuron: count it once
  // every thread of the block reaches this one call (it holds block barriers)
  reduce_partials<BL, E, L>(ba, pos, acc);
}

template <typename IO, int BL, int L, int V, int KS>
hipError_t launch_bwd(const Plan& pl, const BwdArgs& ba, hipStream_t stream) {
  const dim3 grid(static_cast<unsigned>(pl.ntiles * pl.G));
  const bool fast = !ba.s.mask && !ba.gv;
#define DENDSN_BWD(PATH, FAST) \
  { \
    dendsn_bwd_kernel<IO, BL, L, V, KS, PATH, FAST><<<grid, dim3(kThreads), pl.lds, stream>>>(ba); \
    return hipGetLastError(); \
  }
  constexpr int E = BL * kKC<V>;
  if constexpr (!kWideSF<IO, E, V>) {
    if (ba.s.T <= KS) {
      if constexpr (KS == 4) {
        if (ba.s.T == KS && fast) DENDSN_BWD(kOneChunk, true)
        if (ba.s.T == KS) DENDSN_BWD(kOneChunk, false)
        // One to three steps: one copy for all (a tenth of the time is at stake; as
        // segments of a checkpointed sequence they took up to 25 % longer).
        DENDSN_BWD(kPartChunk, false)
      } else {
        if (fast) DENDSN_BWD(kPartChunk, true)
        DENDSN_BWD(kPartChunk, false)
      }
    }
    // Whole segments of narrow stateful bf16 lanes, without the padding's branches
    // (16 steps, K = 4, four branches: 234 against 249 us; K = 8, two branches of
    // two: 222 against 261).  Wider and fp32 lanes spill there (ten bf16
    // compartments 926 against 340 us; 64 steps fp32, K = 8: 234 against 227).
    if constexpr (sizeof(IO) == 2 && !kSL<V> && !kCM<V> && E <= 4)
      if (fast && ba.s.K == KS && ba.s.T % KS == 0) DENDSN_BWD(kExactSegments, true)
  }
  // (channel-major eight-step segments are faster as visits: 16 steps, K = 8, fp32
  // 214 against 242 us)
  if constexpr (!(kCM<V> && KS == 8))
    if (ba.s.K <= KS) {
      if (fast) DENDSN_BWD(kSegments, true)
      DENDSN_BWD(kSegments, false)
    }
  // (eight bf16 branches run longer segments over two lanes, unless those have too
  // many tiles for the fixed scratch: rare, so one kernel with and without gates)
  constexpr bool kRare = BL == 8 && L == 1 && kKC<V> == 1;
  if constexpr (KS == 8 || !long_stash(BL, L, kKC<V>, kCM<V>)) {
    if constexpr (!kRare)
      if (fast) DENDSN_BWD(kVisits, true)
    DENDSN_BWD(kVisits, false)
  }
  return hipErrorInvalidValue;  // (the plan gives segments above 4 steps a mapping and stash compiled for them)
#undef DENDSN_BWD
}

// Fixed-order float64 sum of the partials into the parameter gradients;
// blocks 0 and 1 reduce g_alpha and g_beta.
__global__ void __launch_bounds__(kThreads) dendsn_finalize_kernel(FinArgs f);

}  // namespace dendsn
