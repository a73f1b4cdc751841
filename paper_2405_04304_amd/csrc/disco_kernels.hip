// gfx950 (MI355X) kernels of the DISCO speculative-decoding hot path.
//
// Data layout shared by the kernels
//   * packed weights: 1 KiB tiles of 16 rows x 32 columns in the operand order of
//     v_mfma_f32_16x16x32_bf16 (lane l holds row l % 16, columns 8 * (l / 16) .. + 7), tiles of one
//     16-row group contiguous along K.  A wavefront fetches a tile with one 128-bit load per lane,
//     1 KiB contiguous, and streams a row group as one contiguous slab.
//   * activation panels ("xpack"): the token side of the same instruction.  Activations stay fp32
//     between kernels in value: each is split into bf16 hi = rne(x) and lo = rne(x - hi), so the
//     bf16 matrix unit reproduces fp32-grade products.  For M <= 8 tokens one panel holds hi in
//     columns 0..7 and lo in columns 8..15 (one MFMA per weight tile); for M <= 16 two panels
//     (hi, lo).  Panel element (column n, k) lives at ((kt * 64) + (k % 32 / 8) * 16 + n) * 8 + k % 8,
//     kt = k / 32, panels K * 16 elements apart.
//   * paged KV: [layer][physical page][K | V][kv head] blocks of page_tokens x d_head bf16; a K block
//     is [token][d_head], a V block is transposed, [d_head][token] (see the attention kernel).
#include "disco_internal.h"
#include <type_traits>

#include <mutex>

namespace disco {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

#define NEG_BIG (-1.0e30f)

// ---------------------------------------------------------------------------------------------
// small device helpers
// ---------------------------------------------------------------------------------------------

__device__ __forceinline__ float bf16_to_f32(bf16_t u) { return __uint_as_float(((uint32_t)u) << 16); }

__device__ __forceinline__ bf16_t f32_to_bf16(float f) {  // round to nearest even (the hardware conversion of gfx950)
  return __builtin_bit_cast(bf16_t, (__bf16)f);
}

// Two floats as bf16 in one word, the first in the low half: one instruction (two scalar conversions are put together with two more;
// in the prompt pass's attention they were a quarter of the vector instructions: 0.4 % of a pass over 3001 tokens).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) float f32x2;
  typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{a, b}), bf16x2));
}
// ... and as bf16 hi + lo
struct HiLo { uint32_t hi, lo; };
__device__ __forceinline__ HiLo split_bf16(float a, float b) {
  HiLo r;
  r.hi = pack_bf16(a, b);
  r.lo = pack_bf16(a - __uint_as_float(r.hi << 16), b - __uint_as_float(r.hi & 0xffff0000u));
  return r;
}

__device__ __forceinline__ bool gated(const uint32_t* gate) {
  return gate != nullptr && __builtin_nontemporal_load(gate) != 0u;
}
// The halt flag's value, requested but not waited for: kernels of the draft loop issue their first
// operand loads behind it and test it just before they would wait for those, so that the flag's round
// trip does not stand in front of every launch of the step (a halted step's launches still end there).
__device__ __forceinline__ uint32_t gate_request(const uint32_t* gate) {
  return gate != nullptr ? __builtin_nontemporal_load(gate) : 0u;
}
// Tests a requested flag (the same in every lane).  The value is opaque up to here: left to itself the compiler compares it, and
// so waits for it, where it is requested, in front of the operand loads.
__device__ __forceinline__ bool flag_set(uint32_t v) {
  asm volatile("" : "+v"(v));
  return __builtin_amdgcn_readfirstlane((int)v) != 0;
}

// Stores and loads of data that another workgroup of the SAME launch reads or has written (COH): agent-scope
// relaxed atomics, which on gfx950 are write-through stores and L2-bypassing loads, coherent across the
// eight XCDs' separate L2s.  Without COH they are plain accesses (the consumer is a later launch).
template <bool COH> __device__ __forceinline__ void st_f4(float* p, float a, float b, float c, float d) {
  if (COH) {
    const unsigned long long v0 = (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
    const unsigned long long v1 = (unsigned long long)__float_as_uint(c) | ((unsigned long long)__float_as_uint(d) << 32);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(reinterpret_cast<unsigned long long*>(p) + 1, v1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
  }
}
template <bool COH> __device__ __forceinline__ float4 ld_f4(const float* p) {
  if (COH) {
    const unsigned long long v0 = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned long long v1 = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p) + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return make_float4(__uint_as_float((uint32_t)v0), __uint_as_float((uint32_t)(v0 >> 32)), __uint_as_float((uint32_t)v1), __uint_as_float((uint32_t)(v1 >> 32)));
  }
  return *reinterpret_cast<const float4*>(p);
}
template <bool COH> __device__ __forceinline__ float ld_f1(const float* p) {
  if (COH) return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return *p;
}
template <bool COH> __device__ __forceinline__ void st_f1(float* p, float v) {
  if (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}
template <bool COH> __device__ __forceinline__ void st_u2(bf16_t* p, uint2 v) {
  if (COH) __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)v.x | ((unsigned long long)v.y << 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *reinterpret_cast<uint2*>(p) = v;
}
template <bool COH> __device__ __forceinline__ void st_h1(bf16_t* p, bf16_t v) {
  if (COH) __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

// Store 4 consecutive-k activations of token m into the packed panels as bf16 hi/lo (LO false: the lo panel has no reader).
template <bool COH = false, bool LO = true>
__device__ __forceinline__ void xpack_put4(bf16_t* X, int KT, int M, int m, int k, HiLo x0, HiLo x1) {
  const int kt = k >> 5, grp = (k & 31) >> 3, e = k & 7;
  const size_t base = ((size_t)kt * 64 + grp * 16) * 8 + e;
  size_t off_hi, off_lo;
  if (M <= 8) { off_hi = base + (size_t)m * 8; off_lo = base + (size_t)(m + 8) * 8; }
  else { off_hi = base + (size_t)m * 8; off_lo = (size_t)KT * 512 + base + (size_t)m * 8; }
  st_u2<COH>(X + off_hi, make_uint2(x0.hi, x1.hi));
  if (LO) st_u2<COH>(X + off_lo, make_uint2(x0.lo, x1.lo));
}
template <bool COH = false, bool LO = true>
__device__ __forceinline__ void xpack_store4(bf16_t* X, int KT, int M, int m, int k, const float* v) {
  xpack_put4<COH, LO>(X, KT, M, m, k, split_bf16(v[0], v[1]), split_bf16(v[2], v[3]));
}

// The products a * ga and b * gb as bf16 hi + lo.  EXACT: lo is what hi leaves of the exact product, else of the product rounded to
// fp32.  Written out because a compiler that may contract decides it by what stands around (see norm_row).
template <bool EXACT>
__device__ __forceinline__ HiLo split_product(float a, float ga, float b, float gb) {
#pragma clang fp contract(off)
  const float x = a * ga, y = b * gb;
  HiLo r;
  r.hi = pack_bf16(x, y);
  const float hx = __uint_as_float(r.hi << 16), hy = __uint_as_float(r.hi & 0xffff0000u);
  r.lo = EXACT ? pack_bf16(fmaf(a, ga, -hx), fmaf(b, gb, -hy)) : pack_bf16(x - hx, y - hy);
  return r;
}

// Wavefront reductions on the DPP cross-lane network (no LDS traffic): xor-1, xor-2 inside quads,
// half-row mirror, row mirror, then row broadcasts 15 and 31; lane 63 ends up with the result, which
// is broadcast through a scalar register.  The combination order is fixed, so sums are reproducible.
#define DPP_QUAD_XOR1 0xB1
#define DPP_QUAD_XOR2 0x4E
#define DPP_ROW_HALF_MIRROR 0x141
#define DPP_ROW_MIRROR 0x140
#define DPP_ROW_ROR8 0x128
#define DPP_ROW_BCAST15 0x142
#define DPP_ROW_BCAST31 0x143

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f(float old, float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(old), __float_as_int(v), CTRL, ROW_MASK, 0xF, false));
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ int dpp_i(int old, int v) {
  return __builtin_amdgcn_update_dpp(old, v, CTRL, ROW_MASK, 0xF, false);
}

__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_f<DPP_QUAD_XOR1, 0xF>(0.f, v);
  v += dpp_f<DPP_QUAD_XOR2, 0xF>(0.f, v);
  v += dpp_f<DPP_ROW_HALF_MIRROR, 0xF>(0.f, v);
  v += dpp_f<DPP_ROW_MIRROR, 0xF>(0.f, v);
  v += dpp_f<DPP_ROW_BCAST15, 0xA>(0.f, v);
  v += dpp_f<DPP_ROW_BCAST31, 0xC>(0.f, v);
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp_f<DPP_QUAD_XOR1, 0xF>(v, v));
  v = fmaxf(v, dpp_f<DPP_QUAD_XOR2, 0xF>(v, v));
  v = fmaxf(v, dpp_f<DPP_ROW_HALF_MIRROR, 0xF>(v, v));
  v = fmaxf(v, dpp_f<DPP_ROW_MIRROR, 0xF>(v, v));
  v = fmaxf(v, dpp_f<DPP_ROW_BCAST15, 0xA>(v, v));
  v = fmaxf(v, dpp_f<DPP_ROW_BCAST31, 0xC>(v, v));
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 63));
}

// Hand-off between workgroups of one launch (split reductions).  Data written by one workgroup and
// read by another inside the same kernel moves with agent-scope relaxed atomic stores / loads: on
// gfx950 these are write-through / L2-bypassing accesses (sc1), coherent across the eight XCDs'
// separate L2s without the L2-wide write-back and invalidate that an agent-scope fence costs.  The
// writers drain their stores (s_waitcnt 0) before the workgroup barrier that precedes the ticket.
__device__ __forceinline__ void st_agent2(float* p, float a, float b) {
  const unsigned long long v = (unsigned long long)__float_as_uint(a) | ((unsigned long long)__float_as_uint(b) << 32);
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float2 ld_agent2(const float* p) {
  const unsigned long long v = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
}
// Ticket of a split reduction: true in every thread of the workgroup that arrives last.
// Ordering: the hand-off data moves with write-through stores and L2-bypassing loads (above), so no cache
// maintenance is needed, and an agent-scope release / acquire on the ticket would add exactly that (an
// L2-wide write-back and invalidate, measured at 8 - 13 us per use on MI355X).  What IS needed is that the
// stores have completed before the ticket is taken (the explicit wait) and that the compiler keeps the
// hand-off accesses on their side of the ticket: the two signal fences are compiler-only barriers.
__device__ __forceinline__ bool last_arrival(int* counter, int n, int* s_flag) {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_s_waitcnt(0);                 // this wavefront's hand-off stores have completed
  __syncthreads();
  if (threadIdx.x == 0) {
    const int t = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *s_flag = (t == n - 1) ? 1 : 0;
    if (t == n - 1) __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next launch
  }
  __syncthreads();
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  return *s_flag != 0;
}

// A value and its partner 16 or 32 lanes away, one half of the wavefront each way round (vector instructions; a shuffle goes through
// the LDS unit).  Lanes that are 16 and 32 apart must be active together.
struct Pair32 { float a, b; };
__device__ __forceinline__ Pair32 swap16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return Pair32{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ Pair32 swap32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return Pair32{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ float half_max(float v) { const Pair32 p = swap32(v); return fmaxf(p.a, p.b); }   // lanes l, l^32
__device__ __forceinline__ float half_sum(float v) { const Pair32 p = swap32(v); return p.a + p.b; }
// Across the four 16-lane rows of a wavefront (lanes l, l^16, l^32, l^48), every lane gets the result.
__device__ __forceinline__ float row4_max(float v) { const Pair32 p = swap16(v); return half_max(fmaxf(p.a, p.b)); }
__device__ __forceinline__ float row4_sum(float v) { const Pair32 p = swap16(v); return half_sum(p.a + p.b); }

// Block-wide sum in a fixed order (deterministic); every thread gets the result.
template <int NT>
__device__ __forceinline__ float block_sum(float v, float* smem /* NT/64 + 1 floats */) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = v;
  __syncthreads();
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < NT / 64; ++i) t += smem[i];
  return t;
}

// (value, index) arg-max: larger value wins, lower index on equal values.
struct VI { float v; int i; };
__device__ __forceinline__ VI vi_best(VI a, VI b) {
  return (b.v > a.v || (b.v == a.v && b.i < a.i)) ? b : a;
}
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ VI vi_step(VI x) {
  VI y; y.v = dpp_f<CTRL, ROW_MASK>(x.v, x.v); y.i = dpp_i<CTRL, ROW_MASK>(x.i, x.i);
  return vi_best(x, y);
}
__device__ __forceinline__ VI wave_argmax(VI x) {
  x = vi_step<DPP_QUAD_XOR1, 0xF>(x);
  x = vi_step<DPP_QUAD_XOR2, 0xF>(x);
  x = vi_step<DPP_ROW_HALF_MIRROR, 0xF>(x);
  x = vi_step<DPP_ROW_MIRROR, 0xF>(x);
  x = vi_step<DPP_ROW_BCAST15, 0xA>(x);
  x = vi_step<DPP_ROW_BCAST31, 0xC>(x);
  VI r;
  r.v = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x.v), 63));
  r.i = __builtin_amdgcn_readlane(x.i, 63);
  return r;
}
template <int NT>
__device__ __forceinline__ VI block_argmax(VI x, float* sv, int* si) {
  x = wave_argmax(x);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) { sv[threadIdx.x >> 6] = x.v; si[threadIdx.x >> 6] = x.i; }
  __syncthreads();
  VI r; r.v = sv[0]; r.i = si[0];
#pragma unroll
  for (int i = 1; i < NT / 64; ++i) { VI y; y.v = sv[i]; y.i = si[i]; r = vi_best(r, y); }
  return r;
}

// ---------------------------------------------------------------------------------------------
// weight packing (one-time layout transform)
// ---------------------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_pack(const bf16_t* __restrict__ src, int64_t n, int64_t k,
                                             bf16_t* __restrict__ dst, int64_t tile_mul, int64_t tile_add) {
  // one thread per 8-element group of the destination
  const int64_t KT = k >> 5;
  const int64_t total = n * k / 8;
  for (int64_t gidx = (int64_t)blockIdx.x * 256 + threadIdx.x; gidx < total; gidx += (int64_t)gridDim.x * 256) {
    const int64_t lane = gidx & 63, tile = gidx >> 6;
    const int64_t rt = tile / KT, kt = tile % KT;
    const int64_t row = rt * 16 + (lane & 15), col = kt * 32 + (lane >> 4) * 8;
    const uint4 v = *reinterpret_cast<const uint4*>(src + row * k + col);
    const int64_t drt = rt * tile_mul + tile_add;
    *reinterpret_cast<uint4*>(dst + ((drt * KT + kt) * 64 + lane) * 8) = v;
  }
}

hipError_t launch_pack(const bf16_t* src, int64_t n, int64_t k, bf16_t* dst, int64_t tile_mul,
                       int64_t tile_add, hipStream_t s) {
  const int64_t total = n * k / 8;
  int64_t blocks = (total + 255) / 256;
  if (blocks > 65536) blocks = 65536;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_pack, dim3((unsigned)blocks), dim3(256), 0, s, src, n, k, dst, tile_mul, tile_add);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// skinny GEMM: weights streamed once from HBM, M <= 16 tokens on the matrix unit's column side
// ---------------------------------------------------------------------------------------------
//
// A work unit is (row group b of RT 16-row tiles, k-tile range [kt_begin, kt_end)).  The NW wavefronts
// of the workgroup interleave over the k-tiles of the range, each keeping U k-tiles of loads in
// flight, and reduce through LDS in a fixed order.  When a row group's K range is covered by n_seg > 1
// units (of different workgroups), each stores its partial 16 x 16 tiles to a plane and takes a
// ticket; the last one to arrive adds the planes in range order and runs the epilogue: no float
// atomics, no waiting, bitwise reproducible results.
//
// k_gemm launches a grid of (row groups, K ranges): every workgroup owns one unit.

// Copies from memory into LDS, 16 bytes per lane to consecutive LDS addresses from `lds` on (uniform), without registers:
// base (uniform) + lane_off, or an address per lane.  Completion is counted by vmcnt.
__device__ __forceinline__ void lds_dma_16(const void* base, const uint32_t lane_off, const uint32_t lds) {
  // m0 holds the LDS address of the wavefront's 1 KiB; the instruction has no register outputs
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds), "v"(lane_off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void lds_dma_16(const void* lane_addr, const uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds), "v"(lane_addr) : "memory", "m0");
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) {
  union { u32x4 u; bf16x8 b; } c; c.u = v; return c.b;
}

// Where the keys and values of a position go: physical page and offset in it.
struct KvSlot { int page, off; };
__device__ __forceinline__ KvSlot kv_slot(const GemmArgs& a, const int pos) {
  const int pt = a.page_tokens;
  const bool pow2 = (pt & (pt - 1)) == 0;
  const int lp = pow2 ? pos >> __builtin_ctz(pt) : pos / pt;
  return KvSlot{a.page_table ? a.page_table[lp] : lp, pos - lp * pt};
}

// QKV epilogue of one lane: output features n0 .. n0+3 (lo4) and their rotary partners n0 + d_head/2 ..
// (hi4) of token row m at position pos: rotation, then the query row or the paged K / V entry.
// ROPE false: the model has no rotation (the LayerNorm family has learned positions).  SLOT: the caller has looked up kv_slot.
// factors: the two table entries, where the caller has loaded them.
template <bool COH = false, bool ROPE = true, bool SLOT = false>
__device__ __forceinline__ void qkv_store(const GemmArgs& a, float* q, const int n0, const int m, const int pos, KvSlot slot,
                                          float (&lo4)[4], float (&hi4)[4], const float4* factors = nullptr) {
  const int dsh = a.dh == 128 ? 7 : 6;            // d_head is 64 or 128
  const int head = n0 >> dsh, c = n0 & (a.dh - 1), half = a.dh >> 1;
  const bool is_v = head >= a.nq + a.nkv;
  if (ROPE && a.rope_tab != nullptr && !is_v) {
    // (cos, sin) of pos * base^(-2 (c + v) / d_head), tabulated per cached position
    const float4* tab = factors != nullptr ? factors : reinterpret_cast<const float4*>(a.rope_tab + ((size_t)pos * half + c) * 2);
    const float4 t0 = tab[0], t1 = tab[1];
    const float cs[4] = {t0.x, t0.z, t1.x, t1.z}, sn[4] = {t0.y, t0.w, t1.y, t1.w};
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float x0 = lo4[v], x1 = hi4[v];
      // which product is rounded is stated here: left to the compiler it differed between the kernels that share this code,
      // so that a query or key depended on the launch structure and on the block's length
      lo4[v] = fmaf(x0, cs[v], -(x1 * sn[v]));
      hi4[v] = fmaf(x1, cs[v], x0 * sn[v]);
    }
  }
  if (head < a.nq) {
    float* qp = q + (size_t)m * a.ldq + head * a.dh + c;
    st_f4<COH>(qp, lo4[0], lo4[1], lo4[2], lo4[3]);
    st_f4<COH>(qp + half, hi4[0], hi4[1], hi4[2], hi4[3]);
  } else {
    const int sel = is_v ? 1 : 0;
    const int kvh = head - a.nq - sel * a.nkv;
    if (!SLOT) slot = kv_slot(a, pos);
    const int off = slot.off, pp = slot.page;
    bf16_t* blk = a.kv_layer + (((size_t)pp * 2 + sel) * a.nkv + kvh) * a.page_tokens * a.dh;
    if (!is_v) {                 // K: [token][d_head]
      bf16_t* dst = blk + (size_t)off * a.dh + c;
      st_u2<COH>(dst, make_uint2(pack_bf16(lo4[0], lo4[1]), pack_bf16(lo4[2], lo4[3])));
      st_u2<COH>(dst + half, make_uint2(pack_bf16(hi4[0], hi4[1]), pack_bf16(hi4[2], hi4[3])));
    } else {                     // V: transposed, [d_head][token]
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        st_h1<COH>(blk + (size_t)(c + v) * a.page_tokens + off, f32_to_bf16(lo4[v]));
        st_h1<COH>(blk + (size_t)(c + half + v) * a.page_tokens + off, f32_to_bf16(hi4[v]));
      }
    }
  }
}

template <int EPI> struct EpiTraits { static constexpr bool pair = (EPI == EPI_QKV || EPI == EPI_SWIGLU); };

// Register buffers (k-tiles in flight per wavefront) by row tiles per unit and activation panels: as many as the
// register file of a workgroup of eight wavefronts holds next to the accumulators; with two panels two buffers
// measured best at every tile count (a same-box sweep over 2 / 3 / 4 at the 13B shapes).
constexpr int gemm_buffers(int rt, int panels) { return panels >= 2 ? 2 : (rt >= 8 ? 3 : 4); }

// LDS of one GEMM work unit.
template <int RT, int NW, bool LN = false>
struct GemmSmem {
  f32x4 red[NW][RT][64];
  float red_ssq[NW][64];
  float red_sum[LN ? NW : 1][64];                 // per-tile sums of a deferred LayerNorm
  alignas(16) float ln[LN ? NW : 1][LN ? 64 : 4];        // its vectors: W . g of a wavefront's two tiles (or one), then W . b
  int s_last;
};

// Row tiles of work unit b: RT consecutive tiles, or RT / 2 pairs (tile, tile + grp) for the two-tile epilogues.
template <int RT, int EPI>
__device__ __forceinline__ void gemm_unit_tiles(const GemmArgs& a, const int b, int (&rt)[RT]) {
  constexpr bool PAIR = EpiTraits<EPI>::pair;
  constexpr int UNITS = PAIR ? RT / 2 : RT;
  if (PAIR) {
#pragma unroll
    for (int u = 0; u < UNITS; ++u) {
      const int bp = b * UNITS + u, gs = __builtin_ctz(a.grp);   // the pairing distance is a power of two
      rt[2 * u] = ((bp >> gs) << (gs + 1)) + (bp & (a.grp - 1));
      rt[(2 * u + 1) % RT] = rt[2 * u] + a.grp;
    }
  } else {
#pragma unroll
    for (int r = 0; r < RT; ++r) rt[r] = b * RT + r;
  }
}

// COH: the unit's inputs were written, and its outputs are read, by other workgroups of the same launch
// (persistent kernel): hand-off accesses instead of plain ones; the activation panels are still plain loads
// (the persistent kernel gives every phase panels at addresses that nobody has read before in the launch).
// `hook` runs once, right after the unit's first weight tiles (two steps per wavefront) have been requested and
// before anything that depends on the unit's inputs is touched: a persistent kernel waits there for the grid
// barrier that ends the phase before, so the weight stream is in flight while that phase drains.
struct NoHook { __device__ __forceinline__ void operator()() const {} };

// LN: the input's norm is a LayerNorm (deferred like the RMSNorm: the panels hold g * h, the producer left per-tile
// sums and sums of squares, and the epilogue applies rstd * (y - mean * wg) + wb).
template <int P, int RT, int EPI, int NW, int U, bool COH = false, typename Hook = NoHook, bool LN = false>
__device__ __forceinline__ void gemm_unit(const GemmArgs& a, const int b, const int kt_begin, const int kt_end,
                                          const int seg, const int n_seg, GemmSmem<RT, NW, LN>& sm, const Hook hook = Hook()) {
  constexpr bool PAIR = EpiTraits<EPI>::pair;
  constexpr int UNITS = PAIR ? RT / 2 : RT;       // output units handled by one wavefront each
  static_assert(!PAIR || RT % 2 == 0, "pair epilogues need an even tile count");
  static_assert(UNITS <= NW, "one epilogue wavefront per unit");
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const uint32_t halted = gate_request(a.gate);
  uint32_t aborted = 0u;                          // requested here, used by the last store
  if (EPI == EPI_STORE) aborted = a.abort_word != nullptr ? __builtin_nontemporal_load(a.abort_word) : 0u;
  int rt[RT];
  gemm_unit_tiles<RT, EPI>(a, b, rt);

  // one accumulator per row tile: with two panels (hi, lo) both products are added into it
  f32x4 acc[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int KT = a.KT;
  const u32x4* Wp[RT];
#pragma unroll
  for (int r = 0; r < RT; ++r) Wp[r] = reinterpret_cast<const u32x4*>(a.W) + (size_t)rt[r] * KT * 64 + lane;
  const u32x4* Xp = reinterpret_cast<const u32x4*>(a.X) + lane;

  // U register buffers, one k-tile each: wavefront w takes k-tiles kt_begin + w, + NW, ...; the loads of the next
  // U - 1 steps are in flight while the matrix unit works on a step (U * RT KiB of weights per wavefront: the
  // stream is bound by the bytes in flight, see the launch shapes below).
  auto load_w = [&](u32x4 (&A)[RT], const int k) {
#pragma unroll
    for (int r = 0; r < RT; ++r) A[r] = __builtin_nontemporal_load(Wp[r] + (size_t)k * 64);
  };
  // Columns without a token are not fetched by the units that many workgroups of a wide matrix read their panels for: a result column
  // depends on its own operand column only, and these are never stored (two multi-query layers, 7 tokens: 414.7 -> 408.8 us; the
  // 16- and 32-row units of the draft models got slower: a 68M draft token 68.4 -> 69.2)
  const bool live_col = RT < 4 || (lane & (P == 1 ? 7 : 15)) < a.M;
  auto load_x = [&](u32x4 (&B)[P], const int k) {
    if (live_col) {
#pragma unroll
      for (int p = 0; p < P; ++p) B[p] = Xp[((size_t)p * KT + k) * 64];
    }
  };
  u32x4 A[U][RT], B[U][P];
  const int kt0 = kt_begin + w;
  // the weights of the first U steps depend on nothing: they go out first
#pragma unroll
  for (int i = 0; i < U; ++i)
    if (kt0 + i * NW < kt_end) load_w(A[i], kt0 + i * NW);
  asm volatile("" ::: "memory");
  hook();
#pragma unroll
  for (int i = 0; i < U; ++i)
    if (kt0 + i * NW < kt_end) load_x(B[i], kt0 + i * NW);
  asm volatile("" ::: "memory");

  // deferred RMSNorm: the panels hold g * h (not normalised).  The producer left one sum of squares
  // per token and 16-column tile; every lane fetches a few of them now (lane = token lane % 16,
  // slots (lane / 16) * NW + w + 4 NW k), the loads complete behind the weight stream, and the
  // epilogue adds them up in a fixed order to get 1 / rms.
  constexpr bool NORMED = (EPI != EPI_PARTIAL);
  constexpr int MAXS = NORMED ? 128 / NW : 1;
  static_assert(!LN || NORMED, "only epilogues that read a normalised input defer a LayerNorm");
  float sv[MAXS], su[LN ? MAXS : 1];
  if (NORMED) {
#pragma unroll
    for (int k = 0; k < MAXS; ++k) sv[k] = 0.f;
    if (LN) {
#pragma unroll
      for (int k = 0; k < MAXS; ++k) su[k] = 0.f;
    }
    // rounds of 4 NW slots; the rounds past n_ssq are skipped by a uniform branch (a 768-wide model
    // needs 2 of the 16 rounds: per-lane tests of all 16 cost more than the loads)
    const int rounds = a.ssq != nullptr ? (a.n_ssq + 4 * NW - 1) / (4 * NW) : 0;
#pragma unroll
    for (int k = 0; k < MAXS; ++k) {
      if (k < rounds) {
        const int idx = (lane >> 4) * NW + w + 4 * NW * k;
        sv[k] = idx < a.n_ssq ? a.ssq[idx * 16 + (lane & 15)] : 0.f;   // [slot][token]; plain loads: see k_forward
        if (LN) su[k] = idx < a.n_ssq ? a.sum[idx * 16 + (lane & 15)] : 0.f;
      }
    }
    asm volatile("" ::: "memory");     // keep these loads ahead of the rest of the stream
  }
  // The vectors of a deferred LayerNorm (and the page of the keys and values) are requested here, by the wavefronts that will use
  // them, so that their round trip runs beside the weight stream instead of behind it (a pass of the multi-query draft model, 12
  // layers, 5 tokens: 360 us behind it, 357 now).  The rotary factors of the RMSNorm family stay behind (a pass over two 13B layers
  // 300.2 us, 300.9 with them here), and so do the residual rows of 64-row PARTIAL units, whose stream is long (6144 rows, K 6144 and
  // 24576, a launch: 34.0 us, 35.9 with them here); 16-row units ask here
  constexpr int TPU = PAIR ? 2 : 1;               // tiles per unit
  const bool ep = w < UNITS;                      // this wavefront finishes one output unit
  const int m = lane & 15, g = lane >> 4;         // token column, 4-row group of the 16x16 result
  int urt[TPU];                                   // its tiles; known here only where they are needed here
#pragma unroll
  for (int i = 0; i < TPU; ++i) {
    urt[i] = 0;
#pragma unroll
    for (int rr = 0; rr < RT; ++rr) if (LN && rr == (ep ? w : 0) * TPU + i) urt[i] = rt[rr];
  }
  // A lane holds one element of the two LayerNorm vectors until the reduction puts them into LDS: the 8 or 16 values that it needs
  // itself would take some instances past 128 registers and so leave one resident workgroup per compute unit instead of two (a
  // pass over two LayerNorm layers of 4096, 384 QKV workgroups: 252.7 us, 257.1 with the values in registers, 254.7 behind the
  // stream).  The instances of two panels and four tiles have no register to spare and ask behind the stream (two layers of 5120,
  // 12 tokens: 378.4 us, 380.5 before it)
  float lnv = 0.f;
  KvSlot slot = {0, 0};
  constexpr bool EARLY = LN && !(P == 2 && RT == 4);
  if (EARLY && ep) lnv = ((lane & 32) ? a.wb : a.wg)[(TPU == 2 && (lane & 16) ? urt[TPU - 1] : urt[0]) * 16 + m];
  if (EPI == EPI_QKV && EARLY && ep && m < a.M && urt[0] * 16 >= a.nq * a.dh) slot = kv_slot(a, a.pos0 + m);
  if (EARLY) asm volatile("" ::: "memory");
  float4 h = make_float4(0.f, 0.f, 0.f, 0.f), gn = h;
  float* hp = nullptr;
  auto load_residual = [&] {                      // (depends on no other workgroup of the launch)
    const int col = (b * RT + (ep ? w : 0)) * 16 + 4 * g;
    hp = a.h + (size_t)m * a.ld_out + col;
    if (ep && m < a.M) {
      h = ld_f4<COH>(hp);
      if (a.Xout != nullptr) gn = *reinterpret_cast<const float4*>(a.gain + col);
    }
  };
  if (EPI == EPI_PARTIAL && RT == 1) {
    load_residual();
    asm volatile("" ::: "memory");
  }
  if (flag_set(halted)) return;                       // uniform over the launch; nothing has been written yet
  for (int kt = kt0; kt < kt_end; kt += U * NW) {
#pragma unroll
    for (int i = 0; i < U; ++i) {
      const int k = kt + i * NW;
      if (k < kt_end) {
#pragma unroll
        for (int p = 0; p < P; ++p)                // panel outside: RT independent instructions between two on one accumulator
#pragma unroll
          for (int r = 0; r < RT; ++r)
            acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(A[i][r]), as_bf16x8(B[i][p]), acc[r], 0, 0, 0);
        const int kn = k + U * NW;                 // the buffer's next k-tile
        if (kn < kt_end) { load_w(A[i], kn); load_x(B[i], kn); }
      }
    }
  }

  if (LN && !EARLY && ep) lnv = ((lane & 32) ? a.wb : a.wg)[(TPU == 2 && (lane & 16) ? urt[TPU - 1] : urt[0]) * 16 + m];
  // hi + lo: same panel, columns n and n + 8 (P == 1), or two panels (P == 2)
  __syncthreads();                                // a previous unit of this workgroup has left the buffers
#pragma unroll
  for (int r = 0; r < RT; ++r) {
    f32x4 y = acc[r];
    if (P == 1) {
#pragma unroll
      for (int v = 0; v < 4; ++v) y[v] = acc[r][v] + dpp_f<DPP_ROW_ROR8, 0xF>(0.f, acc[r][v]);
    }
    sm.red[w][r][lane] = y;
  }
  if (NORMED) {
    float part = 0.f;
#pragma unroll
    for (int k = 0; k < MAXS; ++k) {
      asm volatile("" : "+v"(sv[k]));  // first use of the early loads is here, after the stream
      part += sv[k];
    }
    sm.red_ssq[w][lane] = part;
    if (LN) {
      float ps = 0.f;
#pragma unroll
      for (int k = 0; k < MAXS; ++k) {
        asm volatile("" : "+v"(su[k]));
        ps += su[k];
      }
      sm.red_sum[w][lane] = ps;
      asm volatile("" : "+v"(lnv));
      sm.ln[w][lane] = lnv;
    }
  }
  __syncthreads();
  f32x4 y[TPU];
#pragma unroll
  for (int i = 0; i < TPU; ++i) {
    const int r = (ep ? w : 0) * TPU + i;
    // (runtime index into rt[] would spill it: select with a compile-time loop)
#pragma unroll
    for (int rr = 0; rr < RT; ++rr) if (!LN && rr == r) urt[i] = rt[rr];
    y[i] = sm.red[0][r][lane];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) y[i] += sm.red[ww][r][lane];   // fixed order: deterministic
  }

  if (EPI == EPI_PARTIAL && RT > 1) load_residual();   // ahead of the ticket

  if (n_seg > 1) {
    // this unit covers part of K: store the partial tiles, take a ticket; the last unit of the row
    // group to arrive adds all partial tiles in range order (so the sum does not depend on arrival
    // order) and finishes the row group.  Nobody waits for anybody.
    float* plane = a.planes + ((size_t)b * GEMM_MAX_SPLIT * RT) * 256 + (size_t)lane * 4;
    if (ep) {
#pragma unroll
      for (int i = 0; i < TPU; ++i) {
        float* dst = plane + ((size_t)seg * RT + (w * TPU + i)) * 256;
        st_agent2(dst, y[i][0], y[i][1]);
        st_agent2(dst + 2, y[i][2], y[i][3]);
      }
    }
    if (!last_arrival(a.counters + b, n_seg, &sm.s_last)) return;
    if (ep) {
#pragma unroll
      for (int i = 0; i < TPU; ++i) {
        float2 pa[GEMM_MAX_SPLIT], pb[GEMM_MAX_SPLIT];
#pragma unroll
        for (int sp = 0; sp < GEMM_MAX_SPLIT; ++sp)
          if (sp < n_seg) {
            const float* src = plane + ((size_t)sp * RT + (w * TPU + i)) * 256;
            pa[sp] = ld_agent2(src); pb[sp] = ld_agent2(src + 2);
          }
        y[i] = f32x4{pa[0].x, pa[0].y, pb[0].x, pb[0].y};
#pragma unroll
        for (int sp = 1; sp < GEMM_MAX_SPLIT; ++sp)
          if (sp < n_seg) { y[i][0] += pa[sp].x; y[i][1] += pa[sp].y; y[i][2] += pb[sp].x; y[i][3] += pb[sp].y; }
      }
    }
  }
  if (NORMED && a.ssq != nullptr) {
    float ss = 0.f;
#pragma unroll
    for (int ww = 0; ww < NW; ++ww)
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) ss += sm.red_ssq[ww][gg * 16 + m];
    if (LN) {
      float sx = 0.f;
#pragma unroll
      for (int ww = 0; ww < NW; ++ww)
#pragma unroll
        for (int gg = 0; gg < 4; ++gg) sx += sm.red_sum[ww][gg * 16 + m];
      const float mean = sx / (float)a.d_in;
      const float var = fmaxf(ss / (float)a.d_in - mean * mean, 0.f);
      const float rstd = 1.0f / sqrtf(var + a.eps);
#pragma unroll
      for (int i = 0; i < TPU; ++i) {
        const float4 vg = *reinterpret_cast<const float4*>(&sm.ln[LN ? w : 0][i * 16 + 4 * g]), vb = *reinterpret_cast<const float4*>(&sm.ln[LN ? w : 0][32 + i * 16 + 4 * g]);
        y[i][0] = rstd * (y[i][0] - mean * vg.x) + vb.x; y[i][1] = rstd * (y[i][1] - mean * vg.y) + vb.y;
        y[i][2] = rstd * (y[i][2] - mean * vg.z) + vb.z; y[i][3] = rstd * (y[i][3] - mean * vg.w) + vb.w;
      }
    } else {
      const float rstd = 1.0f / sqrtf(ss / (float)a.d_in + a.eps);
#pragma unroll
      for (int i = 0; i < TPU; ++i) y[i] *= rstd;
    }
  }

  if (EPI == EPI_PARTIAL) {
    // residual-stream update h += X.W^T
    if (!ep || m >= a.M) return;
    const int col = urt[0] * 16 + 4 * g;
    h.x += y[0][0]; h.y += y[0][1]; h.z += y[0][2]; h.w += y[0][3];
    st_f4<COH>(hp, h.x, h.y, h.z, h.w);
    if (a.Xout != nullptr) {
      // feed the next RMSNorm'ed GEMM: panels of gain * h and this tile's sum of squares
      const float o[4] = {h.x * gn.x, h.y * gn.y, h.z * gn.z, h.w * gn.w};
      xpack_store4<COH>(a.Xout, a.KT_out, a.M, m, col, o);
      const float sq = row4_sum((h.x * h.x + h.y * h.y) + (h.z * h.z + h.w * h.w));
      if (g == 0) st_f1<COH>(a.ssq_out + urt[0] * 16 + m, sq);              // [slot][token]
      if (a.sum_out != nullptr) {
        const float sx = row4_sum((h.x + h.y) + (h.z + h.w));
        if (g == 0) st_f1<COH>(a.sum_out + urt[0] * 16 + m, sx);
      }
    }
    return;
  }
  if (!ep || m >= a.M) return;
  if (EPI == EPI_STORE) {
    if (a.only_row >= 0 && m != a.only_row) return;
    const size_t row_off = a.only_row >= 0 ? 0 : (size_t)m * a.ld_out;
    if (flag_set(aborted)) y[0] = f32x4{NAN, NAN, NAN, NAN};   // the forward's data is unusable: say so in its result
    st_f4<COH>(a.out + row_off + urt[0] * 16 + 4 * g, y[0][0], y[0][1], y[0][2], y[0][3]);
  } else if (EPI == EPI_QKV) {
    // two tiles: features c .. c+3 and their rotary partners c + dh/2 .. of one head
    float lo4[4], hi4[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) { lo4[v] = y[0][v]; hi4[v] = y[TPU - 1][v]; }
    qkv_store<COH, !LN, EARLY>(a, a.q, urt[0] * 16 + 4 * g, m, a.pos0 + m, slot, lo4, hi4);
  } else if (EPI == EPI_SWIGLU) {
    // tile 0 = gate rows, tile 1 = the matching up rows
    const int f = (urt[0] >> 1) * 16 + 4 * g;
    float act[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float gt = y[0][v];
      act[v] = gt / (1.0f + expf(-gt)) * y[TPU - 1][v];
    }
    xpack_store4<COH>(a.Xout, a.KT_out, a.M, m, f, act);
  } else if (EPI == EPI_GELU) {
    float act[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) act[v] = 0.5f * y[0][v] * (1.0f + erff(y[0][v] * 0.70710678118654752f));
    xpack_store4<COH>(a.Xout, a.KT_out, a.M, m, urt[0] * 16 + 4 * g, act);
  }
}

// Kernels of the decode path take what their first loads need as separate leading arguments (14 dwords at most; the library is built so that
// these arrive in scalar registers with the launch) and the rest as a structure: read from the argument buffer, all of them stood
// in front of the first load (0.36 us a launch: four tokens of the multi-query draft model 1505 us, 1436 with k_gemm changed).
// `early`: the residual rows (PARTIAL) or the sums of squares of the input.
template <int P, int RT, int EPI, int NW, int U, bool LN = false>
__global__ __launch_bounds__(NW * 64) void k_gemm(const bf16_t* W, const bf16_t* X, const uint32_t* gate, const float* early, int KT,
                                                  int split_or_grp, int n_ssq, int M, const float* sum, GemmArgs a) {
  __shared__ GemmSmem<RT, NW, LN> sm;
  a.W = W; a.X = X; a.gate = gate; a.KT = KT; a.M = M;
  if constexpr (EPI == EPI_PARTIAL) { a.h = const_cast<float*>(early); a.n_split = split_or_grp; }
  else { a.ssq = early; a.n_ssq = n_ssq; a.n_split = 1; a.grp = split_or_grp; if (LN) a.sum = sum; }
  const int n_split = a.n_split;
  const int split = blockIdx.y;
  const int kt_begin = n_split == 1 ? 0 : (int)((unsigned)(KT * split) / (unsigned)n_split);
  const int kt_end = n_split == 1 ? KT : (int)((unsigned)(KT * (split + 1)) / (unsigned)n_split);
  gemm_unit<P, RT, EPI, NW, U, false, NoHook, LN>(a, blockIdx.x, kt_begin, kt_end, split, a.n_split, sm);
  // (behind the unit: a store in front of it would be waited for with its loads)
  if constexpr (EPI == EPI_STORE) {
    if (a.done != nullptr && blockIdx.x == 0 && threadIdx.x == 0) __hip_atomic_store(a.done, a.done_value, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

template <int P, int RT, int EPI, int NW, int U>
static hipError_t launch_gemm_cfg(const GemmArgs& a, hipStream_t s) {
  constexpr int rows = RT * 16;
  if (a.n_rows % rows) return hipErrorInvalidValue;
  if constexpr (EPI == EPI_QKV || EPI == EPI_GELU || EPI == EPI_STORE) {
    if (a.sum != nullptr) {                       // deferred LayerNorm
      hipLaunchKernelGGL((k_gemm<P, RT, EPI, NW, U, true>), dim3(a.n_rows / rows, a.n_split), dim3(NW * 64), 0, s, a.W, a.X, a.gate,
                         EPI == EPI_PARTIAL ? a.h : a.ssq, a.KT, EPI == EPI_PARTIAL ? a.n_split : a.grp, a.n_ssq, a.M, a.sum, a);
      return hipGetLastError();
    }
  }
  hipLaunchKernelGGL((k_gemm<P, RT, EPI, NW, U>), dim3(a.n_rows / rows, a.n_split), dim3(NW * 64), 0, s, a.W, a.X, a.gate,
                         EPI == EPI_PARTIAL ? a.h : a.ssq, a.KT, EPI == EPI_PARTIAL ? a.n_split : a.grp, a.n_ssq, a.M, a.sum, a);
  return hipGetLastError();
}

// Launch shapes, from sweeps on MI355X at the 13B-class and 68M-class sizes.  Eight wavefronts per
// workgroup and one k-tile per wavefront and step (two register buffers) were best everywhere.  The
// activation panels are re-read from L2 by every workgroup, so wide outputs take 64 or 128 rows per
// workgroup; narrow outputs (d_model rows) take 64 rows and split K so that about 480 workgroups are
// in flight, small matrices take 16-row workgroups.
// Share of the chip's 256 compute units that stay busy when `wgs` equal workgroups are spread over them.
static double cu_fill(long wgs) { return wgs <= 0 ? 0.0 : (double)wgs / (256.0 * (double)((wgs + 255) / 256)); }

int gemm_split_for(int n_rows, int KT, int M) {
  (void)M;
  int s;
  if (n_rows % 64 == 0 && n_rows >= 2048) {
    // about 480 workgroups for a short K, about 240 for a long one (fewer, longer streams), but never a count that
    // leaves a large part of the chip idle in the last round (288 workgroups keep 56 % of the units busy, 480 keep 94 %)
    // and not more than two rounds (96 row groups: 480 workgroups measured 1 - 1.5 % better than 768)
    const int groups = n_rows / 64, target = KT > 256 ? 240 : 480;
    double best = -1.0;
    s = 1;
    for (int c = 1; c <= GEMM_MAX_SPLIT && c <= KT / 16; ++c) {
      const long wgs = (long)groups * c;
      if (c > 1 && wgs > 512) break;
      const double dist = (double)(wgs > target ? wgs - target : target - wgs) / target;
      const double score = cu_fill(wgs) - 0.05 * dist;
      if (score > best + 1e-9) { best = score; s = c; }
    }
  } else {
    s = KT / 24;
  }
  return s < 1 ? 1 : (s > GEMM_MAX_SPLIT ? GEMM_MAX_SPLIT : s);
}

template <int P, int EPI>
static hipError_t launch_gemm_p(const GemmArgs& a, hipStream_t s) {
  constexpr bool PAIR = EpiTraits<EPI>::pair;
  const int n = a.n_rows;
  if constexpr (EPI == EPI_PARTIAL) {
    if (n % 64 == 0 && n >= 2048) return launch_gemm_cfg<P, 4, EPI, 8, gemm_buffers(4, P)>(a, s);
    if (n % 32 == 0 && (int64_t)(n / 32) * a.n_split >= 200) return launch_gemm_cfg<P, 2, EPI, 8, gemm_buffers(2, P)>(a, s);
    return launch_gemm_cfg<P, 1, EPI, 8, gemm_buffers(1, P)>(a, s);
  } else {
    if (EPI != EPI_QKV && a.KT >= 64 && n % 128 == 0 && n / 128 >= 200) return launch_gemm_cfg<P, 8, EPI, 8, gemm_buffers(8, P)>(a, s);
    // 96-row workgroups where they fill the compute units clearly better than 64 rows (24576 rows: 256 workgroups against 384)
    if (EPI != EPI_QKV && a.KT >= 64 && n % 96 == 0 && n / 96 >= 200 && cu_fill(n / 96) > cu_fill(n / 64) + 0.1)
      return launch_gemm_cfg<P, 6, EPI, 8, gemm_buffers(6, P)>(a, s);
    if (n % 64 == 0 && n / 64 >= 200) {
      // a short K (a wavefront sees at most four k-tiles: the 68M-class LM head) is served best by two buffers
      if constexpr (EPI == EPI_STORE) { if (a.KT <= 32) return launch_gemm_cfg<P, 4, EPI, 8, 2>(a, s); }
      return launch_gemm_cfg<P, 4, EPI, 8, gemm_buffers(4, P)>(a, s);
    }
    if constexpr (PAIR) {
      return launch_gemm_cfg<P, 2, EPI, 8, gemm_buffers(2, P)>(a, s);
    } else {
      if (n % 32 == 0 && n / 32 >= 200) return launch_gemm_cfg<P, 2, EPI, 8, gemm_buffers(2, P)>(a, s);
      return launch_gemm_cfg<P, 1, EPI, 8, gemm_buffers(1, P)>(a, s);
    }
  }
}

hipError_t launch_gemm(const GemmArgs& a0, int epi, hipStream_t s) {
  if (a0.M < 1 || a0.M > 16 || a0.KT < 1 || (a0.n_rows & 15)) return hipErrorInvalidValue;
  GemmArgs a = a0;
  if (a.n_split < 1) a.n_split = 1;
  if (epi != EPI_PARTIAL && a.n_split != 1) return hipErrorInvalidValue;
  if (epi == EPI_PARTIAL && (a.h == nullptr || a.n_split > GEMM_MAX_SPLIT || (a.n_split > 1 && (a.counters == nullptr || a.planes == nullptr)))) return hipErrorInvalidValue;
  if (a.ssq != nullptr && (a.n_ssq < 1 || a.n_ssq > 512)) return hipErrorInvalidValue;
  if (a.n_split > a.KT) return hipErrorInvalidValue;
  if (epi != EPI_QKV) a.grp = 1;
  if ((epi == EPI_QKV || epi == EPI_SWIGLU) && (a.n_rows % 32)) return hipErrorInvalidValue;
  if (epi == EPI_QKV && (a.grp < 1 || (a.grp & (a.grp - 1)) != 0 || (a.dh != 64 && a.dh != 128))) return hipErrorInvalidValue;
  const bool p1 = a.M <= 8;
  switch (epi) {
    case EPI_PARTIAL: return p1 ? launch_gemm_p<1, EPI_PARTIAL>(a, s) : launch_gemm_p<2, EPI_PARTIAL>(a, s);
    case EPI_STORE: return p1 ? launch_gemm_p<1, EPI_STORE>(a, s) : launch_gemm_p<2, EPI_STORE>(a, s);
    case EPI_GELU: return p1 ? launch_gemm_p<1, EPI_GELU>(a, s) : launch_gemm_p<2, EPI_GELU>(a, s);
    case EPI_QKV: return p1 ? launch_gemm_p<1, EPI_QKV>(a, s) : launch_gemm_p<2, EPI_QKV>(a, s);
    case EPI_SWIGLU: return p1 ? launch_gemm_p<1, EPI_SWIGLU>(a, s) : launch_gemm_p<2, EPI_SWIGLU>(a, s);
    default: return hipErrorInvalidValue;
  }
}

// ---------------------------------------------------------------------------------------------
// (embedding +) LayerNorm / RMSNorm -> packed activation panels
// ---------------------------------------------------------------------------------------------

// One workgroup per token row.  The row lives in registers: embedding gather (written to the
// residual stream) or the residual stream itself, then the statistics, then the normalised row as
// packed bf16 hi/lo panels -- or, for a deferred RMSNorm, gain * h panels plus the sum of squares.
// tok_override >= 0 replaces the token id read from a.tokens (embedding mode).  COH: the row is handed to other
// workgroups of the same launch.
template <int NT, bool COH = false>
__device__ __forceinline__ void norm_row(const NormArgs& a, const int row, const int tok_override, float* red /* NT / 64 + 1 */,
                                         const uint32_t halted) {
  constexpr int VPT = 2;                       // float4 per thread: d <= NT * 8
  // row = token slot; slots beyond 16 belong to further groups of 16 (prompt pass), whose panels and
  // sums of squares follow those of group 0
  const int m = row & 15, grp = row >> 4, t = threadIdx.x, d = a.d;
  float* h = a.h + (size_t)row * d;
  bf16_t* Xout = a.Xout + (size_t)grp * d * 32;
  float4 v[VPT];
  const bf16_t* e = nullptr; const bf16_t* pe = nullptr;
  if (a.tokens || tok_override >= 0) {
    int tok = tok_override >= 0 ? tok_override : ((a.n_tok == 0 || row < a.n_tok) ? a.tokens[row] : 0);   // padding slots: token 0
    tok = tok < 0 ? 0 : (tok >= a.vocab ? a.vocab - 1 : tok);
    int pos = a.pos0 + row;
    if (pos >= a.max_pos) pos = a.max_pos - 1;
    e = a.tok_emb + (size_t)tok * a.tok_stride;
    pe = a.pos_emb ? a.pos_emb + (size_t)pos * d : nullptr;
  }
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int k = (i * NT + t) * 4;
    v[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (k < d) {
      if (e) {
        const uint2 u = *reinterpret_cast<const uint2*>(e + k);
        v[i] = make_float4(bf16_to_f32(u.x & 0xFFFF), bf16_to_f32(u.x >> 16), bf16_to_f32(u.y & 0xFFFF), bf16_to_f32(u.y >> 16));
        if (pe) {
          const uint2 p = *reinterpret_cast<const uint2*>(pe + k);
          v[i].x += bf16_to_f32(p.x & 0xFFFF); v[i].y += bf16_to_f32(p.x >> 16);
          v[i].z += bf16_to_f32(p.y & 0xFFFF); v[i].w += bf16_to_f32(p.y >> 16);
        }
      } else {
        v[i] = ld_f4<COH>(h + k);
      }
    }
  }
  if (flag_set(halted)) return;                       // uniform over the launch; nothing has been written yet
  if (e) {
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int k = (i * NT + t) * 4;
      if (k < d) st_f4<COH>(h + k, v[i].x, v[i].y, v[i].z, v[i].w);
    }
  }
  if (a.ssq_out != nullptr) {
    // deferred RMSNorm: panels of gain * h, and the row's sum of squares in slot 0 of its ssq row
    float ss = 0.f;
#pragma unroll
    for (int i = 0; i < VPT; ++i) ss += (v[i].x * v[i].x + v[i].y * v[i].y) + (v[i].z * v[i].z + v[i].w * v[i].w);
    ss = block_sum<NT>(ss, red);
    float* sq = a.ssq_out + (size_t)grp * a.n_ssq_out * 16;
    for (int i = t; i < a.n_ssq_out; i += NT) st_f1<COH>(sq + i * 16 + m, (i == 0) ? ss : 0.f);   // [slot][token]
    if (a.sum_out != nullptr) {                   // the consumer's norm is a LayerNorm: the row's sum as well
      float sx = 0.f;
#pragma unroll
      for (int i = 0; i < VPT; ++i) sx += (v[i].x + v[i].y) + (v[i].z + v[i].w);   // zero beyond d
      sx = block_sum<NT>(sx, red);
      float* su = a.sum_out + (size_t)grp * a.n_ssq_out * 16;
      for (int i = t; i < a.n_ssq_out; i += NT) st_f1<COH>(su + i * 16 + m, (i == 0) ? sx : 0.f);
    }
    const int KT = d >> 5;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int k = (i * NT + t) * 4;
      if (k < d) {
        const float4 g = *reinterpret_cast<const float4*>(a.g + k);
        // Which lo the chunks hold is stated: either is as close as the panel's own rounding, but a panel that changes moves cache
        // entries by a bf16 step and the logits by 1e-4, and the compiler's choice changed with unrelated code
        const HiLo x0 = i == 0 ? split_product<true>(v[i].x, g.x, v[i].y, g.y) : split_product<false>(v[i].x, g.x, v[i].y, g.y);
        const HiLo x1 = i == 0 ? split_product<true>(v[i].z, g.z, v[i].w, g.w) : split_product<false>(v[i].z, g.z, v[i].w, g.w);
        xpack_put4<COH>(Xout, KT, a.M, m, k, x0, x1);
      }
    }
    return;
  }
  float mean = 0.f;
  if (a.layernorm) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < VPT; ++i) s += (v[i].x + v[i].y) + (v[i].z + v[i].w);   // zero beyond d
    mean = block_sum<NT>(s, red) / (float)d;
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    if ((i * NT + t) * 4 < d) {
      const float x0 = v[i].x - mean, x1 = v[i].y - mean, x2 = v[i].z - mean, x3 = v[i].w - mean;
      ss += (x0 * x0 + x1 * x1) + (x2 * x2 + x3 * x3);
    }
  }
  const float var = block_sum<NT>(ss, red) / (float)d;
  const float rstd = 1.0f / sqrtf(var + a.eps);
  const int KT = d >> 5;
#pragma unroll
  for (int i = 0; i < VPT; ++i) {
    const int k = (i * NT + t) * 4;
    if (k < d) {
      const float4 g = *reinterpret_cast<const float4*>(a.g + k);
      float o[4] = {(v[i].x - mean) * rstd * g.x, (v[i].y - mean) * rstd * g.y, (v[i].z - mean) * rstd * g.z, (v[i].w - mean) * rstd * g.w};
      if (a.b) {
        const float4 bb = *reinterpret_cast<const float4*>(a.b + k);
        o[0] += bb.x; o[1] += bb.y; o[2] += bb.z; o[3] += bb.w;
      }
      xpack_store4<COH>(Xout, KT, a.M, m, k, o);
    }
  }
}

// GROUPS: wide rows of a prompt pass, in groups of sixteen.
template <int NT, bool GROUPS>
__global__ __launch_bounds__(NT) void k_norm(const int32_t* tokens, const bf16_t* tok_emb, const bf16_t* pos_emb, float* h, const uint32_t* gate, int d, int pos0,
                                             int n_tok, int vocab, NormArgs a) {
  a.tokens = tokens; a.tok_emb = tok_emb; a.pos_emb = pos_emb; a.h = h; a.gate = gate; a.d = d; a.pos0 = pos0; a.n_tok = n_tok; a.vocab = vocab;
  __shared__ float red[NT / 64 + 1];
  // GROUPS: the sixteen rows of a group go to one XCD (ids go round-robin to the eight), whose L2 then puts their panel's lines together, which four
  // rows share; the last groups of a number that is not a multiple of eight go round-robin.
  // (Rows round-robin: embedding of 511 rows of 5120 17 us, 2048 rows 53, 3008 of 6144 98; now 11.6, 41 and 79.)
  const int id = blockIdx.x;
  int row = id;
  if (GROUPS) {
    const int groups = gridDim.x >> 4, whole = groups & ~7, rest = groups & 7;
    if (id < whole * 16) row = ((id >> 7) * 8 + (id & 7)) * 16 + ((id >> 3) & 15);
    else row = (whole + (id - whole * 16) % rest) * 16 + (id - whole * 16) / rest;
  }
  norm_row<NT>(a, row, -1, red, gate_request(a.gate));
}

// One-token activation panel of an fp32 vector (the operand of the GEMVs that give the correction vectors of a
// deferred LayerNorm, W . g and W . b).
__global__ __launch_bounds__(256) void k_vec_panel(const float* __restrict__ v, int d, bf16_t* __restrict__ Xout) {
  const int k = (blockIdx.x * 256 + threadIdx.x) * 4;
  if (k >= d) return;
  float o[4] = {0.f, 0.f, 0.f, 0.f};
  if (v != nullptr) { const float4 x = *reinterpret_cast<const float4*>(v + k); o[0] = x.x; o[1] = x.y; o[2] = x.z; o[3] = x.w; }
  xpack_store4(Xout, d >> 5, 1, 0, k, o);
}

hipError_t launch_vec_panel(const float* v, int d, bf16_t* Xout, hipStream_t s) {
  if (d < 32 || (d & 31) || Xout == nullptr) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_vec_panel, dim3((d / 4 + 255) / 256), dim3(256), 0, s, v, d, Xout);
  return hipGetLastError();
}

// The LayerNorm of a long prompt pass: one workgroup per group of 16 tokens, one wavefront per row, the row in registers (the same two-pass
// variance as norm_row).  The panels are built in LDS, 512 columns at a time, and leave as whole 1 KiB tiles: one row per
// workgroup wrote 16-byte pieces of lines that sixteen workgroups shared, and was bound by those partial lines (78 us against
// 51 for 3008 rows of 6144).  16-byte chunks sit at (token xor eighth of the columns) in LDS, so that neither side has more
// than two lanes on a bank.  Rows of up to 6144 values are held in registers (96 of the 128 that sixteen wavefronts leave a lane; nine
// more go to scratch memory, 40 bytes a lane).
constexpr int NORM_GROUPS_MAX_D = 6144;
__global__ __launch_bounds__(1024) void k_norm_groups(NormArgs a) {
  constexpr int NC = NORM_GROUPS_MAX_D / 256;     // float4 per lane
  __shared__ u32x4 s_hi[2][64][16], s_lo[2][64][16];             // [buffer][eight columns][token]
  const int lane = threadIdx.x & 63, m = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), grp = blockIdx.x, d = a.d, KT = d >> 5;
  const float* h = a.h + (size_t)(grp * 16 + m) * d;
  float4 x[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int k = c * 256 + lane * 4;
    x[c] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (k < d) x[c] = *reinterpret_cast<const float4*>(h + k);
  }
  float mean = 0.f;
  if (a.layernorm) {
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < NC; ++c) sum += (x[c].x + x[c].y) + (x[c].z + x[c].w);   // zero beyond d
    mean = wave_sum(sum) / (float)d;
  }
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < NC; ++c)
    if (c * 256 + lane * 4 < d) {
      const float x0 = x[c].x - mean, x1 = x[c].y - mean, x2 = x[c].z - mean, x3 = x[c].w - mean;
      ss += (x0 * x0 + x1 * x1) + (x2 * x2 + x3 * x3);
    }
  ss = wave_sum(ss);
  const float scale = 1.0f / sqrtf(ss / (float)d + a.eps);
  u32x4* X = reinterpret_cast<u32x4*>(a.Xout + (size_t)grp * d * 32);
#pragma unroll
  for (int c0 = 0; c0 < NC; c0 += 2) {
    if (c0 * 256 < d) {                           // uniform
      const int buf = (c0 >> 1) & 1;
#pragma unroll
      for (int c = c0; c < c0 + 2; ++c) {
        const int k = c * 256 + lane * 4;
        if (k < d) {
          const float4 g = *reinterpret_cast<const float4*>(a.g + k);
          float o[4] = {(x[c].x - mean) * scale * g.x, (x[c].y - mean) * scale * g.y, (x[c].z - mean) * scale * g.z, (x[c].w - mean) * scale * g.w};
          if (a.b) {
            const float4 b = *reinterpret_cast<const float4*>(a.b + k);
            o[0] += b.x; o[1] += b.y; o[2] += b.z; o[3] += b.w;
          }
          const HiLo x0 = split_bf16(o[0], o[1]), x1 = split_bf16(o[2], o[3]);
          const uint2 hi = make_uint2(x0.hi, x1.hi), lo = make_uint2(x0.lo, x1.lo);
          const int e8 = (c - c0) * 32 + (lane >> 1), at = m ^ (e8 & 15);
          reinterpret_cast<uint2*>(&s_hi[buf][e8][at])[lane & 1] = hi;
          reinterpret_cast<uint2*>(&s_lo[buf][e8][at])[lane & 1] = lo;
        }
      }
      __syncthreads();                            // the chunk is complete; its buffer is written again two chunks on
      const int e8 = threadIdx.x >> 4, t = threadIdx.x & 15, ke = c0 * 32 + e8;      // eight columns, token
      if (ke * 8 < d) {
        X[(size_t)ke * 16 + t] = s_hi[buf][e8][t ^ (e8 & 15)];
        X[(size_t)KT * 64 + (size_t)ke * 16 + t] = s_lo[buf][e8][t ^ (e8 & 15)];
      }
    }
  }
}

// a workgroup per group needs groups for half the compute units: the embedding of 511 rows of 5120 (32 groups) took 39 us that
// way against 17 (11.6 since the rows of a group share an XCD), so fewer groups, and the embedding, which gathers, keep a workgroup per row
bool norm_groups_fit(int d, int n_groups) { return n_groups >= 128 && d <= NORM_GROUPS_MAX_D; }

hipError_t launch_norm(const NormArgs& a, hipStream_t s) {
  if (a.M < 1 || a.M > 16 || (a.d & 31) || a.d > 8192) return hipErrorInvalidValue;
  // prompt pass: n_groups groups of 16 slots each (then M == 16: two-panel layout)
  if (a.n_groups < 0 || (a.n_groups > 0 && a.M != 16)) return hipErrorInvalidValue;
  if (a.tokens == nullptr && a.ssq_out == nullptr && a.gate == nullptr && norm_groups_fit(a.d, a.n_groups)) {
    hipLaunchKernelGGL(k_norm_groups, dim3((unsigned)a.n_groups), dim3(1024), 0, s, a);
    return hipGetLastError();
  }
  const unsigned rows = a.n_groups > 0 ? 16u * (unsigned)a.n_groups : (unsigned)a.M;
  const int nt = a.d <= 2048 ? 256 : 1024;
  // reading the grid's size costs a launch about 0.2 us, more than narrow rows gain (twelve layers of 768 columns at 39 tokens 633 -> 638 us a
  // pass), and fewer than eight groups have no XCD of their own
  const bool groups = nt == 1024 && a.n_groups >= 8;
  hipLaunchKernelGGL((nt == 256 ? k_norm<256, false> : (groups ? k_norm<1024, true> : k_norm<1024, false>)), dim3(rows), dim3(nt), 0, s, a.tokens, a.tok_emb, a.pos_emb, a.h, a.gate, a.d, a.pos0,
                     a.n_tok, a.vocab, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// paged attention: M <= 16 queries of one head against cached positions, causal inside the block
// ---------------------------------------------------------------------------------------------

// Workgroup = (query head, range of split_len cached positions), 8 wavefronts; a wavefront takes 32
// positions per step straight from the paged cache into matrix-unit operands:
//   S^T[key][query]  = K[16 keys x d_head] . Q^T      (16x16x32 bf16; K rows are 128-bit loads;
//                                                     q is fp32 split into bf16 hi + lo)
//   O^T[chan][query] = V^T[16 chan x 16 keys] . P^T   (16x16x16 bf16; the S accumulator layout is
//                                                     exactly this instruction's P operand layout,
//                                                     so probabilities never leave registers)
// which is why V is cached transposed ([d_head][token] inside a page).  Soft-max statistics run
// per query across the four 16-lane rows; P is fed as bf16 hi + lo.  The wavefronts merge
// their (max, sum, O) through LDS and write one partial record per (head, range, query).

typedef __attribute__((ext_vector_type(4))) short s16x4;

// One wavefront's share of the attention of one head: 32 cached positions per step.
// QCOH: the queries were written by other workgroups of this launch (hand-off loads); VCOH: so were entries of
// the transposed V blocks, in 128-byte lines that an earlier step of the same launch may have read (a draft loop
// inside one launch), so V tiles are fetched with L2-bypassing loads.
// LO: q and P enter the matrix unit as bf16 hi + lo (fp32 grade); without it as bf16 only (the prompt pass with bf16
// activations: half the matrix instructions).
template <int DH, bool QCOH = false, bool VCOH = false, bool LO = true>
struct AttnWave {
  static constexpr int KS = DH / 32, CT = DH / 16;
  // raw operands of one step: K rows of two 16-position tiles, V^T tiles of the same positions
  struct Raw { u32x4 k[2][KS]; uint2 v[2][CT]; };
  const AttnArgs& a;
  const float* qb;
  int j, g, kvh, total, s1, pt, pshift, qpos;
  size_t kv_head_elems, page_elems;
  bf16x8 qh[KS], ql[KS];
  f32x4 O[CT];
  float m_run, l_run;

  // pos0_ / q_: first position and query rows of this object's token group when they are not the launch's (prompt pass:
  // one workgroup serves two groups of 16 tokens); s1_ < 0: the range ends with the group's own tokens
  __device__ __forceinline__ AttnWave(const AttnArgs& a_, int head, int s1_, int pos0_ = -1, const float* q_ = nullptr) : a(a_) {
    const int lane = threadIdx.x & 63;
    j = lane & 15; g = lane >> 4;
    kvh = a.nkv == 1 ? 0 : (a.nq == a.nkv ? head : head / (a.nq / a.nkv));
    const int pos0 = pos0_ < 0 ? a.pos0 : pos0_;
    qb = q_ != nullptr ? q_ : a.q;
    total = pos0 + a.M; s1 = s1_ < 0 ? total : s1_; pt = a.page_tokens;
    pshift = (pt & (pt - 1)) == 0 ? __builtin_ctz(pt) : -1;     // power-of-two pages: shifts instead of divisions
    qpos = pos0 + j;                                              // last position query j may see
    kv_head_elems = (size_t)pt * DH;                              // one head's K (or V) block in a page
    page_elems = 2 * (size_t)a.nkv * kv_head_elems;
#pragma unroll
    for (int c = 0; c < CT; ++c) O[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    m_run = NEG_BIG; l_run = 0.f;
  }

  // every load of a step is issued at once; none depends on the queries
  __device__ __forceinline__ void issue(Raw& r, const int base) const {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kb = base + 16 * t;
      if (kb < s1) {
        const int p = min(kb + j, total - 1), lp = pshift >= 0 ? p >> pshift : p / pt, off = p - lp * pt;
        const int pp = a.page_table ? a.page_table[lp] : lp;
        const bf16_t* kp = a.kv_layer + (size_t)pp * page_elems + (size_t)kvh * kv_head_elems + (size_t)off * DH + 8 * g;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) r.k[t][ks] = *reinterpret_cast<const u32x4*>(kp + ks * 32);
      }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kb = base + 16 * t;
      if (kb < s1) {
        // V^T operand: channel row = lane % 16 of each 16-channel tile, 4 consecutive positions
        const int p0 = kb + 4 * g;
        const int pc = min(p0, (total - 1) & ~3), lp = pshift >= 0 ? pc >> pshift : pc / pt, off = pc - lp * pt;
        const int pp = a.page_table ? a.page_table[lp] : lp;
        const bf16_t* vp = a.kv_layer + (size_t)pp * page_elems + (size_t)(a.nkv + kvh) * kv_head_elems + (size_t)j * pt + off;
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          if (VCOH) {
            const unsigned long long u = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(vp + (size_t)c * 16 * pt), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            r.v[t][c] = make_uint2((uint32_t)u, (uint32_t)(u >> 32));
          } else {
            r.v[t][c] = *reinterpret_cast<const uint2*>(vp + (size_t)c * 16 * pt);
          }
        }
      }
    }
  }

  // query operand: column j holds query min(j, M-1) (surplus columns are never stored)
  __device__ __forceinline__ void load_q(int head) {
    const float* qp = qb + (size_t)min(j, a.M - 1) * a.ldq + head * DH + 8 * g;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const float4 x0 = ld_f4<QCOH>(qp + ks * 32), x1 = ld_f4<QCOH>(qp + ks * 32 + 4);
      const float xv[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
      u32x4 h, l;
#pragma unroll
      for (int i = 0; i < 4; ++i) { const HiLo x = split_bf16(xv[2 * i], xv[2 * i + 1]); h[i] = x.hi; l[i] = LO ? x.lo : 0u; }
      qh[ks] = as_bf16x8(h); ql[ks] = as_bf16x8(l);
    }
  }

  // scores, running soft-max and P.V of one step
  __device__ __forceinline__ void step(const Raw& r, const int base) {
    f32x4 S[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kb = base + 16 * t;
      S[t] = f32x4{NEG_BIG, NEG_BIG, NEG_BIG, NEG_BIG};
      if (kb < s1) {
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          const bf16x8 kk = as_bf16x8(r.k[t][ks]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk, qh[ks], acc, 0, 0, 0);
          if (LO) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk, ql[ks], acc, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int pos = kb + 4 * g + v;
          if (pos < s1 && pos <= qpos) S[t][v] = acc[v] * a.scale;
        }
      }
    }
    float mx = fmaxf(fmaxf(fmaxf(S[0][0], S[0][1]), fmaxf(S[0][2], S[0][3])), fmaxf(fmaxf(S[1][0], S[1][1]), fmaxf(S[1][2], S[1][3])));
    mx = row4_max(mx);
    const float m_new = fmaxf(m_run, mx);
    const float alpha = __expf(m_run - m_new);
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float e = (S[t][v] > 0.5f * NEG_BIG) ? __expf(S[t][v] - m_new) : 0.f;   // hardware exp2: a few ulp, far inside the bf16 split of P
        S[t][v] = e;
        sum += e;
      }
    sum = row4_sum(sum);
    l_run = l_run * alpha + sum;
    m_run = m_new;
#pragma unroll
    for (int c = 0; c < CT; ++c) O[c] *= alpha;
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int kb = base + 16 * t;
      if (kb < s1) {
        union { uint32_t u[2]; s16x4 v; } ph, pl;
#pragma unroll
        for (int v = 0; v < 2; ++v) { const HiLo x = split_bf16(S[t][2 * v], S[t][2 * v + 1]); ph.u[v] = x.hi; pl.u[v] = LO ? x.lo : 0u; }
        // positions at or beyond `total` hold stale bytes: zero them (0 * NaN would poison the sum)
        const int p0 = kb + 4 * g;
        uint2 keep;
        keep.x = (p0 < total ? 0x0000FFFFu : 0u) | (p0 + 1 < total ? 0xFFFF0000u : 0u);
        keep.y = (p0 + 2 < total ? 0x0000FFFFu : 0u) | (p0 + 3 < total ? 0xFFFF0000u : 0u);
#pragma unroll
        for (int c = 0; c < CT; ++c) {
          uint2 raw = r.v[t][c];
          raw.x &= keep.x; raw.y &= keep.y;
          union { uint2 u; s16x4 v; } vv; vv.u = raw;
          O[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vv.v, ph.v, O[c], 0, 0, 0);
          if (LO) O[c] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vv.v, pl.v, O[c], 0, 0, 0);
        }
      }
    }
  }
};

// LDS of one attention work unit of NWV wavefronts.
template <int DH, int NWV>
struct AttnSmem {
  f32x4 o_s[NWV][DH / 16][64];
  float m_s[NWV][16], l_s[NWV][16];
  int s_last;
};

// Sums of two ranges brought to a common maximum.  The roundings are written out here and in what follows it (the panels of the
// quotients, see split_product), since ranges are merged by more than one kernel.
__device__ __forceinline__ float merged(float a, float fa, float b, float fb) { return fmaf(a, fa, b * fb); }
constexpr bool RANGES_LO_EXACT = true;
// ... and the sum of the wavefronts' parts of a range: part(i), rescaled by scale(i), i = 0 .. N - 1
template <int N, typename PartOf, typename ScaleOf>
__device__ __forceinline__ f32x4 range_sum(PartOf part, ScaleOf scale) {
  const f32x4 p0 = part(0), p1 = part(1);
  f32x4 o;
#pragma unroll
  for (int v = 0; v < 4; ++v) o[v] = merged(p0[v], scale(0), p1[v], scale(1));
#pragma unroll
  for (int i = 2; i < N; ++i) {
    const f32x4 p = part(i);
#pragma unroll
    for (int v = 0; v < 4; ++v) o[v] = fmaf(p[v], scale(i), o[v]);
  }
  return o;
}

// Work unit (query head, range `split` of split_len cached positions) run by NWV wavefronts; the last range of
// a head to finish merges all of the head's records and writes the O-projection panels.
// `hook` runs once before anything that other workgroups of the launch may still be writing is touched (the queries,
// cache entries at or beyond `safe_end`): a wavefront whose first 32 positions lie below safe_end requests them
// before the hook, so those loads are in flight while the hook waits.  The workgroup that merges the head also
// zeroes `reset_word` (the counter the hook waited on), if given.
template <int DH, int NWV, bool COH = false, bool VCOH = false, bool QCOH = false, typename Hook = NoHook>
__device__ __forceinline__ void attn_range(const AttnArgs& a, const int head, const int split, AttnSmem<DH, NWV>& sm,
                                           const uint32_t halted, const Hook hook = Hook(), const int safe_end = 0x7fffff00,
                                           int* reset_word = nullptr) {
  constexpr int CT = DH / 16, WKEYS = 32;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int total = a.pos0 + a.M;
  const int s0 = split * a.split_len, s1 = min(s0 + a.split_len, total);
  AttnWave<DH, QCOH, VCOH> aw(a, head, s1);      // (a persistent kernel gives the queries a fresh address per layer)
  typename AttnWave<DH, QCOH, VCOH>::Raw r0, r1;
  // the first step's cache loads go out ahead of the q loads; later steps' loads are in flight during
  // the arithmetic of the step before
  constexpr int STEP = NWV * WKEYS;
  constexpr bool WAITS = !std::is_same<Hook, NoHook>::value;     // there is a wait to fill: two steps' loads go out before it
  int base = s0 + w * WKEYS;
  const bool early0 = base + WKEYS <= safe_end, early1 = WAITS && base + STEP + WKEYS <= safe_end;
  if (base < s1 && early0) aw.issue(r0, base);
  if (base + STEP < s1 && early1) aw.issue(r1, base + STEP);
  hook();
  if (base < s1 && !early0) aw.issue(r0, base);
  aw.load_q(head);
  if (flag_set(halted)) return;                       // uniform over the launch; nothing has been written yet
  if (base + STEP < s1 && !early1) aw.issue(r1, base + STEP);
  while (base < s1) {
    aw.step(r0, base);
    if (base + 2 * STEP < s1) aw.issue(r0, base + 2 * STEP);
    base += STEP;
    if (base >= s1) break;
    aw.step(r1, base);
    if (base + 2 * STEP < s1) aw.issue(r1, base + 2 * STEP);
    base += STEP;
  }

  // merge the wavefronts (fixed order), then one record per query: o[DH], max, sum
  __syncthreads();                                // a previous unit of this workgroup has left the buffers
#pragma unroll
  for (int c = 0; c < CT; ++c) sm.o_s[w][c][lane] = aw.O[c];
  if (g == 0) { sm.m_s[w][j] = aw.m_run; sm.l_s[w][j] = aw.l_run; }
  __syncthreads();
  float mm = sm.m_s[0][j];
#pragma unroll
  for (int ww = 1; ww < NWV; ++ww) mm = fmaxf(mm, sm.m_s[ww][j]);
  float f[NWV], ll = 0.f;
#pragma unroll
  for (int ww = 0; ww < NWV; ++ww) { f[ww] = expf(sm.m_s[ww][j] - mm); ll += sm.l_s[ww][j] * f[ww]; }
  if (j < a.M) {
    float* rec = a.part + (((size_t)head * a.n_splits + split) * 16 + j) * (DH + 2);
    // channel tiles are dealt to the wavefronts: tiles w, w + NWV, ..
#pragma unroll
    for (int ci = 0; ci < (CT + NWV - 1) / NWV; ++ci) {
      const int c = w + ci * NWV;
      if (c < CT) {
        const f32x4 o = range_sum<NWV>([&](int ww) { return sm.o_s[ww][c][lane]; }, [&](int ww) { return f[ww]; });
        st_agent2(rec + c * 16 + 4 * g, o[0], o[1]);
        st_agent2(rec + c * 16 + 4 * g + 2, o[2], o[3]);
      }
    }
    if (w == 0 && g == 0) st_agent2(rec + DH, mm, ll);
  }
  // the last range of this head to finish merges all ranges (in range order) into the panels that
  // feed the O-projection
  if (!last_arrival(a.counters + head, a.n_splits, &sm.s_last)) return;
  if (reset_word != nullptr && threadIdx.x == 0) __hip_atomic_store(reset_word, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  // 8 channels per thread: DH / 8 threads per query, so that all 16 queries of a block are merged in one
  // pass (a second pass would put a second round trip to the records behind the first)
  constexpr int TPQ = DH / 8;
  const int tq = threadIdx.x % TPQ;
  for (int qm = threadIdx.x / TPQ; qm < a.M; qm += NWV * 64 / TPQ) {
    const float* rbase = a.part + (((size_t)head * a.n_splits) * 16 + qm) * (DH + 2);
    const size_t stride = (size_t)16 * (DH + 2);
    // running (max, sum, o) over the ranges in range order; eight ranges' records are fetched at a
    // time so that their round trips overlap
    float mx = NEG_BIG, L = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int sp0 = 0; sp0 < a.n_splits; sp0 += 8) {
      float2 ml[8], v[8][4];
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (sp0 + i < a.n_splits) {
          const float* rc = rbase + (size_t)(sp0 + i) * stride;
          ml[i] = ld_agent2(rc + DH);
#pragma unroll
          for (int c = 0; c < 4; ++c) v[i][c] = ld_agent2(rc + 8 * tq + 2 * c);
        }
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (sp0 + i < a.n_splits) {
          const float m_new = fmaxf(mx, ml[i].x);
          const float f_old = expf(mx - m_new), f_new = expf(ml[i].x - m_new);
          L = merged(L, f_old, ml[i].y, f_new);
#pragma unroll
          for (int c = 0; c < 4; ++c) {
            o[2 * c] = merged(o[2 * c], f_old, v[i][c].x, f_new);
            o[2 * c + 1] = merged(o[2 * c + 1], f_old, v[i][c].y, f_new);
          }
          mx = m_new;
        }
    }
    const float inv = 1.0f / L;
#pragma unroll
    for (int i = 0; i < 8; i += 4)
      xpack_put4<COH>(a.Xout, (a.nq * DH) >> 5, a.M, qm, head * DH + 8 * tq + i, split_product<RANGES_LO_EXACT>(o[i], inv, o[i + 1], inv),
                      split_product<RANGES_LO_EXACT>(o[i + 2], inv, o[i + 3], inv));
  }
}

// Leading arguments of the attention kernels (see k_gemm).  A query row is as wide as its heads (the launcher checks it).
#define ATTN_EARLY const bf16_t* kv_layer, const int32_t* page_table, const float* q, const uint32_t* gate, int page_tokens, int nq, int nkv, \
                   int pos0, int M, int split_len
#define ATTN_EARLY_SET(a) do { a.kv_layer = kv_layer; a.page_table = page_table; a.q = q; a.gate = gate; a.page_tokens = page_tokens; \
  a.nq = nq; a.nkv = nkv; a.ldq = nq * DH; a.pos0 = pos0; a.M = M; a.split_len = split_len; } while (0)
#define ATTN_EARLY_ARGS(a) a.kv_layer, a.page_table, a.q, a.gate, a.page_tokens, a.nq, a.nkv, a.pos0, a.M, a.split_len
template <int DH>
__global__ __launch_bounds__(512) void k_attn_partial(ATTN_EARLY, AttnArgs a) {
  ATTN_EARLY_SET(a);
  __shared__ AttnSmem<DH, 8> sm;                  // eight wavefronts: a range of 256 positions is one step each (measured
  attn_range<DH, 8>(a, blockIdx.x, blockIdx.y, sm, gate_request(a.gate));   // 1.3 % of a 13B verification block against four)
}

// Whole head: one workgroup of eight wavefronts takes all positions of a head (256 at most, one step of a wavefront), merges its
// wavefronts through LDS and writes the O-projection panels itself: no partial records, no hand-off between workgroups.  request() asks
// for the cache entries as far as they lie below safe_end and may run long before run().  split_len 128: the wavefronts
// are merged as two ranges would be, rounding for rounding, so that it does not show which kernel took a context of that deal.
template <int DH, bool QCOH = false>
struct AttnWhole {
  static constexpr int CT = DH / 16, NWV = 8, WKEYS = 32;
  AttnWave<DH, QCOH> aw;
  typename AttnWave<DH, QCOH>::Raw r;
  int head, first;
  __device__ __forceinline__ AttnWhole(const AttnArgs& a, int head_) : aw(a, head_, -1), head(head_), first((int)(threadIdx.x >> 6) * WKEYS) {}
  __device__ __forceinline__ void request(const int safe_end) {
    if (first + WKEYS <= safe_end) aw.issue(r, first);
  }
  // `requested`: the safe_end that request() was given
  __device__ __forceinline__ void run(AttnSmem<DH, NWV>& sm, const int requested, const uint32_t halted) {
    const AttnArgs& a = aw.a;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, j = lane & 15, g = lane >> 4, total = aw.total;
    if (first + WKEYS > requested && first < total) aw.issue(r, first);
    aw.load_q(head);
    if (flag_set(halted)) return;                 // uniform over the launch; nothing has been written yet
    if (first < total) aw.step(r, first);
    __syncthreads();                              // the phase before has left the buffers
#pragma unroll
    for (int c = 0; c < CT; ++c) sm.o_s[w][c][lane] = aw.O[c];
    if (g == 0) { sm.m_s[w][j] = aw.m_run; sm.l_s[w][j] = aw.l_run; }
    __syncthreads();
    if (w >= CT || j >= a.M) return;              // wavefront w finishes channel tile w
    struct Part { float m, l; };
    // maximum and sum of wavefronts w0 .. w0 + N - 1, and what brings each to that maximum
    auto part = [&](const int w0, auto& f) {
      constexpr int N = sizeof(f) / sizeof(f[0]);
      Part p{sm.m_s[w0][j], 0.f};
#pragma unroll
      for (int i = 1; i < N; ++i) p.m = fmaxf(p.m, sm.m_s[w0 + i][j]);
#pragma unroll
      for (int i = 0; i < N; ++i) { f[i] = expf(sm.m_s[w0 + i][j] - p.m); p.l = fmaf(sm.l_s[w0 + i][j], f[i], p.l); }
      return p;
    };
    bf16_t* const X = a.Xout;
    const int KT = (a.nq * DH) >> 5, k = head * DH + w * 16 + 4 * g;
    if (a.split_len >= NWV * WKEYS) {             // uniform
      float f[NWV];
      const Part p = part(0, f);
      const float inv = 1.0f / p.l;
      f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < NWV; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = fmaf(sm.o_s[i][w][lane][v], f[i], o[v]);
      xpack_put4(X, KT, a.M, j, k, split_product<true>(o[0], inv, o[1], inv), split_product<true>(o[2], inv, o[3], inv));
    } else {
      constexpr int N = NWV / 2;
      float f0[N], f1[N];
      const Part p0 = part(0, f0), p1 = part(N, f1);
      const float m = fmaxf(p0.m, p1.m), e0 = expf(p0.m - m), e1 = expf(p1.m - m), inv = 1.0f / merged(p0.l, e0, p1.l, e1);
      const f32x4 o0 = range_sum<N>([&](int i) { return sm.o_s[i][w][lane]; }, [&](int i) { return f0[i]; });
      const f32x4 o1 = range_sum<N>([&](int i) { return sm.o_s[N + i][w][lane]; }, [&](int i) { return f1[i]; });
      f32x4 o;
#pragma unroll
      for (int v = 0; v < 4; ++v) o[v] = merged(o0[v], e0, o1[v], e1);
      xpack_put4(X, KT, a.M, j, k, split_product<RANGES_LO_EXACT>(o[0], inv, o[1], inv), split_product<RANGES_LO_EXACT>(o[2], inv, o[3], inv));
    }
  }
};

template <int DH>
__global__ __launch_bounds__(512) void k_attn_head(ATTN_EARLY, AttnArgs a) {
  ATTN_EARLY_SET(a);
  __shared__ AttnSmem<DH, 8> sm;
  AttnWhole<DH> at(a, blockIdx.x);
  const uint32_t halted = gate_request(a.gate);
  at.request(0x7fffff00);
  at.run(sm, 0x7fffff00, halted);
}

// Prompt pass: workgroup = (query head, two consecutive groups of 16 prompt tokens).  Group r sits at positions
// pos0 + 16 r .. and sees everything up to its own tokens.  The eight wavefronts share the cached positions (32 per
// wavefront and step); every K and V tile a wavefront fetches serves the queries of both groups (half the cache reads
// and half the workgroups of one group per workgroup: the kernel waits on those reads), each group with its own
// running soft-max.  The groups are merged across the wavefronts one after the other through one LDS buffer.  The
// longest ranges are scheduled first.
constexpr int ATTN_MG = 2;
template <int DH, bool LO>
__global__ __launch_bounds__(512) void k_attn_groups(const bf16_t* kv_layer, const int32_t* page_table, const float* q, int page_tokens, int nq, int nkv, int ldq,
                                                     int pos0, int n_groups, AttnArgs a, size_t x_stride) {    // (leading arguments: see k_gemm)
  a.kv_layer = kv_layer; a.page_table = page_table; a.q = q; a.page_tokens = page_tokens; a.nq = nq; a.nkv = nkv;
  a.ldq = ldq; a.pos0 = pos0; a.M = 16;
  constexpr int CT = DH / 16, NWV = 8, WKEYS = 32, STEP = NWV * WKEYS, NG = ATTN_MG;
  __shared__ f32x4 o_s[NWV][CT][64];
  __shared__ float m_s[NWV][16], l_s[NWV][16];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int head = blockIdx.x;
  const int nb = (n_groups + NG - 1) / NG;
  const int r0g = (nb - 1 - (int)blockIdx.y) * NG;                // first group of this workgroup
  const int ng = min(NG, n_groups - r0g);
  auto grp = [&](int i) { return r0g + min(i, ng - 1); };          // a surplus slot repeats the last group and stores nothing
  auto wave_of = [&](int i) { return AttnWave<DH, false, false, LO>(a, head, -1, a.pos0 + 16 * grp(i), a.q + (size_t)grp(i) * 16 * a.ldq); };
  AttnWave<DH, false, false, LO> aw[NG] = {wave_of(0), wave_of(1)};
  static_assert(NG == 2, "the initialiser above lists two groups");
  const int total = aw[NG - 1].total;                              // the longest range: its object issues the loads
  // one set of raw operands per wavefront (two would not fit beside the state of two groups); the other wavefront of
  // the SIMD covers the wait (re-issuing the K loads between the two halves of a step measured slower)
  typename AttnWave<DH, false, false, LO>::Raw ra;
  int base = w * WKEYS;
  if (base < total) aw[NG - 1].issue(ra, base);
#pragma unroll
  for (int i = 0; i < NG; ++i) aw[i].load_q(head);
  while (base < total) {
#pragma unroll
    for (int i = 0; i < NG; ++i)
      if (base < aw[i].total) aw[i].step(ra, base);
    base += STEP;
    if (base < total) aw[NG - 1].issue(ra, base);
  }
#pragma unroll
  for (int i = 0; i < NG; ++i) {
    if (i > 0) __syncthreads();                                    // the merge of the group before has read the buffer
#pragma unroll
    for (int c = 0; c < CT; ++c) o_s[w][c][lane] = aw[i].O[c];
    if (g == 0) { m_s[w][j] = aw[i].m_run; l_s[w][j] = aw[i].l_run; }
    __syncthreads();
    if (i < ng && w < CT) {                                        // wavefront w finishes channel tile w
      float mm = m_s[0][j];
#pragma unroll
      for (int ww = 1; ww < NWV; ++ww) mm = fmaxf(mm, m_s[ww][j]);
      float ll = 0.f;
      f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ww = 0; ww < NWV; ++ww) {                           // fixed order: deterministic
        const float f = expf(m_s[ww][j] - mm);
        ll += l_s[ww][j] * f;
        o += o_s[ww][w][lane] * f;
      }
      const float inv = 1.0f / ll;
      const float out4[4] = {o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv};
      xpack_store4(a.Xout + (size_t)(r0g + i) * x_stride, (a.nq * DH) >> 5, a.M, j, head * DH + w * 16 + 4 * g, out4);
    }
  }
}

// Prompt pass, tiled: a wavefront owns 32 query columns (32 tokens of one head); the four wavefronts of a workgroup share one
// K / V head: as many query heads of its group as divide four, times 32-token blocks.  K and V come through LDS in tiles of 64
// positions (copied straight from the pages, two buffers: the next tile arrives during the arithmetic of this one), so a
// cache entry is fetched once per 128 query columns instead of once per 32, and the matrix unit works on 32x32x16 instructions:
//   S^T[key][query] = K . Q^T (q as hi + lo in registers), soft-max per query column (lane l and l + 32 share a column),
//   O^T[chan][query] += V^T . P^T: the S accumulators are P's operand after one half-wavefront swap per register.
// LDS chunks of 16 bytes are stored at (chunk xor row) so that both the copies (whole rows) and the fragment reads (one chunk
// column of 16 rows) are free of bank conflicts.  Bound by the matrix unit and the soft-max's vector instructions, about
// equal at hi + lo.  Measured per layer, 48 heads on one K / V head, 3001 tokens after 333: 333 us against 749 with 32 query
// columns per pass over the cache; 40 heads, 2048 tokens, bf16 operands: 87 against 211.
// Needs pages of a power of two of at least 8 tokens (a V^T chunk is 8 tokens of a channel) and of fewer than 2^32 elements
// (offsets inside a page are 32-bit; the page's own offset is 64-bit).
template <int DH, bool LO>
__global__ __launch_bounds__(256, 2) void k_attn_tiles(AttnArgs a, int n_groups, size_t x_stride, int hw_log2) {
  constexpr int KB = 64, S16 = DH / 16, CB = DH / 32, CK = DH / 8, RPI = 64 / CK, PER = DH / 32;   // PER: copies of K (and of V) per wavefront and tile
  __shared__ u32x4 ks[2][KB * CK], vs[2][DH * (KB / 8)];
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 31, hf = lane >> 5;
  const int HW = 1 << hw_log2, TW = 4 >> hw_log2, rep = a.nq / a.nkv, hgs = rep >> hw_log2;
  const int kvh = blockIdx.x / hgs, head = kvh * rep + (blockIdx.x - kvh * hgs) * HW + (w & (HW - 1));
  const int tbg = gridDim.y - 1 - blockIdx.y;                      // the longest ranges are scheduled first
  const int rows = 16 * n_groups, r0 = 32 * (tbg * TW + (w >> hw_log2));
  const int end = a.pos0 + min(32 * TW * (tbg + 1), rows);         // positions at or beyond it: not read (K) or not used (V)
  const int w_end = r0 < rows ? a.pos0 + min(r0 + 32, rows) : 0;   // this wavefront's (0: no tokens of its own, it only copies)
  const int r = min(r0 + col, rows - 1), qpos = a.pos0 + r, pt = a.page_tokens, pshift = __builtin_ctz(pt);
  const uint32_t head_elems = (uint32_t)pt * DH, page_elems = 2u * (uint32_t)a.nkv * head_elems;   // below 2^32 (attn_tiles_fit)

  // positions this lane copies in a tile: K row of instruction i, V chunk (the same chunk of every channel it copies)
  auto k_row = [&](const int i) { return RPI * (w + 4 * i) + lane / CK; };
  const int v_swz = ((8 * w + (lane >> 3)) >> 1) & 7, v_chunk = (lane & 7) ^ v_swz;    // channel 8 (w + 4 i) + lane / 8: the swizzle does not depend on i
  auto k_pos = [&](const int base, const int i) { return min(base + k_row(i), end - 1); };
  auto v_pos = [&](const int base) { return min(base + 8 * v_chunk, (end - 1) & ~7); };
  // physical pages of those positions; the next tile's are looked up one tile ahead
  uint32_t kp[PER], vp;
  auto pages = [&](const int base) {
#pragma unroll
    for (int i = 0; i < PER; ++i) kp[i] = (uint32_t)k_pos(base, i) >> pshift;
    vp = (uint32_t)v_pos(base) >> pshift;
    if (a.page_table) {
#pragma unroll
      for (int i = 0; i < PER; ++i) kp[i] = (uint32_t)a.page_table[kp[i]];
      vp = (uint32_t)a.page_table[vp];
    }
  };
  const uint32_t lds_k = lds_address(&ks[0][0]), lds_v = lds_address(&vs[0][0]);
  auto copy = [&](const int base, const int buf) {
#pragma unroll
    for (int i = 0; i < PER; ++i) {
      const int kr = k_row(i), off = k_pos(base, i) & (pt - 1);
      const int c = (lane % CK) ^ (DH == 128 ? kr & 15 : (kr >> 1) & 7);
      lds_dma_16(a.kv_layer + (uint64_t)kp[i] * page_elems + (uint32_t)(kvh * head_elems + off * DH + c * 8),
                 lds_k + (uint32_t)(buf * KB * CK + (w + 4 * i) * 64) * 16u);
    }
    const int off = v_pos(base) & (pt - 1);
    const bf16_t* vb = a.kv_layer + (uint64_t)vp * page_elems + (uint32_t)((a.nkv + kvh) * head_elems + (lane >> 3) * pt + off);
#pragma unroll
    for (int i = 0; i < PER; ++i)
      lds_dma_16(vb + 8 * (w + 4 * i) * pt, lds_v + (uint32_t)(buf * DH * 8 + (w + 4 * i) * 64) * 16u);
  };
  const int n_kt = (end + KB - 1) / KB;
  pages(0);
  copy(0, 0);
  if (n_kt > 1) pages(KB);

  bf16x8 qh[S16], ql[LO ? S16 : 1];
  {
    const float* qp = a.q + (size_t)r * a.ldq + head * DH + 8 * hf;
#pragma unroll
    for (int s = 0; s < S16; ++s) {
      const float4 x0 = *reinterpret_cast<const float4*>(qp + 16 * s), x1 = *reinterpret_cast<const float4*>(qp + 16 * s + 4);
      const float xv[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
      u32x4 h, l;
#pragma unroll
      for (int i = 0; i < 4; ++i) { const HiLo x = split_bf16(xv[2 * i], xv[2 * i + 1]); h[i] = x.hi; l[i] = LO ? x.lo : 0u; }
      qh[s] = as_bf16x8(h);
      if (LO) ql[LO ? s : 0] = as_bf16x8(l);
    }
  }
  f32x16 O[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c)
#pragma unroll
    for (int v = 0; v < 16; ++v) O[c][v] = 0.f;
  // of column `col` (both halves hold the maximum; each its own keys' sum).  The maximum starts far above DROPPED, so that keys
  // without a score weigh nothing even where a column has met no other
  constexpr float DROPPED = -1.0e33f;
  float m_run = 0.5f * NEG_BIG / a.scale, l_run = 0.f;
  const float ce = a.scale * 1.44269504088896f;   // exp(scale (s - m)) = exp2(ce s - ce m)
  float top = INFINITY;
  asm("" : "+v"(top));                            // (with the constant in sight the compiler makes two instructions of each median)

  // 32 positions (half kb of the tile in buffer buf, from position base on)
  auto step = [&](const int base, const int buf, const int kb) {
    const bool edge = base + 31 > a.pos0 + r0;    // some of them lie beyond the first query's (uniform)
    const u32x4* kt = &ks[buf][(32 * kb + col) * CK];
    const u32x4* vt = &vs[buf][col * 8];
    const int kx = DH == 128 ? col & 15 : (col >> 1) & 7, vx = (col >> 1) & 7;
    auto k_frag = [&](const int s) { return as_bf16x8(kt[(2 * s + hf) ^ kx]); };
    auto v_frag = [&](const int s, const int c) { return vt[32 * c * 8 + ((4 * kb + 2 * s + hf) ^ vx)]; };
    f32x16 S;
#pragma unroll
    for (int v = 0; v < 16; ++v) S[v] = 0.f;
    bf16x8 kk[3];                                 // fragments are read two steps ahead of their products
    kk[0] = k_frag(0);
    kk[1] = k_frag(1);
#pragma unroll
    for (int s = 0; s < S16; ++s) {
      if (s + 2 < S16) kk[(s + 2) % 3] = k_frag(s + 2);
      S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[s % 3], qh[s], S, 0, 0, 0);
      if (LO) S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kk[s % 3], ql[LO ? s : 0], S, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    u32x4 vv[2][CB];
#pragma unroll
    for (int c = 0; c < CB; ++c) vv[0][c] = v_frag(0, c);
    if (edge) {
#pragma unroll
      for (int v = 0; v < 16; ++v)
        if (base + 8 * (v >> 2) + 4 * hf + (v & 3) > qpos) S[v] = DROPPED;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) S[v] = __builtin_amdgcn_fmed3f(S[v], DROPPED, top);        // NaN becomes DROPPED, the rest stays
    float mx = S[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, S[v]);
    mx = half_max(mx);
    const float m_new = fmaxf(m_run, mx);
    if (__builtin_amdgcn_ballot_w64(m_new > m_run) != 0ull) {      // some column's maximum moved
      const float alpha = __builtin_amdgcn_exp2f((m_run - m_new) * ce);
      l_run *= alpha;
#pragma unroll
      for (int c = 0; c < CB; ++c)
#pragma unroll
        for (int v = 0; v < 16; ++v) O[c][v] *= alpha;
      m_run = m_new;
    }
    const float mc = m_run * ce;
    uint32_t ph[4][2], pl[4][2];
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const float e0 = __builtin_amdgcn_exp2f(fmaf(S[4 * i + 2 * t], ce, -mc)), e1 = __builtin_amdgcn_exp2f(fmaf(S[4 * i + 2 * t + 1], ce, -mc));
        sum += e0 + e1;
        const HiLo x = split_bf16(e0, e1);
        ph[i][t] = x.hi;
        pl[i][t] = LO ? x.lo : 0u;
      }
    l_run += sum;
    // lane half h holds keys 16 s + 4 h .. + 3 (chunk 2 s) and 16 s + 8 + 4 h .. + 3 (chunk 2 s + 1); the operand wants 16 s + 8 h .. + 7
    auto operand = [&](const uint32_t (&x)[2], const uint32_t (&y)[2]) {
      const auto a0 = __builtin_amdgcn_permlane32_swap(x[0], y[0], false, false), a1 = __builtin_amdgcn_permlane32_swap(x[1], y[1], false, false);
      return as_bf16x8(u32x4{(uint32_t)a0[0], (uint32_t)a1[0], (uint32_t)a0[1], (uint32_t)a1[1]});
    };
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (s == 0)
#pragma unroll
        for (int c = 0; c < CB; ++c) vv[1][c] = v_frag(1, c);
      const bf16x8 bh = operand(ph[2 * s], ph[2 * s + 1]);
      bf16x8 bl = bh;
      if constexpr (LO) bl = operand(pl[2 * s], pl[2 * s + 1]);
      if (edge) {                                 // entries at or beyond w_end may be stale bytes: 0 * NaN would poison the sum
        const int nv = w_end - (base + 16 * s + 8 * hf);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const uint32_t keep = nv >= 2 * i + 2 ? 0xFFFFFFFFu : (nv == 2 * i + 1 ? 0xFFFFu : 0u);
#pragma unroll
          for (int c = 0; c < CB; ++c) vv[s][c][i] &= keep;
        }
      }
#pragma unroll
      for (int c = 0; c < CB; ++c) O[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vv[s][c]), bh, O[c], 0, 0, 0);
      if (LO)
#pragma unroll
        for (int c = 0; c < CB; ++c) O[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(vv[s][c]), bl, O[c], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  for (int t = 0; t < n_kt; ++t) {
    const int base = t * KB, buf = t & 1;
    // tile t has arrived and every wavefront has left the other buffer
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
    if (t + 1 < n_kt) {
      copy(base + KB, buf ^ 1);
      if (t + 2 < n_kt) pages(base + 2 * KB);
    }
#pragma unroll 1
    for (int kb = 0; kb < 2; ++kb) {
      const int b = base + 32 * kb;
      if (b >= w_end) break;
      step(b, buf, kb);
    }
  }
  if (w_end == 0 || r0 + col >= rows) return;
  const float inv = 1.0f / half_sum(l_run);
  bf16_t* X = a.Xout + (size_t)(r >> 4) * x_stride;
#pragma unroll
  for (int c = 0; c < CB; ++c)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float out4[4] = {O[c][4 * i] * inv, O[c][4 * i + 1] * inv, O[c][4 * i + 2] * inv, O[c][4 * i + 3] * inv};
      xpack_store4<false, LO>(X, (a.nq * DH) >> 5, 16, r & 15, head * DH + 32 * c + 8 * i + 4 * hf, out4);
    }
}

constexpr int ATTN_HEAD_MAX_CTX = 256;    // positions up to which the whole-head kernel is used (one step per wavefront);
                                          // beyond it the arithmetic of a head is worth spreading over several compute units

// Positions per attention workgroup: short ranges give many workgroups but one hand-off record per
// range and query; measured best on MI355X at the 13B-class shape: 128 up to ~768 positions, then
// about total / 4 .. total / 8.
int attn_split_len(int total) {
  if (total <= ATTN_HEAD_MAX_CTX) return ATTN_HEAD_MAX_CTX;       // (one workgroup per head)
  if (total <= 768) return ATTN_SPLIT_LEN;
  if (total <= 1536) return 2 * ATTN_SPLIT_LEN;
  if (total <= 3072) return 4 * ATTN_SPLIT_LEN;
  return 8 * ATTN_SPLIT_LEN;
}

hipError_t launch_attn(const AttnArgs& a, hipStream_t s) {
  if (a.M < 1 || a.M > 16 || a.n_splits < 1 || a.counters == nullptr || a.ldq != a.nq * a.dh) return hipErrorInvalidValue;
  if (a.pos0 + a.M <= ATTN_HEAD_MAX_CTX) {
    if (a.dh == 128) hipLaunchKernelGGL(k_attn_head<128>, dim3(a.nq), dim3(512), 0, s, ATTN_EARLY_ARGS(a), a);
    else if (a.dh == 64) hipLaunchKernelGGL(k_attn_head<64>, dim3(a.nq), dim3(512), 0, s, ATTN_EARLY_ARGS(a), a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
  }
  const dim3 g1(a.nq, a.n_splits);
  if (a.dh == 128) hipLaunchKernelGGL(k_attn_partial<128>, g1, dim3(512), 0, s, ATTN_EARLY_ARGS(a), a);
  else if (a.dh == 64) hipLaunchKernelGGL(k_attn_partial<64>, g1, dim3(512), 0, s, ATTN_EARLY_ARGS(a), a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

// The tiled kernel walks the positions one tile after another, so it needs workgroups for half the compute units: hi + lo, us
// (tiles / groups), 48 heads on one K / V head 333 / 749 at 3001 tokens (1128 workgroups), 40 heads 32 / 39 at 511 (160),
// but 12 heads of 64 channels 20 / 12 at 511 (48); a whole pass of one 13B layer at 130 after 333 (80) 376 / 366
static int attn_tiles_hw_log2(int nq, int nkv) { const int rep = nq / nkv; return rep % 4 == 0 ? 2 : (rep % 2 == 0 ? 1 : 0); }   // log2 of the heads per workgroup
static dim3 attn_tiles_grid(int nq, int nkv, int n_groups) {
  const int hw = attn_tiles_hw_log2(nq, nkv), tbs = (n_groups + 1) / 2, tw = 4 >> hw;
  return dim3(nq >> hw, (tbs + tw - 1) / tw);
}
bool attn_tiles_fit(int nq, int nkv, int dh, int page_tokens, int n_groups) {
  const dim3 g = attn_tiles_grid(nq, nkv, n_groups);
  const bool small_page = 2ull * (unsigned long long)nkv * page_tokens * dh < 1ull << 32;   // the kernel's offsets inside a page are 32 bits wide
  return small_page && page_tokens >= 8 && (page_tokens & (page_tokens - 1)) == 0 && (dh == 64 || dh == 128) && (long)g.x * g.y >= 128;
}

hipError_t launch_attn_groups(const AttnArgs& a, int n_groups, size_t x_stride, bool bf16_operands, hipStream_t s) {
  if (a.M != 16 || n_groups < 1 || n_groups > 65535) return hipErrorInvalidValue;
  if (attn_tiles_fit(a.nq, a.nkv, a.dh, a.page_tokens, n_groups)) {
    const dim3 g = attn_tiles_grid(a.nq, a.nkv, n_groups);
    const int hw = attn_tiles_hw_log2(a.nq, a.nkv);
    if (a.dh == 128) {
      if (bf16_operands) hipLaunchKernelGGL((k_attn_tiles<128, false>), g, dim3(256), 0, s, a, n_groups, x_stride, hw);
      else hipLaunchKernelGGL((k_attn_tiles<128, true>), g, dim3(256), 0, s, a, n_groups, x_stride, hw);
    } else {
      if (bf16_operands) hipLaunchKernelGGL((k_attn_tiles<64, false>), g, dim3(256), 0, s, a, n_groups, x_stride, hw);
      else hipLaunchKernelGGL((k_attn_tiles<64, true>), g, dim3(256), 0, s, a, n_groups, x_stride, hw);
    }
    return hipGetLastError();
  }
  const dim3 g1(a.nq, (n_groups + ATTN_MG - 1) / ATTN_MG);
  if (a.dh == 128) {
    if (bf16_operands) hipLaunchKernelGGL((k_attn_groups<128, false>), g1, dim3(512), 0, s, a.kv_layer, a.page_table, a.q, a.page_tokens, a.nq, a.nkv, a.ldq, a.pos0, n_groups, a, x_stride);
    else hipLaunchKernelGGL((k_attn_groups<128, true>), g1, dim3(512), 0, s, a.kv_layer, a.page_table, a.q, a.page_tokens, a.nq, a.nkv, a.ldq, a.pos0, n_groups, a, x_stride);
  } else if (a.dh == 64) {
    if (bf16_operands) hipLaunchKernelGGL((k_attn_groups<64, false>), g1, dim3(512), 0, s, a.kv_layer, a.page_table, a.q, a.page_tokens, a.nq, a.nkv, a.ldq, a.pos0, n_groups, a, x_stride);
    else hipLaunchKernelGGL((k_attn_groups<64, true>), g1, dim3(512), 0, s, a.kv_layer, a.page_table, a.q, a.page_tokens, a.nq, a.nkv, a.ldq, a.pos0, n_groups, a, x_stride);
  } else return hipErrorInvalidValue;
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Eq. 2 in one launch: soft-max top-10, entropy, arg-max -> classifier -> halt decision
// ---------------------------------------------------------------------------------------------

struct ClfOut {  // mirrors disco_clf_out
  int32_t token; float feats[12]; float score; uint32_t halt; uint32_t executed;
};

constexpr int FEAT_NT = 1024;

// One workgroup, the whole logit vector in registers (V4 float4 per thread, one round of 128-bit
// loads).  Arg-max, soft-max sums and entropy are DPP wave reductions merged across the 16
// wavefronts in a fixed order.  Top-10: every wavefront finds the ten largest of the values its
// lanes hold by ten cross-lane arg-max rounds, and one wavefront picks the ten largest of those 160.
constexpr int CM_NT = 512;     // threads per slice inside the persistent draft loop (its workgroups have 512 threads): 2048 logits
constexpr int CM_SLICE = 1024;     // logits of a workgroup of the many-workgroup launch (32 of them at vocab 32000, 64 at most)
constexpr int CM_MULTI_NT = 256;   // its threads
constexpr int CM_REC = 16;     // floats per record

// Order-preserving map float -> uint32 (larger float <=> larger key; -inf maps above key 0, which marks
// a dropped slot) and back.
__device__ __forceinline__ uint32_t f32_key(float x) {
  const uint32_t u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float key_f32(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}
// Wavefront maximum of unsigned keys: the cross-lane moves fold into the max instructions (one DPP
// instruction per step; 0 is the identity, so lanes a step does not reach keep their value).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_max_u32(uint32_t v) {
  const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, true);
  return v > o ? v : o;
}
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
  v = dpp_max_u32<DPP_QUAD_XOR1, 0xF>(v);
  v = dpp_max_u32<DPP_QUAD_XOR2, 0xF>(v);
  v = dpp_max_u32<DPP_ROW_HALF_MIRROR, 0xF>(v);
  v = dpp_max_u32<DPP_ROW_MIRROR, 0xF>(v);
  v = dpp_max_u32<DPP_ROW_BCAST15, 0xA>(v);
  v = dpp_max_u32<DPP_ROW_BCAST31, 0xC>(v);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The ten largest of the N values per lane held by one wavefront, descending, written by lane 0 to
// out10: ten rounds of a cross-lane maximum over order-preserving integer keys; the first lane that
// holds the maximum drops one instance of it (branch-free).  No LDS traffic and no workgroup barrier
// inside; c is consumed.
template <int N>
__device__ __forceinline__ void wave_top10(float (&c)[N], float* out10) {
  const int lane = threadIdx.x & 63;
  uint32_t k[N];
#pragma unroll
  for (int e = 0; e < N; ++e) k[e] = f32_key(c[e]);
#pragma unroll 1
  for (int rnd = 0; rnd < 10; ++rnd) {
    uint32_t cur = k[0];
#pragma unroll
    for (int e = 1; e < N; ++e) cur = cur > k[e] ? cur : k[e];
    const uint32_t w = wave_max_u32(cur);
    if (lane == 0) out10[rnd] = key_f32(w);
    const unsigned long long owners = __ballot(cur == w);
    bool drop = owners != 0ull && lane == __builtin_ctzll(owners);
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const bool hit = drop && k[e] == w;
      k[e] = hit ? 0u : k[e];
      drop = drop && !hit;
    }
  }
}

template <int V4>
__global__ __launch_bounds__(FEAT_NT) void k_classify(ClassifyArgs a) {
  ClfOut* out = reinterpret_cast<ClfOut*>(a.out);
  if (a.gate != nullptr && *a.gate != 0u) {
    if (threadIdx.x == 0) out->executed = 0u;
    return;
  }
  __shared__ float sv[FEAT_NT / 64 + 1];
  __shared__ int si[FEAT_NT / 64 + 1];
  __shared__ float wtop[FEAT_NT / 64][10];
  __shared__ float top_s[10];
  __shared__ float feat_s[12];
  const int t = threadIdx.x, V = a.vocab, lane = t & 63, wv = t >> 6;
  const float* x = a.logits;

  float4 r[V4];
#pragma unroll
  for (int i = 0; i < V4; ++i) {
    const int idx = (i * FEAT_NT + t) * 4;
    if (idx + 3 < V) {
      r[i] = *reinterpret_cast<const float4*>(x + idx);
    } else {
      r[i].x = idx < V ? x[idx] : -INFINITY;
      r[i].y = idx + 1 < V ? x[idx + 1] : -INFINITY;
      r[i].z = idx + 2 < V ? x[idx + 2] : -INFINITY;
      r[i].w = -INFINITY;
    }
  }

  // maximum and arg-max (lowest index on ties); `mine` is this thread's own maximum
  VI mine; mine.v = -INFINITY; mine.i = 0x7fffffff;
#pragma unroll
  for (int i = 0; i < V4; ++i) {
    const int idx = (i * FEAT_NT + t) * 4;
    VI y;
    y.v = r[i].x; y.i = idx; mine = vi_best(mine, y);
    y.v = r[i].y; y.i = idx + 1; mine = vi_best(mine, y);
    y.v = r[i].z; y.i = idx + 2; mine = vi_best(mine, y);
    y.v = r[i].w; y.i = idx + 3; mine = vi_best(mine, y);
  }
  VI best = block_argmax<FEAT_NT>(mine, sv, si);
  int force = -1;
  if (a.force_token) { force = *a.force_token; if (force >= V) force = -1; }
  if (force >= 0) {
    const float forced_val = best.v + 4.0f;
    best.v = forced_val; best.i = force;
#pragma unroll
    for (int i = 0; i < V4; ++i) {
      const int idx = (i * FEAT_NT + t) * 4;
      if (force == idx) r[i].x = forced_val;
      if (force == idx + 1) r[i].y = forced_val;
      if (force == idx + 2) r[i].z = forced_val;
      if (force == idx + 3) r[i].w = forced_val;
    }
    if ((force >> 2) % FEAT_NT == t) { mine.v = forced_val; mine.i = force; a.logits[force] = forced_val; }
  }
  const float mx = best.v;

  // S = sum e^(x - max), T = sum e^(x - max) (x - max)
  float S = 0.f, T = 0.f;
#pragma unroll
  for (int i = 0; i < V4; ++i) {
    const float d0 = r[i].x - mx, d1 = r[i].y - mx, d2 = r[i].z - mx, d3 = r[i].w - mx;
    const float e0 = expf(d0), e1 = expf(d1), e2 = expf(d2), e3 = expf(d3);
    S += (e0 + e1) + (e2 + e3);
    // e^(-inf) * (-inf) would be NaN: padded slots contribute nothing
    T += (e0 > 0.f ? e0 * d0 : 0.f) + (e1 > 0.f ? e1 * d1 : 0.f) + (e2 > 0.f ? e2 * d2 : 0.f) + (e3 > 0.f ? e3 * d3 : 0.f);
  }
  S = block_sum<FEAT_NT>(S, sv);
  T = block_sum<FEAT_NT>(T, sv);

  // ten largest logits: every wavefront's ten by cross-lane maximum rounds over the values its lanes
  // hold (the first lane that holds the maximum drops one instance; the row is not needed afterwards),
  // then wavefront 0 picks from the 160 candidates
  {
#pragma unroll 1
    for (int rnd = 0; rnd < 10; ++rnd) {
      float cur = -INFINITY;
#pragma unroll
      for (int i = 0; i < V4; ++i) cur = fmaxf(cur, fmaxf(fmaxf(r[i].x, r[i].y), fmaxf(r[i].z, r[i].w)));
      const float wn = wave_max(cur);
      if (lane == 0) wtop[wv][rnd] = wn;
      const unsigned long long owners = __ballot(cur == wn);
      if (owners != 0ull && lane == __builtin_ctzll(owners)) {
        bool done = false;
#pragma unroll
        for (int i = 0; i < V4; ++i) {
          if (!done && r[i].x == wn) { r[i].x = -INFINITY; done = true; }
          if (!done && r[i].y == wn) { r[i].y = -INFINITY; done = true; }
          if (!done && r[i].z == wn) { r[i].z = -INFINITY; done = true; }
          if (!done && r[i].w == wn) { r[i].w = -INFINITY; done = true; }
        }
      }
    }
    __syncthreads();
    if (wv == 0) {
      float c3[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const int ci = lane + 64 * k;
        c3[k] = ci < (FEAT_NT / 64) * 10 ? wtop[ci / 10][ci % 10] : -INFINITY;
      }
      wave_top10<3>(c3, top_s);
    }
  }
  __syncthreads();
  if (t < 10) feat_s[t] = (top_s[t] == -INFINITY) ? 0.f : expf(top_s[t] - mx) / S;
  if (t == 10) feat_s[10] = logf(S) - T / S;
  if (t == 11) feat_s[11] = a.pos_feature;
  __syncthreads();

  // classifier: hidden unit per thread
  float contrib = 0.f;
  if (a.clf_params && t < a.hidden) {
    const float* W1 = a.clf_params + t * 12;
    float acc = a.clf_params[a.hidden * 12 + t];
#pragma unroll
    for (int i = 0; i < 12; ++i) acc += W1[i] * feat_s[i];
    contrib = fmaxf(acc, 0.f) * a.clf_params[a.hidden * 13 + t];
  }
  const float z = block_sum<FEAT_NT>(contrib, sv);
  if (t == 0) {
    float score = __builtin_nanf("");
    uint32_t halt = a.force_halt ? 1u : 0u;
    if (a.clf_params) {
      score = 1.0f / (1.0f + expf(-(z + a.clf_params[a.hidden * 14])));
      if (score < a.tau) halt = 1u;
    }
    // reference lookahead: a token that differs from the known continuation ends the block and is
    // not part of it (bit 1 of halt)
    bool mismatch = false;
    if (a.ref_token) { const int ref = *a.ref_token; mismatch = ref >= 0 && best.i != ref; }
    if (mismatch) halt = 3u;
    // perplexity rule (App. F's rule-based baseline): the block's draft tokens so far have perplexity
    // exp(-(1/j) sum ln p_i), p_i the draft's probability of its own token (the largest one); above the
    // threshold this token is the block's last.  The running sum sits in the word after sl_count.
    if (a.ppl_threshold > 0.f && a.sl_count) {
      float* nll = reinterpret_cast<float*>(a.sl_count + 1);
      const float sum = *nll - logf(feat_s[0]);
      *nll = sum;
      score = expf(sum / (float)(*a.sl_count + 1));
      if (score > a.ppl_threshold) halt |= 1u;
    }
    out->token = best.i;
#pragma unroll
    for (int i = 0; i < 12; ++i) out->feats[i] = feat_s[i];
    out->score = score; out->halt = halt; out->executed = 1u;
    if (!mismatch) {
      if (a.token_next) *a.token_next = best.i;
      if (a.block_slot) *a.block_slot = best.i;
      if (a.sl_count) *a.sl_count += 1;
    }
    if (a.gate && halt) *a.gate = 1u;
  }
}

// Classifier coefficients of one thread (hidden unit threadIdx.x), fetched early by the caller.
struct ClfCoef { float w1[12]; float b1, w2, b2; };

// {max, arg-max, sum e^(x - max), sum e^(x - max) (x - max)} of some logits, and the same of two sets together.
struct SoftStat { float m; int i; float S, T; };
__device__ __forceinline__ SoftStat stat_rescaled(SoftStat a, const float m) {      // relative to another maximum, m >= a.m
  const float d = a.m - m, f = expf(d);
  a.T = f > 0.f ? f * (a.T + d * a.S) : 0.f;                                        // (nothing was there: 0, not 0 * -inf)
  a.S = a.S == 0.f ? 0.f : f * a.S;                                                 // (a logit that is not a number stays one however small its neighbours)
  return a;
}

// LDS of the computation in one workgroup of NT threads.
template <int NT>
struct ClassifySmem {
  SoftStat st[NT / 64];
  alignas(16) float wtop[NT / 64 * 10];
  alignas(16) float feat[12];
  float top[10], sum[NT / 64 + 1];
  int last;
};

// Score, halting decision and the loop's words, from the features and the classifier's sum z: by one thread.  lost: the features are
// not this row's (a wait has given up): token -1, a score that is not a number, and a halt.
__device__ __forceinline__ void classify_decide(const ClassifyArgs& a, const float* feat_s, const float z, const float b2, const int arg_max, const bool lost = false) {
  const int best_i = lost ? -1 : arg_max;
  ClfOut* out = reinterpret_cast<ClfOut*>(a.out);
  float score = __builtin_nanf("");
  uint32_t halt = a.force_halt ? 1u : 0u;
  if (a.clf_params) {
    score = 1.0f / (1.0f + expf(-(z + b2)));
    if (score < a.tau) halt = 1u;
  }
  // reference lookahead: a token that differs from the known continuation ends the block and is
  // not part of it (bit 1 of halt)
  bool mismatch = false;
  if (a.ref_token) { const int ref = *a.ref_token; mismatch = ref >= 0 && best_i != ref && !lost; }
  if (mismatch) halt = 3u;
  // perplexity rule (App. F's rule-based baseline): the block's draft tokens so far have perplexity
  // exp(-(1/j) sum ln p_i), p_i the draft's probability of its own token (the largest one); above the
  // threshold this token is the block's last.  The running sum sits in the word after sl_count.
  // (the loop's words may have been written by another workgroup of the same launch: hand-off accesses)
  const int sl_before = a.sl_count ? __hip_atomic_load(a.sl_count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
  if (a.ppl_threshold > 0.f && a.sl_count) {
    float* nll = reinterpret_cast<float*>(a.sl_count + 1);
    const float sum = ld_f1<true>(nll) - logf(feat_s[0]);
    st_f1<true>(nll, sum);
    score = expf(sum / (float)(sl_before + 1));
    if (score > a.ppl_threshold) halt |= 1u;
  }
  if (lost) { score = __builtin_nanf(""); halt = 1u; }
  out->token = best_i;
#pragma unroll
  for (int i = 0; i < 12; ++i) out->feats[i] = feat_s[i];
  out->score = score; out->halt = halt; out->executed = 1u;
  if (!mismatch) {
    if (a.token_next) *a.token_next = best_i;
    if (a.block_slot) *a.block_slot = best_i;
    if (a.sl_count) __hip_atomic_store(a.sl_count, sl_before + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (a.gate && halt) __hip_atomic_store(a.gate, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Position of candidate `me` in descending order among NC candidates: how many beat it (larger, or equal with a lower slot): a
// permutation of 0 .. NC - 1 without a dependent cross-lane chain.
template <int NC>
__device__ __forceinline__ int rank_of(const float* cand, const int me, const float mine) {
  float o[NC];
#pragma unroll
  for (int j = 0; j < NC; ++j) o[j] = cand[j];            // all reads in flight at once (broadcasts)
  int rank = 0;
#pragma unroll
  for (int j = 0; j < NC; ++j) rank += (o[j] > mine || (o[j] == mine && j < me)) ? 1 : 0;
  return rank;
}

// Last stage of the feature / classifier computation, run by ONE workgroup of NT threads over nb <= 64
// records {max, arg-max, S, T relative to the record's max, its ten largest values} (16 floats each,
// written with agent-scope stores by the workgroups that reduced the logits).  The first wavefront merges the statistics (a record
// per lane) while the others pick the ten largest of the nb * 10 candidates; then the forced logit in closed
// form, features, classifier, halt decision and the loop's bookkeeping words.  What bounds it is the chain: two selections and the
// hand-off.  Workgroup-wide reductions one after another (a maximum, two sums, the selection; two barriers each, twice) took 10.3 us a
// call at 32000 logits; with reductions inside wavefronts that meet behind one barrier 8.5.
template <int NT>
__device__ __forceinline__ int classify_merge_finish(const ClassifyArgs& a, const float* recs, const int nb, const int force,
                                                      const float xf, const ClfCoef& k, ClassifySmem<NT>& sm) {
  constexpr int NW = NT / 64, NC = (NW - 1) * 10;
  constexpr int CPT = (640 * 256 / NT + (NT - 64) - 1) / (NT - 64);          // at most 64 slices (65536 logits at NT = 256): 640 candidates
  ClfOut* out = reinterpret_cast<ClfOut*>(a.out);
  const int t = threadIdx.x, wv = t >> 6;
  float* top_s = sm.top;
  float* feat_s = sm.feat;
  if (wv == 0) {
    SoftStat r{-INFINITY, 0x7fffffff, 0.f, 0.f};
    if (t < nb) {
      const float2 p0 = ld_agent2(recs + (size_t)t * CM_REC), p1 = ld_agent2(recs + (size_t)t * CM_REC + 2);
      r = SoftStat{p0.x, __float_as_int(p0.y), p1.x, p1.y};
    }
    const VI best = wave_argmax(VI{r.m, r.i});
    r = stat_rescaled(r, best.v);
    const float S = wave_sum(r.S), T = wave_sum(r.T);
    if (t == 0) sm.st[0] = SoftStat{best.v, best.i, S, T};
  } else {
    float cc[CPT];
#pragma unroll
    for (int q = 0; q < CPT; ++q) {
      const int ci = t - 64 + q * (NT - 64);                 // candidate ci = record ci / 10, slot ci % 10
      cc[q] = ci < nb * 10 ? ld_f1<true>(recs + (size_t)(ci / 10) * CM_REC + 4 + ci % 10) : -INFINITY;
    }
    wave_top10<CPT>(cc, sm.wtop + (wv - 1) * 10);
  }
  __syncthreads();
  float mx = sm.st[0].m, Sg = sm.st[0].S, Tg = sm.st[0].T;
  int best_i = sm.st[0].i;
  if (t < NC) {
    const float mine = sm.wtop[t];
    const int rank = rank_of<NC>(sm.wtop, t, mine);
    if (rank < 10) {
      if (force < 0) feat_s[rank] = (mine == -INFINITY) ? 0.f : expf(mine - mx) / Sg;
      else top_s[rank] = mine;
    }
  }
  if (force >= 0) {
    __syncthreads();
    // raise logit[force] from x_f to M + 4: shift every term to the new maximum, take the old
    // contribution of x_f out and put the new one (e^0 = 1, with (x - max) = 0) in
    const float mnew = mx + 4.0f;
    const float sh = expf(-4.0f), ef = expf(xf - mnew);
    Tg = sh * (Tg - 4.0f * Sg) - (ef > 0.f ? ef * (xf - mnew) : 0.f);
    Sg = sh * Sg - ef + 1.0f;
    if (t == 0) {
      // new top ten: M + 4 first, then the old ones without one instance of x_f (or without the last)
      float old[10];
      for (int i = 0; i < 10; ++i) old[i] = top_s[i];
      int drop = 9;
      for (int i = 9; i >= 0; --i) if (old[i] == xf) drop = i;
      top_s[0] = mnew;
      for (int i = 0, o = 1; i < 10 && o < 10; ++i) if (i != drop) top_s[o++] = old[i];
      st_f1<true>(a.logits + force, mnew);
    }
    mx = mnew; best_i = force;
    __syncthreads();
    if (t < 10) feat_s[t] = (top_s[t] == -INFINITY) ? 0.f : expf(top_s[t] - mx) / Sg;
  }
  if (t == NT - 1) feat_s[10] = logf(Sg) - Tg / Sg;
  if (t == NT - 2) feat_s[11] = a.pos_feature;
  __syncthreads();
  float contrib = 0.f;
  if (a.clf_params && t < a.hidden) {
    float acc = k.b1;
#pragma unroll
    for (int i = 0; i < 12; ++i) acc += k.w1[i] * feat_s[i];
    contrib = fmaxf(acc, 0.f) * k.w2;
  }
  float z = wave_sum(contrib);
  if (a.hidden > 64) z = block_sum<NT>(contrib, sm.sum);     // (up to 64 units: all in the first wavefront, which finishes)
  if (t == 0) classify_decide(a, feat_s, z, k.b2, best_i);
  // (the launch of many workgroups polls these records: they are left empty)
  for (int i = t; i < nb * CM_REC; i += NT) __hip_atomic_store(reinterpret_cast<uint32_t*>(const_cast<float*>(recs)) + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return best_i;
}

// The same computation spread over ceil(V / (4 NT)) workgroups of a persistent launch.  Each workgroup reduces its slice of the logits (4 per thread) to a record {max, arg-max, S, T relative to its own
// max, its ten largest values}; the last workgroup to finish (ticket, no waiting) merges the
// records in index order: S = sum S_b e^(m_b - M), T = sum e^(m_b - M) (T_b + (m_b - M) S_b), the ten
// largest of the records' candidates (ten per record), then features, classifier and halt decision.  Forcing a token
// to max + 4 is applied to the merged sums in closed form.
// b = index of this workgroup's slice of NT * 4 logits, nb = number of slices.  Returns the arg-max token in
// every thread of the workgroup that finished the computation (the last to arrive), -1 in all others.
// The logits were written by other workgroups of the same launch.
template <int NT>
__device__ __forceinline__ int classify_unit(const ClassifyArgs& a, const int b, const int nb, const uint32_t halted) {
  constexpr int NW = NT / 64;
  ClfOut* out = reinterpret_cast<ClfOut*>(a.out);
  __shared__ ClassifySmem<NT> sm;
  const int t = threadIdx.x, V = a.vocab;
  const float* x = a.logits;
  float* rec = a.scratch + 64 + (size_t)b * CM_REC;          // scratch[0] is the ticket counter
  const int idx = (b * NT + t) * 4;
  float r4[4];
  if (idx + 3 < V) {
    const float4 v = ld_f4<true>(x + idx);
    r4[0] = v.x; r4[1] = v.y; r4[2] = v.z; r4[3] = v.w;
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) r4[e] = idx + e < V ? ld_f1<true>(x + idx + e) : -INFINITY;
  }
  // operands of the final stage that depend on no reduction are fetched now, so that the merging
  // workgroup does not pay their round trips one after another at the end
  int force = -1;
  float xf = 0.f;
  if (a.force_token) { force = *a.force_token; if (force >= V) force = -1; }
  if (force >= 0) xf = ld_f1<true>(x + force);
  float w1[12], cb1 = 0.f, cw2 = 0.f, cb2 = 0.f;
#pragma unroll
  for (int i = 0; i < 12; ++i) w1[i] = 0.f;
  if (a.clf_params) {
    cb2 = a.clf_params[a.hidden * 14];
    if (t < a.hidden) {
#pragma unroll
      for (int i = 0; i < 12; ++i) w1[i] = a.clf_params[t * 12 + i];
      cb1 = a.clf_params[a.hidden * 12 + t];
      cw2 = a.clf_params[a.hidden * 13 + t];
    }
  }
  if (flag_set(halted)) {                         // uniform over the launch; the loads above are dropped
    if (threadIdx.x == 0 && b == 0) out->executed = 0u;
    return -1;
  }
  // every wavefront reduces its own 256 logits; the workgroup's record is merged from those behind one barrier
  const int wv = t >> 6;
  VI mine; mine.v = -INFINITY; mine.i = 0x7fffffff;
#pragma unroll
  for (int e = 0; e < 4; ++e) { VI y; y.v = r4[e]; y.i = idx + e; mine = vi_best(mine, y); }
  const VI wb = wave_argmax(mine);
  float S = 0.f, T = 0.f;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float d = r4[e] - wb.v, ex = r4[e] == -INFINITY ? 0.f : expf(d);
    S += ex; T += ex > 0.f ? ex * d : 0.f;
  }
  S = wave_sum(S); T = wave_sum(T);
  if ((t & 63) == 0) sm.st[wv] = SoftStat{wb.v, wb.i, S, T};
  wave_top10<4>(r4, sm.wtop + wv * 10);
  __syncthreads();
  if (t < NW * 10) {
    const float v = sm.wtop[t];
    const int rank = rank_of<NW * 10>(sm.wtop, t, v);
    if (rank < 10) st_f1<true>(rec + 4 + rank, v);
  }
  if (t == NT - 1) {
    VI best{sm.st[0].m, sm.st[0].i};
#pragma unroll
    for (int w = 1; w < NW; ++w) best = vi_best(best, VI{sm.st[w].m, sm.st[w].i});
    float Sg = 0.f, Tg = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { const SoftStat r = stat_rescaled(sm.st[w], best.v); Sg += r.S; Tg += r.T; }
    st_agent2(rec, best.v, __int_as_float(best.i)); st_agent2(rec + 2, Sg, Tg);
  }
  if (!last_arrival(reinterpret_cast<int*>(a.scratch), nb, &sm.last)) return -1;

  ClfCoef k;
#pragma unroll
  for (int i = 0; i < 12; ++i) k.w1[i] = w1[i];
  k.b1 = cb1; k.w2 = cw2; k.b2 = cb2;
  return classify_merge_finish<NT>(a, a.scratch + 64, nb, force, xf, k, sm);
}

// The ten largest of a wavefront's keys (N a lane; 0: none), as a list of candidates: a lower bound of the tenth largest, and every key that reaches it.
// The lanes' maxima are taken over four lanes (16 groups); ten of those reach the tenth largest of them, which is the bound (about 15 of 1024
// keys pass it).  Ten rounds of a wavefront-wide maximum, one key out per round, are a chain of 1 us; they remain for lists that do not fit
// (many equal keys).
__device__ __forceinline__ uint32_t row4_max_u32(uint32_t v) {
  const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  const uint32_t m = max(r[0], r[1]);
  const auto q = __builtin_amdgcn_permlane32_swap(m, m, false, false);
  return max(q[0], q[1]);
}
template <int D> __device__ __forceinline__ int reaches(const uint32_t g) {           // whether the lane D further on in the row has a key >= g
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)g, 0x120 + D, 0xF, 0xF, false) >= g ? 1 : 0;
}
__device__ __forceinline__ uint32_t tenth_bound(uint32_t g /* the lane's maximum */) {
  g = row4_max_u32(g);
  const int c = 1 + ((((reaches<1>(g) + reaches<2>(g)) + (reaches<3>(g) + reaches<4>(g))) + ((reaches<5>(g) + reaches<6>(g)) + (reaches<7>(g) + reaches<8>(g)))) +
                     (((reaches<9>(g) + reaches<10>(g)) + (reaches<11>(g) + reaches<12>(g))) + ((reaches<13>(g) + reaches<14>(g)) + reaches<15>(g))));
  uint32_t t = c >= 10 ? g : 0u;                  // the largest of those that ten reach: the same in every row of 16 lanes
  t = dpp_max_u32<DPP_QUAD_XOR1, 0xF>(t);
  t = dpp_max_u32<DPP_QUAD_XOR2, 0xF>(t);
  t = dpp_max_u32<DPP_ROW_HALF_MIRROR, 0xF>(t);
  return dpp_max_u32<DPP_ROW_MIRROR, 0xF>(t);
}
// As wave_top10, over keys.
template <int N>
__device__ __forceinline__ void rounds_of_ten(uint32_t (&k)[N], uint32_t* out10) {
  const int lane = threadIdx.x & 63;
#pragma unroll 1
  for (int rnd = 0; rnd < 10; ++rnd) {
    uint32_t cur = k[0];
#pragma unroll
    for (int e = 1; e < N; ++e) cur = max(cur, k[e]);
    const uint32_t w = wave_max_u32(cur);
    if (w == 0u) break;                           // none left
    if (lane == 0) out10[rnd] = w;
    const unsigned long long owners = __ballot(cur == w);
    bool drop = lane == __builtin_ctzll(owners);
#pragma unroll
    for (int e = 0; e < N; ++e) {
      const bool hit = drop && k[e] == w;
      k[e] = hit ? 0u : k[e];
      drop = drop && !hit;
    }
  }
}
// Appends the keys >= bound to list (64 places); returns how many there are (more than 64: the list is not complete).  SORTED: a lane's keys descend.
template <int N, bool SORTED>
__device__ __forceinline__ int append_keys(const uint32_t (&k)[N], const uint32_t bound, uint32_t* list) {
  int n = 0;
#pragma unroll
  for (int e = 0; e < N; ++e) {
    const bool in = k[e] >= bound;
    const unsigned long long b = __ballot(in);
    if (SORTED && b == 0ull) break;
    const int at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
    if (in && at < 64) list[at] = k[e];
    n += __builtin_popcountll(b);
  }
  __builtin_amdgcn_wave_barrier();
  return n;
}
// The ten largest keys (of them those that reach the bound) in descending order to out10 (LDS; places without a key: minus infinity's).  list: 64 words of LDS.
constexpr uint32_t KEY_NEG_INF = 0x007FFFFFu;
template <int N, bool SORTED>
__device__ __forceinline__ void select_ten(uint32_t (&k)[N], const uint32_t bound, uint32_t* list, uint32_t* out10) {
  const int lane = threadIdx.x & 63;
  if (lane < 10) out10[lane] = KEY_NEG_INF;
  const int n = append_keys<N, SORTED>(k, bound, list);
  if (n > 64) { rounds_of_ten(k, out10); return; }
  // position of a candidate: how many beat it (larger, or equal and in front of it); lanes without one hold 0, which beats none
  const uint32_t v = lane < n ? list[lane] : 0u;
  int rank = 0;
#pragma unroll 1
  for (int j0 = 0; j0 < n; j0 += 8) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)v, j0 + q);
      rank += o > (lane > j0 + q ? v - 1u : v) ? 1 : 0;
    }
  }
  if (lane < n && rank < 10) out10[rank] = v;
  __builtin_amdgcn_wave_barrier();
}

// The many-workgroup form.  A workgroup reduces 1024 logits to a record of 16 words: {max, arg-max + 1, S, T, its ten largest}, floats as their
// order-preserving keys, so that no word is 0.  The LAST workgroup of the grid polls the records until no word is 0 (the data is its own flag, see
// k_chain; a record's statistics and its largest leave from two wavefronts, a store instruction each), merges them and leaves them at 0 for the next
// launch.  It waits for workgroups that were started before it, and not without a bound: after `limit` polls it reports token -1, a score that is not
// a number, and a halt, and marks the scratch (abort_word).  A workgroup that was late then leaves a record that nothing clears, so every later launch on a marked
// scratch reports the same, until it is initialised.  What bounds it: a chain of dependent instructions, of about ten cycles each: load 0.7 us, a wavefront's 256 logits 1.1, the
// workgroup's 1.4, hand-off 1, final selection 1, features and classifier 1.  32000 logits 8.5 -> 7.65 us a call (a ticket, 0.3 us, and a load in place of the
// polls, ten rounds of maxima in place of the candidate lists; one wavefront for all 1024 logits of a workgroup 8.5: 3.4 us for the first two).
struct MultiSmem {
  alignas(16) uint32_t list[4][64], all[64], top[12];
  uint32_t n[4], bound[4];
  SoftStat st[4], best;
  alignas(16) float feat[12];
  float sum[CM_MULTI_NT / 64 + 1];
  int lost[2];                         // of the two polling wavefronts
  int last;
};
// POLL false (launch mode 2): no workgroup waits; the last of the nb to arrive, by a ticket, merges.
template <bool POLL>
__global__ __launch_bounds__(CM_MULTI_NT) void k_classify_multi(float* logits, const float* clf_params, const int32_t* force_token, uint32_t* gate, float* scratch,
                                                                int vocab, int hidden, ClassifyArgs a) {
  a.logits = logits; a.clf_params = clf_params; a.force_token = force_token; a.gate = gate; a.scratch = scratch; a.vocab = vocab; a.hidden = hidden;
  __shared__ MultiSmem sm;
  const int t = threadIdx.x, lane = t & 63, wv = __builtin_amdgcn_readfirstlane(t >> 6), V = vocab, b = blockIdx.x, nb = gridDim.x - (POLL ? 1 : 0);
  const uint32_t halted = gate_request(gate);
  uint32_t* recs = reinterpret_cast<uint32_t*>(scratch + 64);
  if (b < nb) {
    const int idx = (b * CM_MULTI_NT + t) * 4;
    float r[4];
    uint32_t key[4];
    if (idx + 3 < V) {
      const float4 v = *reinterpret_cast<const float4*>(logits + idx);
      r[0] = v.x; r[1] = v.y; r[2] = v.z; r[3] = v.w;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) r[e] = idx + e < V ? logits[idx + e] : -INFINITY;
    }
    if (flag_set(halted)) {                       // uniform over the launch; the loads above are dropped
      if (t == 0 && b == 0) reinterpret_cast<ClfOut*>(a.out)->executed = 0u;
      return;
    }
    // every wavefront reduces its own 256 logits
    {
      VI mine{-INFINITY, 0x7fffffff};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        mine = vi_best(mine, VI{r[e], idx + e});
        key[e] = idx + e < V ? f32_key(r[e]) : 0u;
      }
      const uint32_t bound = max(tenth_bound(max(max(key[0], key[1]), max(key[2], key[3]))), 1u);
      int n = append_keys<4, false>(key, bound, sm.list[wv]);
      const VI wb = wave_argmax(mine);
      float S = 0.f, T = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float d = r[e] - wb.v, ex = r[e] == -INFINITY ? 0.f : expf(d);
        S += ex; T += ex > 0.f ? ex * d : 0.f;
      }
      S = wave_sum(S); T = wave_sum(T);
      if (n > 64) {
        if (lane < 10) sm.list[wv][lane] = 0u;
        rounds_of_ten(key, sm.list[wv]);
        n = 10;
      }
      if (lane == 0) { sm.st[wv] = SoftStat{wb.v, wb.i, S, T}; sm.bound[wv] = bound; sm.n[wv] = (uint32_t)n; }
    }
    __syncthreads();
    if (wv == 0) {                                // the workgroup's ten largest, from the wavefronts' candidates
      const uint32_t bound = max(max(sm.bound[0], sm.bound[1]), max(sm.bound[2], sm.bound[3]));
#pragma unroll
      for (int w = 0; w < 4; ++w) { const uint32_t c = sm.list[w][lane]; key[w] = (uint32_t)lane < sm.n[w] ? c : 0u; }
      select_ten<4, false>(key, bound, sm.all, sm.top);
      if (lane < 12)
        __hip_atomic_store(recs + b * CM_REC + 4 + lane, max(sm.top[min(lane, 9)], 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);      // (a key is 0 for one bit pattern of a NaN)
    } else if (wv == 1) {                         // its statistics, a wavefront's in each of four lanes
      SoftStat q = sm.st[lane & 3];
      VI best = vi_step<DPP_QUAD_XOR1, 0xF>(VI{q.m, q.i});
      best = vi_step<DPP_QUAD_XOR2, 0xF>(best);
      q = stat_rescaled(q, best.v);
      float Sg = 0.f, Tg = 0.f;
      Sg += dpp_f<0x00, 0xF>(0.f, q.S); Sg += dpp_f<0x55, 0xF>(0.f, q.S); Sg += dpp_f<0xAA, 0xF>(0.f, q.S); Sg += dpp_f<0xFF, 0xF>(0.f, q.S);
      Tg += dpp_f<0x00, 0xF>(0.f, q.T); Tg += dpp_f<0x55, 0xF>(0.f, q.T); Tg += dpp_f<0xAA, 0xF>(0.f, q.T); Tg += dpp_f<0xFF, 0xF>(0.f, q.T);
      const uint32_t w = lane == 0 ? f32_key(best.v) : (lane == 1 ? (uint32_t)best.i + 1u : f32_key(lane == 2 ? Sg : Tg));
      if (lane < 4) __hip_atomic_store(recs + b * CM_REC + lane, max(w, 1u), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (POLL) return;
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);                // this wavefront's write-through stores have completed
    __syncthreads();
    if (t == 0) {
      int* ticket = reinterpret_cast<int*>(scratch);
      sm.last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nb - 1 ? 1 : 0;
      if (sm.last != 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (sm.last == 0) return;
  }
  // the last workgroup; operands of the final stage that depend on no record first
  int force = -1;
  float xf = 0.f;
  ClfCoef k;
#pragma unroll
  for (int i = 0; i < 12; ++i) k.w1[i] = 0.f;
  k.b1 = 0.f; k.w2 = 0.f; k.b2 = 0.f;
  if (force_token) { force = *force_token; if (force >= V) force = -1; }
  if (force >= 0) xf = logits[force];
  const uint32_t lost_before = __hip_atomic_load(a.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (clf_params) {
    k.b2 = clf_params[hidden * 14];
    if (t < hidden) {
#pragma unroll
      for (int i = 0; i < 12; ++i) k.w1[i] = clf_params[t * 12 + i];
      k.b1 = clf_params[hidden * 12 + t];
      k.w2 = clf_params[hidden * 13 + t];
    }
  }
  if (flag_set(halted)) return;
  if (wv == 1 || wv == 2) {
    // a record per lane: the first wavefront of the two selects, the other merges the statistics
    constexpr int Q = 3;
    const uint32_t* rec = recs + min(lane, nb - 1) * CM_REC;
    const int q0 = wv == 1 ? 1 : 0, nq = wv == 1 ? Q : 1;
    u32x4 v[Q];
    bool lost = POLL && a.limit < 0;
    for (int spins = 0;; ++spins) {
      bool ok = true;
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const unsigned long long* p = reinterpret_cast<const unsigned long long*>(rec + (q0 + (q < nq ? q : 0)) * 4);
        const unsigned long long x = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), y = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        v[q] = u32x4{(uint32_t)x, (uint32_t)(x >> 32), (uint32_t)y, (uint32_t)(y >> 32)};
        ok = ok && v[q][0] != 0u && v[q][1] != 0u && v[q][2] != 0u && v[q][3] != 0u;
      }
      if (!POLL || lost || __ballot(!ok) == 0ull) break;      // (the ticket says that all records are there)
      if (spins >= a.limit) { lost = true; break; }
    }
    if (lane == 0) {
      sm.lost[wv - 1] = lost ? 1 : 0;
      if (lost) __hip_atomic_store(a.abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (lane < nb) {                              // empty for the next launch
#pragma unroll
      for (int q = 0; q < Q; ++q)
        if (q < nq) *reinterpret_cast<u32x4*>(recs + lane * CM_REC + (q0 + q) * 4) = u32x4{0u, 0u, 0u, 0u};
    }
    if (wv == 1) {
      uint32_t key[10];
#pragma unroll
      for (int e = 0; e < 10; ++e) key[e] = lane < nb ? v[e >> 2][e & 3] : 0u;
      select_ten<10, true>(key, max(tenth_bound(key[0]), 1u), sm.all, sm.top);
    } else {
      SoftStat r{-INFINITY, 0x7fffffff, 0.f, 0.f};
      if (lane < nb) r = SoftStat{key_f32(v[0][0]), (int)(v[0][1] - 1u), key_f32(v[0][2]), key_f32(v[0][3])};
      const VI best = wave_argmax(VI{r.m, r.i});
      r = stat_rescaled(r, best.v);
      const float S = wave_sum(r.S), T = wave_sum(r.T);
      if (lane == 0) sm.best = SoftStat{best.v, best.i, S, T};
    }
  }
  __syncthreads();
  float mx = sm.best.m, Sg = sm.best.S, Tg = sm.best.T;
  int best_i = sm.best.i;
  if (wv == 0) {
    float top = lane < 10 ? key_f32(sm.top[lane]) : -INFINITY;
    if (force >= 0) {
      // raise logit[force] from x_f to M + 4: shift every term to the new maximum, take the old
      // contribution of x_f out and put the new one (e^0 = 1, with (x - max) = 0) in
      const float mnew = mx + 4.0f;
      const float sh = expf(-4.0f), ef = expf(xf - mnew);
      Tg = sh * (Tg - 4.0f * Sg) - (ef > 0.f ? ef * (xf - mnew) : 0.f);
      Sg = sh * Sg - ef + 1.0f;
      // new top ten: M + 4 first, then the old ones without one instance of x_f (or without the last)
      const unsigned long long same = __ballot(lane < 10 && top == xf);
      const int drop = same != 0ull ? __builtin_ctzll(same) : 9;
      const float before = __shfl(top, max(lane - 1, 0));
      top = lane == 0 ? mnew : (lane <= drop ? before : top);
      if (lane == 0) a.logits[force] = mnew;
      mx = mnew; best_i = force;
    }
    if (lane < 10) sm.feat[lane] = (top == -INFINITY) ? 0.f : expf(top - mx) / Sg;
    if (lane == 10) sm.feat[10] = logf(Sg) - Tg / Sg;
    if (lane == 11) sm.feat[11] = a.pos_feature;
    __builtin_amdgcn_wave_barrier();
  }
  if (hidden > 64) __syncthreads();
  else if (wv != 0) return;                       // (up to 64 units: all in the first wavefront, which finishes)
  float contrib = 0.f;
  if (clf_params && t < hidden) {
    float acc = k.b1;
#pragma unroll
    for (int i = 0; i < 12; ++i) acc += k.w1[i] * sm.feat[i];
    contrib = fmaxf(acc, 0.f) * k.w2;
  }
  const float z = hidden > 64 ? block_sum<CM_MULTI_NT>(contrib, sm.sum) : wave_sum(contrib);
  if (t == 0) {
    // (the two poll different words, so one of them can give up alone)
    classify_decide(a, sm.feat, z, k.b2, best_i, (sm.lost[0] | sm.lost[1]) != 0 || flag_set(lost_before));
  }
}

hipError_t launch_classify(const ClassifyArgs& a, hipStream_t s) {
  if (a.vocab < 1 || a.vocab > 65536) return hipErrorInvalidValue;
  if (a.scratch != nullptr && a.vocab >= 4096) {
    if (a.abort_word == nullptr) return hipErrorInvalidValue;
    // 32000 logits, kernel time: 6.97 us polling, 7.27 by tickets
    const int nb = (a.vocab + CM_SLICE - 1) / CM_SLICE;
    if (a.ticket) hipLaunchKernelGGL(k_classify_multi<false>, dim3(nb), dim3(CM_MULTI_NT), 0, s, a.logits, a.clf_params, a.force_token, a.gate, a.scratch, a.vocab, a.hidden, a);
    else hipLaunchKernelGGL(k_classify_multi<true>, dim3(nb + 1), dim3(CM_MULTI_NT), 0, s, a.logits, a.clf_params, a.force_token, a.gate, a.scratch, a.vocab, a.hidden, a);
    return hipGetLastError();
  }
  if (a.vocab <= 8192) hipLaunchKernelGGL(k_classify<2>, dim3(1), dim3(FEAT_NT), 0, s, a);
  else if (a.vocab <= 32768) hipLaunchKernelGGL(k_classify<8>, dim3(1), dim3(FEAT_NT), 0, s, a);
  else hipLaunchKernelGGL(k_classify<16>, dim3(1), dim3(FEAT_NT), 0, s, a);
  return hipGetLastError();
}

// Scratch of the allocation-free form of the classify call (callers that cannot allocate): one copy of
// this array per GPU, held from module load until the process ends.  In host code the name is only a
// handle for hipGetSymbolAddress; kernels and clears get the device address looked up below.
static __device__ __align__(256) unsigned char scratch[CLASSIFY_SCRATCH_BYTES];

constexpr int MAX_DEVICES = 64;
static std::mutex g_scratch_mu;
static float* g_scratch_ptr[MAX_DEVICES];        // device address of `scratch` on each GPU, once looked up

// Device address of the current GPU's copy of `scratch` (looked up once per device, with that device current).
hipError_t classify_static_scratch(float** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (p == nullptr) return hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

// ---------------------------------------------------------------------------------------------
// per-row arg-max of the verification logits; acceptance; KV fill; draft-loop bookkeeping
// ---------------------------------------------------------------------------------------------

// abort_word (may be null): set by a persistent forward whose grid barrier gave up; the rows then get -1.
__global__ __launch_bounds__(1024) void k_argmax_rows(const float* __restrict__ logits, int vocab, int32_t* __restrict__ out,
                                                      const unsigned* abort_word) {
  __shared__ float sv[17];
  __shared__ int si[17];
  const float* x = logits + (size_t)blockIdx.x * vocab;
  VI mine; mine.v = -INFINITY; mine.i = 0x7fffffff;
  if ((vocab & 3) == 0 && (reinterpret_cast<uintptr_t>(x) & 15) == 0) {
    // eight 128-bit loads per thread in flight at once (a row of 32768 logits in one round), then the comparisons
    const float4* x4 = reinterpret_cast<const float4*>(x);
    const int n4 = vocab >> 2;
    for (int base = 0; base < n4; base += 8 * 1024) {
      float4 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = base + k * 1024 + threadIdx.x;
        v[k] = i < n4 ? x4[i] : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int i = 4 * (base + k * 1024 + threadIdx.x);
        const float e[4] = {v[k].x, v[k].y, v[k].z, v[k].w};
#pragma unroll
        for (int c = 0; c < 4; ++c) { VI y; y.v = e[c]; y.i = i + c; if (i + c < vocab) mine = vi_best(mine, y); }
      }
    }
  } else {
    for (int i = threadIdx.x; i < vocab; i += 1024) { VI y; y.v = x[i]; y.i = i; mine = vi_best(mine, y); }
  }
  const VI b = block_argmax<1024>(mine, sv, si);
  if (threadIdx.x == 0) out[blockIdx.x] = (abort_word != nullptr && *abort_word != 0u) ? -1 : b.i;
}

hipError_t launch_argmax_rows(const float* logits, int M, int vocab, int32_t* out, const unsigned* abort_word, hipStream_t s) {
  hipLaunchKernelGGL(k_argmax_rows, dim3(M), dim3(1024), 0, s, logits, vocab, out, abort_word);
  return hipGetLastError();
}

struct AcceptOut { int32_t n; int32_t n_emit; int32_t emit[16]; };

__global__ void k_accept(const int32_t* block, const int32_t* argmax, int n_block, const int32_t* dev_n_block,
                         AcceptOut* out, AcceptOut* host_out) {
  if (threadIdx.x != 0) return;
  int nb = n_block;
  if (dev_n_block) { const int v = *dev_n_block; nb = v < 1 ? 1 : (v > n_block ? n_block : v); }
  int n = 0;
  while (n < nb - 1 && block[n + 1] == argmax[n]) ++n;
  AcceptOut r;
  r.n = n; r.n_emit = n + 1;
  for (int i = 0; i < 16; ++i) r.emit[i] = (i < n) ? block[i + 1] : (i == n ? argmax[n] : -1);
  *out = r;
  if (host_out) { *host_out = r; __threadfence_system(); }
}

hipError_t launch_accept(const int32_t* block, const int32_t* argmax, int n_block, const int32_t* dev_n_block,
                         void* dev_out, void* host_out, hipStream_t s) {
  hipLaunchKernelGGL(k_accept, dim3(1), dim3(64), 0, s, block, argmax, n_block, dev_n_block,
                     reinterpret_cast<AcceptOut*>(dev_out), reinterpret_cast<AcceptOut*>(host_out));
  return hipGetLastError();
}

__global__ __launch_bounds__(256) void k_kv_fill(const bf16_t* __restrict__ src, bf16_t* __restrict__ pages,
                                                 const int32_t* __restrict__ page_table, int n_layers, int n_pages,
                                                 int pt, int nkv, int dh, int ctx) {
  // src [layer][sel][pos][kvh][dh]; one thread per 8 elements
  const int64_t vec_per_row = dh / 8;
  const int64_t total = (int64_t)n_layers * 2 * ctx * nkv * vec_per_row;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < total; i += (int64_t)gridDim.x * 256) {
    int64_t r = i;
    const int cv = (int)(r % vec_per_row); r /= vec_per_row;
    const int kvh = (int)(r % nkv); r /= nkv;
    const int pos = (int)(r % ctx); r /= ctx;
    const int sel = (int)(r % 2); r /= 2;
    const int layer = (int)r;
    const int lp = pos / pt, off = pos % pt;
    const int pp = page_table ? page_table[lp] : lp;
    const size_t blk = ((((size_t)layer * n_pages + pp) * 2 + sel) * nkv + kvh) * pt * dh;
    const uint4 val = *reinterpret_cast<const uint4*>(src + i * 8);
    if (sel == 0) {                                   // K: [token][d_head]
      *reinterpret_cast<uint4*>(pages + blk + (size_t)off * dh + cv * 8) = val;
    } else {                                          // V: transposed, [d_head][token]
      const uint32_t wv[4] = {val.x, val.y, val.z, val.w};
#pragma unroll
      for (int e = 0; e < 8; ++e)
        pages[blk + (size_t)(cv * 8 + e) * pt + off] = (bf16_t)(wv[e >> 1] >> ((e & 1) * 16));
    }
  }
}

hipError_t launch_kv_fill(const bf16_t* src, bf16_t* pages, const int32_t* page_table, int n_layers, int n_pages,
                          int page_tokens, int nkv, int dh, int ctx, hipStream_t s) {
  const int64_t total = (int64_t)n_layers * 2 * ctx * nkv * (dh / 8);
  int64_t blocks = (total + 255) / 256;
  if (blocks > 16384) blocks = 16384;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_kv_fill, dim3((unsigned)blocks), dim3(256), 0, s, src, pages, page_table, n_layers, n_pages,
                     page_tokens, nkv, dh, ctx);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// sampling at temperature > 0: draws by inverse CDF in vocabulary order, speculative acceptance
// ---------------------------------------------------------------------------------------------
//
// One workgroup of 1024 threads per row; the row lives in registers (V4 float4 per thread, one round of 128-bit loads).
// Wavefront w holds the w-th sixteenth of the row (nseg segments of 256 consecutive elements, four per lane), so the
// cumulative sum in vocabulary order is wavefront by wavefront, segment by segment, lane by lane: sixteen totals in LDS
// tell every wavefront whether the draw falls into its part, and only that wavefront scans its segments and its lanes.
// (Scanning every segment across the whole workgroup, as before, read 256 LDS words per thread: 29 us for five rows of
// 32000, 8.8 us now.)  All sums are fp32.  The exponential is expf: a shorter form on the hardware's exp2 took 0.4 us less for
// a block of five at 32000 (17.4 of 17.8 us) and 3.6 us at 65536 (of 32.6), but flushed weights below 2^-126 to zero, and its
// rows were further from 64 bits (4.4e-8 rms of a weight against 3.6e-8).

constexpr int SMP_NT = 1024;
constexpr int SMP_NW = SMP_NT / 64;

__device__ __forceinline__ int smp_segments(int V) { return (V + 4 * SMP_NT - 1) / (4 * SMP_NT); }   // per wavefront, <= V4
__device__ __forceinline__ int smp_index(int i, int nseg) {
  return (((int)(threadIdx.x >> 6) * nseg + i) * 64 + (int)(threadIdx.x & 63)) * 4;
}

// Loads a row; elements beyond V (and segments beyond nseg) become `pad`.
template <int V4>
__device__ __forceinline__ void smp_load(float4 (&r)[V4], const float* x, int V, int nseg, float pad) {
#pragma unroll
  for (int i = 0; i < V4; ++i) {
    const int idx = smp_index(i, nseg);
    r[i] = (i < nseg && idx < V) ? *reinterpret_cast<const float4*>(x + idx) : make_float4(pad, pad, pad, pad);   // V % 4 == 0
  }
}

// Sixteen values, one per wavefront, in LDS: every thread gets them all.
struct SmpTot { float v[SMP_NW]; };
__device__ __forceinline__ SmpTot smp_share(float mine, float* smem) {
  if ((threadIdx.x & 63) == 0) smem[threadIdx.x >> 6] = mine;
  __syncthreads();
  SmpTot t;
#pragma unroll
  for (int i = 0; i < SMP_NW / 4; ++i) {
    const float4 f = reinterpret_cast<const float4*>(smem)[i];
    t.v[4 * i] = f.x; t.v[4 * i + 1] = f.y; t.v[4 * i + 2] = f.z; t.v[4 * i + 3] = f.w;
  }
  return t;
}

// Sum of N values pairwise: a value goes through log2 N roundings, where one after another it goes through up to N.
template <int N>
__device__ __forceinline__ float smp_pairwise(float (&s)[N]) {
#pragma unroll
  for (int w = 1; w < N; w *= 2)
#pragma unroll
    for (int i = 0; i + w < N; i += 2 * w) s[i] += s[i + w];
  return s[0];
}

// Lane sum of a wavefront's part of the row.
template <int V4>
__device__ __forceinline__ float smp_lane_sum(const float4 (&r)[V4]) {
  float s[V4];
#pragma unroll
  for (int i = 0; i < V4; ++i) s[i] = (r[i].x + r[i].y) + (r[i].z + r[i].w);
  return smp_pairwise<V4>(s);
}

// r := e^((x - max) / T) elementwise (padding becomes 0); returns the row's maximum, tot gets the wavefronts' sums.
template <int V4>
__device__ __forceinline__ float smp_softmax(float4 (&r)[V4], float inv_t, float* smem_a, float* smem_b, SmpTot& tot) {
  float mx = -INFINITY;
#pragma unroll
  for (int i = 0; i < V4; ++i) mx = fmaxf(mx, fmaxf(fmaxf(r[i].x, r[i].y), fmaxf(r[i].z, r[i].w)));
  const SmpTot ms = smp_share(wave_max(mx), smem_a);
  float m = ms.v[0];
#pragma unroll
  for (int i = 1; i < SMP_NW; ++i) m = fmaxf(m, ms.v[i]);
#pragma unroll
  for (int i = 0; i < V4; ++i) {
    r[i].x = expf((r[i].x - m) * inv_t); r[i].y = expf((r[i].y - m) * inv_t);
    r[i].z = expf((r[i].z - m) * inv_t); r[i].w = expf((r[i].w - m) * inv_t);
  }
  tot = smp_share(wave_sum(smp_lane_sum<V4>(r)), smem_b);
  return m;
}
__device__ __forceinline__ float smp_total(const SmpTot& t) {
  float s[SMP_NW];
#pragma unroll
  for (int i = 0; i < SMP_NW; ++i) s[i] = t.v[i];
  return smp_pairwise<SMP_NW>(s);
}

// Inverse CDF at u * total over weights r with the wavefronts' sums tot: the smallest index whose cumulative sum exceeds
// the target (the last index with a positive weight if rounding leaves the target at the very end; 0 if there is no
// positive weight).  Returns true in the one thread that holds the drawn element.
template <int V4>
__device__ __forceinline__ bool smp_draw(const float4 (&r)[V4], const SmpTot& tot, float u, int nseg, int& token) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const float target = u * smp_total(tot);
  int win = -1;
  float base = 0.f, run = 0.f;
#pragma unroll
  for (int i = 0; i < SMP_NW; ++i) {
    if (tot.v[i] > 0.f && run <= target) { win = i; base = run; }
    run += tot.v[i];
  }
  token = 0;
  if (win < 0) return threadIdx.x == 0;
  if (wv != win) return false;
  // this wavefront's segments, then the lanes of the one that holds the target
  float own = 0.f, seg_base = base;
  int seg = 0;
  run = base;
  float4 g = r[0];
#pragma unroll
  for (int i = 0; i < V4; ++i) {
    const float mine = (r[i].x + r[i].y) + (r[i].z + r[i].w);
    const float st = wave_sum(mine);
    if (st > 0.f && run <= target) { seg = i; seg_base = run; own = mine; g = r[i]; }
    run += st;
  }
  float inc = own;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const float o = __shfl_up(inc, d);
    if (lane >= d) inc += o;
  }
  float c = seg_base + (inc - own);
  const unsigned long long at = __ballot(own > 0.f && c <= target);
  const int pick_lane = at != 0ull ? 63 - __builtin_clzll(at) : 0;
  if (lane != pick_lane) return false;
  const float w4[4] = {g.x, g.y, g.z, g.w};
  int pick = -1, last_pos = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (w4[e] > 0.f) last_pos = e;
    c += w4[e];
    if (pick < 0 && c > target) pick = e;
  }
  token = ((win * nseg + seg) * 64 + lane) * 4 + (pick >= 0 ? pick : last_pos);
  return true;
}

// Draw one token per row from softmax(logits / T); optionally store the probability row.
template <int V4>
__global__ __launch_bounds__(SMP_NT) void k_sample_rows(SampleArgs a) {
  const uint32_t halted = gate_request(a.gate);
  __shared__ __align__(16) float smem[2][SMP_NW];
  const int row = blockIdx.x, V = a.vocab, nseg = smp_segments(V);
  float4 r[V4];
  smp_load<V4>(r, a.logits + (size_t)row * a.ld, V, nseg, -INFINITY);
  const float u = a.u[row];
  if (flag_set(halted)) return;                       // uniform over the launch; nothing has been written yet
  SmpTot tot;
  smp_softmax<V4>(r, a.inv_t, smem[0], smem[1], tot);
  int tok;
  if (smp_draw<V4>(r, tot, u, nseg, tok)) {
    a.tokens[row] = tok;
    if (row == 0 && a.token_next) *a.token_next = tok;
    if (row == 0 && a.block_slot) *a.block_slot = tok;
  }
  if (a.probs) {
    float* p = a.probs + (size_t)row * V;
    const float inv_s = 1.0f / smp_total(tot);
#pragma unroll
    for (int i = 0; i < V4; ++i) {
      const int idx = smp_index(i, nseg);
      if (i < nseg && idx < V) *reinterpret_cast<float4*>(p + idx) = make_float4(r[i].x * inv_s, r[i].y * inv_s, r[i].z * inv_s, r[i].w * inv_s);
    }
  }
}

hipError_t launch_sample_rows(const SampleArgs& a, int n_rows, hipStream_t s) {
  if (n_rows < 1 || a.vocab < 4 || (a.vocab & 3) || a.vocab > 65536 || (a.ld & 3)) return hipErrorInvalidValue;
  if (a.vocab <= 8192) hipLaunchKernelGGL(k_sample_rows<2>, dim3(n_rows), dim3(SMP_NT), 0, s, a);
  else if (a.vocab <= 32768) hipLaunchKernelGGL(k_sample_rows<8>, dim3(n_rows), dim3(SMP_NT), 0, s, a);
  else if (a.vocab <= 49152) hipLaunchKernelGGL(k_sample_rows<12>, dim3(n_rows), dim3(SMP_NT), 0, s, a);
  else hipLaunchKernelGGL(k_sample_rows<16>, dim3(n_rows), dim3(SMP_NT), 0, s, a);
  return hipGetLastError();
}

// Speculative sampling over one block: keep d_j while u_j q_j(d_j) < p_{j-1}(d_j); the last token is
// drawn from norm(max(0, p_n - q_n)) at the first rejection, from p_SL when everything is kept.
//
// Row j's keep test and the draw that would follow its rejection need no other row, so every row has a workgroup of its
// own: it leaves KEPT or the drawn token in out->emit[j], and a second launch of one wavefront finds the first row that
// was not kept and writes the record.  (One workgroup going through the rows took about 10 us a row: 43 - 61 us for a
// block of five at 32000, 8.1 + 1.4 us now; above 49152 logits 22 registers go to scratch memory.  The library has no memory of its own that calls on several
// streams could share safely, hence the second launch instead of a ticket.)
constexpr int ACCEPT_KEPT = -2;

__device__ __forceinline__ int accept_last_row(const AcceptSampleArgs& a) {
  int nb = a.n_block;
  if (a.dev_n_block) { const int v = *a.dev_n_block; nb = v < 1 ? 1 : (v > a.n_block ? a.n_block : v); }
  return nb - 1;
}

// Keep test and draw of row j: kept (uniform), or the token drawn; true in the one thread that holds the outcome.
template <int V4>
__device__ __forceinline__ bool accept_row(const AcceptSampleArgs& a, const int j, const int sl, float (&smem)[3][SMP_NW], bool& kept, int& token) {
  const int V = a.vocab, nseg = smp_segments(V);
  const float* x = a.target_logits + (size_t)j * V;
  const float* q = a.draft_probs + (size_t)j * V;
  float4 r[V4];
  smp_load<V4>(r, x, V, nseg, -INFINITY);
  const float u_res = a.u_resample[j];
  float xt = 0.f, qt = 0.f, u_acc = 0.f;
  if (j < sl) {
    const int tok = min(max(a.block[j + 1], 0), V - 1);
    xt = x[tok]; qt = q[tok]; u_acc = a.u_accept[j];
  }
  SmpTot tot;
  const float m = smp_softmax<V4>(r, a.inv_t, smem[0], smem[1], tot);
  kept = false;
  if (j < sl) {
    const float inv_s = 1.0f / smp_total(tot);
    const float p = expf((xt - m) * a.inv_t) * inv_s;
    if (u_acc * qt < p) {                         // the same values in every thread
      kept = true;
      token = ACCEPT_KEPT;
      return threadIdx.x == 0;
    }
    // residual max(0, p - q) of this row
#pragma unroll
    for (int i = 0; i < V4; ++i) {
      const int idx = smp_index(i, nseg);
      float4 qq = make_float4(0.f, 0.f, 0.f, 0.f);
      if (i < nseg && idx < V) qq = *reinterpret_cast<const float4*>(q + idx);
      r[i].x = fmaxf(0.f, r[i].x * inv_s - qq.x); r[i].y = fmaxf(0.f, r[i].y * inv_s - qq.y);
      r[i].z = fmaxf(0.f, r[i].z * inv_s - qq.z); r[i].w = fmaxf(0.f, r[i].w * inv_s - qq.w);
    }
    tot = smp_share(wave_sum(smp_lane_sum<V4>(r)), smem[2]);
  }
  return smp_draw<V4>(r, tot, u_res, nseg, token);
}

template <int V4>
__global__ __launch_bounds__(SMP_NT) void k_accept_rows(AcceptSampleArgs a) {
  __shared__ __align__(16) float smem[3][SMP_NW];
  const int j = blockIdx.x, sl = accept_last_row(a);
  if (j > sl) return;                             // whole workgroup
  bool kept;
  int tok;
  if (accept_row<V4>(a, j, sl, smem, kept, tok)) reinterpret_cast<AcceptOut*>(a.out)->emit[j] = tok;
}

// The same for a record that overlaps an input (a block that lies in it, say): one workgroup goes through the rows and writes only
// when everything has been read.
__global__ __launch_bounds__(SMP_NT) void k_accept_in_place(AcceptSampleArgs a) {
  __shared__ __align__(16) float smem[3][SMP_NW];
  const int sl = accept_last_row(a);
  int n = -1, tok;
  bool kept, mine;
  do {                                            // uniform; row sl is never kept
    if (++n > 0) __syncthreads();                 // smem is free again
    mine = accept_row<16>(a, n, sl, smem, kept, tok);
  } while (kept);
  if (!mine) return;
  AcceptOut o;
  o.n = n; o.n_emit = n + 1;
  for (int i = 0; i < 16; ++i) o.emit[i] = (i < n) ? a.block[i + 1] : (i == n ? tok : -1);
  *reinterpret_cast<AcceptOut*>(a.out) = o;
  if (a.host_out) { *reinterpret_cast<AcceptOut*>(a.host_out) = o; __threadfence_system(); }
}

__global__ __launch_bounds__(64) void k_accept_finish(AcceptSampleArgs a) {
  const int sl = accept_last_row(a), i = threadIdx.x;
  AcceptOut* out = reinterpret_cast<AcceptOut*>(a.out);
  const int mine = i <= sl ? out->emit[i] : 0;
  const int drafted = i < sl ? a.block[i + 1] : -1;
  const int n = __builtin_ctzll(__ballot(i >= sl || mine != ACCEPT_KEPT));     // row sl always holds a drawn token
  const int e = i < n ? drafted : (i == n ? mine : -1);
  auto put = [&](AcceptOut* o) {
    if (i == 0) { o->n = n; o->n_emit = n + 1; }
    if (i < 16) o->emit[i] = e;
  };
  put(out);
  if (a.host_out) { put(reinterpret_cast<AcceptOut*>(a.host_out)); __threadfence_system(); }
}

hipError_t launch_accept_sample(const AcceptSampleArgs& a, hipStream_t s) {
  if (a.n_block < 1 || a.n_block > 16 || a.vocab < 4 || (a.vocab & 3) || a.vocab > 65536) return hipErrorInvalidValue;
  // the rows' workgroups leave their outcomes in the record while others still read the inputs: nothing may overlap it
  auto overlaps = [&](const void* p, size_t words) {
    const uintptr_t o = reinterpret_cast<uintptr_t>(a.out), q = reinterpret_cast<uintptr_t>(p);
    return p != nullptr && q < o + sizeof(AcceptOut) && o < q + words * 4;
  };
  const size_t n = a.n_block, V = a.vocab;
  if (overlaps(a.block, n) || overlaps(a.dev_n_block, 1) || overlaps(a.u_accept, n - 1) || overlaps(a.u_resample, n) ||
      overlaps(a.draft_probs, (n - 1) * V) || overlaps(a.target_logits, n * V)) {
    hipLaunchKernelGGL(k_accept_in_place, dim3(1), dim3(SMP_NT), 0, s, a);
    return hipGetLastError();
  }
  const dim3 rows(a.n_block);
  if (a.vocab <= 8192) hipLaunchKernelGGL(k_accept_rows<2>, rows, dim3(SMP_NT), 0, s, a);
  else if (a.vocab <= 32768) hipLaunchKernelGGL(k_accept_rows<8>, rows, dim3(SMP_NT), 0, s, a);
  else if (a.vocab <= 49152) hipLaunchKernelGGL(k_accept_rows<12>, rows, dim3(SMP_NT), 0, s, a);
  else hipLaunchKernelGGL(k_accept_rows<16>, rows, dim3(SMP_NT), 0, s, a);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_accept_finish, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// classifier training and evaluation (the step after the loop: features and labels in, parameters out)
// ---------------------------------------------------------------------------------------------
//
// One workgroup.  A unit of work is a tile of 16 examples, and both products of a gradient step are contractions over at most 16
// (the 12 features, a constant 1 for b1, three zeros; 16 examples), so they run on the matrix instruction.  The fp32 form of it
// would be most of a step (two products of 200 examples and 64 units: 1.7 us), so operands go in as sums of three bf16 (24 bits:
// x = x0 + x1 + x2), and the products that matter at fp32 are taken: forward f0 w0 + f0 w1 + f1 w0 + f1 w1 + f0 w2 + f2 w0 (what is left
// out is below 2^-25 of a term) as three instructions of K = 32, and backward mask . (e F) in three parts, where the mask is exact: two
// instructions of K = 32, the second half empty.
// Forward, D[example][unit]: lane l holds unit l % 16 and the examples 4 (l / 16) + v, so the pre-sigmoid output is a weighted sum over
// the lanes of a row.  A wavefront takes TP tiles at a time, and the sums of its 4 TP values are merged on the way (every exchange step halves the
// number of registers), which leaves every lane of a row with the finished output of an example of its own (TP = 4; with TP = 1 four lanes share one): the
// sigmoid and the loss are computed once per example.  The errors come back as in-row broadcasts, and the masked activations are already the B
// operand of the backward product G[feature][unit] = (e F)^T . mask, whose k index runs over l / 16.  The gradient of w2 needs no sum over
// the examples: sum_n e_n relu(w . f_n) = w . G.  Tiles are dealt round-robin; the wavefronts' G are added up in wavefront order through LDS
// and every parameter is updated by the thread that owns it: results do not depend on timing.  Everything else is fp32 but the feature
// statistics (double).
// What bounds it: the instructions of one compute unit and, between them, two barriers with their LDS round trips.  200 examples with 64
// units take 2.0 us a step (5000 cycles: products and masks 1800 for the two wavefronts of a SIMD, sums and sigmoid 800, backward 900,
// update 1100), 4.4 on the fp32 matrix instruction; 1000 examples 7.6 (14.7), 200 examples with 128 units 3.5 (10.3).  More workgroups
// would put a hand-off between workgroups (about 2.5 us) into every step.  Features that are not numbers make all parameters and the loss NaN.
// Error against 64 bits over 1000 runs of 60 .. 2000 examples and 16 .. 128 units (relative 2-norms; in brackets the fp32 matrix
// instruction on the same runs): loss 7.0e-8 (9.0e-8) in the geometric mean, scores 1.04e-7 (1.11e-7).  Where rounding moves an activation
// over the kink of the ReLU the path jumps: scores are more than 1e-5 off in 15 (19) runs, 2.1e-4 at most in either; 9 runs are more
// than three times further off than on the fp32 instruction, 27 more than three times nearer.

constexpr int TRAIN_MAX_N = 2560;               // examples that fit in LDS (12 floats each)

// Workgroup barrier that orders LDS accesses only: __syncthreads also waits for the wavefront's stores to memory (the
// loss of the step), a round trip of half a microsecond.
__device__ __forceinline__ void lds_barrier() {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Two floats as sums of three bf16 each; a part holds the first float's in its low half.
struct Bf16x3 { uint32_t p[3]; };
__device__ __forceinline__ Bf16x3 split3(float a, float b) {
  Bf16x3 s;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    s.p[i] = pack_bf16(a, b);
    a -= __uint_as_float(s.p[i] << 16); b -= __uint_as_float(s.p[i] & 0xffff0000u);
  }
  return s;
}
// max(x, 0), one instruction (fmaxf is two).  Not in assembly: what reads a matrix instruction's result must be visible to the compiler,
// which puts the wait states in between.
__device__ __forceinline__ float relu(float x) { return __int_as_float(max(__float_as_int(x), 0)); }
// 1.0 (bf16) where an activation is positive, 0 where it is not: its bits as bf16 (none set only at 0 or below 2^-134) cut to one, times
// 1.0's.  (The minimum in assembly: the compiler makes a comparison and a select of every half of the pair; the product is
// left to it, since it has to know what a matrix instruction reads.)
__device__ __forceinline__ uint32_t relu_mask(float a, float b) {
  typedef __attribute__((ext_vector_type(2))) unsigned short u16x2;
  uint32_t m = pack_bf16(a, b);
  asm("v_pk_min_u16 %0, %0, %1" : "+v"(m) : "v"(0x00010001u));
  return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, m) * (u16x2){0x3F80, 0x3F80}));
}
// own ? b : a of this lane plus the other of the two from the lane that CTRL names
template <int CTRL>
__device__ __forceinline__ float merge_halves(float a, float b, bool own) {
  const float mine = own ? b : a, other = own ? a : b;
  return mine + dpp_f<CTRL, 0xF>(0.f, other);
}

// HT: 16-unit tiles of the hidden layer; NW wavefronts; TP: example tiles per wavefront and round; PW: unit tiles per reduction
// pass; NMAX: examples that the LDS array holds.  One round (NMAX = 16 NW TP): the examples' operands stay in registers.
template <int HT, int NW, int TP, int PW, int NMAX>
__global__ __launch_bounds__(NW * 64) void k_clf_train(TrainArgs a) {
  constexpr int NP = HT / PW, ROUND = NW * TP;
  constexpr bool ONE = NMAX == ROUND * 16, YS = NMAX <= TRAIN_MAX_N / 2;      // YS: room for the labels too
  static_assert(HT % PW == 0 && PW <= NW && (TP == 1 || TP == 2 || TP == 4), "one owner thread per parameter and pass");
  __shared__ __align__(16) float fs[NMAX * 12];   // standardised examples
  __shared__ u32x4 wS[3][HT][2][16];              // [W1 | b1] in three parts: [unit tile][eight columns][unit]: reads without conflicts
  __shared__ float w2s[HT * 16];
  __shared__ f32x4 red[NW][PW][64];
  __shared__ float2 red3[NW][64];
  __shared__ float ys[YS ? NMAX : 1];
  __shared__ float mu_s[16], isd_s[16], b2_s;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6), col = lane & 15, g = lane >> 4;
  const int N = a.n, H = a.hidden, tiles = (N + 15) >> 4;
  for (int f = w; f < 12; f += NW) {              // mean and deviation of a feature, in a fixed order
    double sum = 0.0;
    for (int n = lane; n < N; n += 64) sum += (double)a.feats[(size_t)n * 12 + f];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d);
    const double mu = sum / N;
    double var = 0.0;
    for (int n = lane; n < N; n += 64) { const double x = (double)a.feats[(size_t)n * 12 + f] - mu; var += x * x; }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) var += __shfl_xor(var, d);
    double sd = sqrt(var / N);
    if (sd < 1e-6) sd = 1e-6;
    if (lane == 0) { mu_s[f] = (float)mu; isd_s[f] = (float)(1.0 / sd); }
  }
  __syncthreads();
  for (int i = t; i < tiles * 16 * 12; i += NW * 64) fs[i] = i < N * 12 ? (a.feats[i] - mu_s[i % 12]) * isd_s[i % 12] : 0.f;
  if (YS) for (int i = t; i < tiles * 16; i += NW * 64) ys[i] = i < N ? (float)a.labels[i] : 0.f;
  // thread (w, lane) owns, of unit tile p PW + w, unit `col` and columns 4 g .. 4 g + 3 (12 weights, then b1), and a copy of its w2
  float own[NP][4], own2[NP];
  auto unit = [&](int p) { return (p * PW + w) * 16 + col; };
  auto put_w = [&](int p) {
    const Bf16x3 s0 = split3(own[p][0], own[p][1]), s1 = split3(own[p][2], own[p][3]);
#pragma unroll
    for (int i = 0; i < 3; ++i) reinterpret_cast<uint2*>(&wS[i][p * PW + w][g >> 1][col])[g & 1] = make_uint2(s0.p[i], s1.p[i]);
    if (g == 0) w2s[unit(p)] = own2[p];
  };
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if (w < PW) {
      const int h = unit(p);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int i = 4 * g + v;
        own[p][v] = h < H && i < 12 ? a.params[h * 12 + i] : (h < H && i == 12 ? a.params[H * 12 + h] : 0.f);
      }
      own2[p] = h < H ? a.params[H * 13 + h] : 0.f;
      put_w(p);
    }
  }
  float b2 = a.params[H * 14];
  if (t == 0) b2_s = b2;
  __syncthreads();
  const float inv_n = 1.0f / (float)N;
  // operands of the examples of tile q of a round that begins at tile `base`
  struct Fwd { u32x4 p0, p1, p02; };              // A operands: f0 | f0, f1 | f1, f0 | f2 (16 columns each)
  struct Bwd { float x[4]; };                     // column `col` of examples 4 g + v
  auto tile_of = [&](int base, int q) { return base + w + NW * q; };
  auto fwd_operand = [&](int tile, Fwd& f) {
    const float* row = fs + (min(tile, tiles - 1) * 16 + col) * 12 + ((g & 1) ? 8 : 0);
    const float4 x = *reinterpret_cast<const float4*>(row), y4 = *reinterpret_cast<const float4*>(row + ((g & 1) ? 0 : 4));
    const float4 y = (g & 1) ? make_float4(1.f, 0.f, 0.f, 0.f) : y4;
    const Bf16x3 s[4] = {split3(x.x, x.y), split3(x.z, x.w), split3(y.x, y.y), split3(y.z, y.w)};
#pragma unroll
    for (int i = 0; i < 4; ++i) { f.p0[i] = s[i].p[0]; f.p1[i] = s[i].p[1]; f.p02[i] = g < 2 ? s[i].p[0] : s[i].p[2]; }
  };
  auto bwd_operand = [&](int tile, Bwd& f) {
    const int n0 = min(tile, tiles - 1) * 16 + 4 * g;
    float x[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) x[v] = fs[(n0 + v) * 12 + min(col, 11)];
    asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));            // (loads for every lane: no branch around them)
#pragma unroll
    for (int v = 0; v < 4; ++v) f.x[v] = col < 12 ? x[v] : (col == 12 ? 1.f : 0.f);
  };
  const int q_mine = col & (TP - 1), v_mine = col >> 2;           // this lane's example of a round: tile q_mine, row 4 g + v_mine
  const bool counts = TP == 4 || (TP == 2 ? (col & 2) == 0 : (col & 3) == 0);   // one lane per example
  Fwd fk[ONE ? TP : 1];
  Bwd bk[ONE ? TP : 1];
  if constexpr (ONE) {
#pragma unroll
    for (int q = 0; q < TP; ++q) { fwd_operand(tile_of(0, q), fk[q]); bwd_operand(tile_of(0, q), bk[q]); }
  }
  for (int ep = 0; ep < a.epochs; ++ep) {
    f32x4 G[HT];
    float gb2 = 0.f, loss = 0.f;
#pragma unroll
    for (int r = 0; r < HT; ++r) G[r] = f32x4{0.f, 0.f, 0.f, 0.f};
    const float bias2 = b2_s;
    for (int base = 0; base + w < tiles; base += ROUND) {
      const int mine = (base + w + NW * q_mine) * 16 + 4 * g + v_mine;
      const bool live = mine < N;
      const float y = YS ? ys[live ? mine : 0] : (float)a.labels[live ? mine : 0];
      u32x4 m01[HT], m23[HT];                     // masks of rows 0, 1 and 2, 3 (component q)
      float z[TP][4];
#pragma unroll
      for (int q = 0; q < TP; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) z[q][v] = 0.f;
      Fwd ft[TP];
#pragma unroll
      for (int q = 0; q < TP; ++q) {
        if constexpr (ONE) ft[q] = fk[q];
        else fwd_operand(tile_of(base, q), ft[q]);
      }
      // the products of several unit tiles go out before the first result is read: an instruction's result takes longer than its issue
      constexpr int RB = HT < 8 / TP ? HT : 8 / TP;
#pragma unroll
      for (int r0 = 0; r0 < HT; r0 += RB) {
        f32x4 p[RB][TP];
        float w2[RB];
#pragma unroll
        for (int rr = 0; rr < RB; ++rr) {
          const int r = r0 + rr;
          const u32x4 w01 = wS[g >> 1][r][g & 1][col], w20 = wS[g < 2 ? 2 : 0][r][g & 1][col];
          w2[rr] = w2s[r * 16 + col];
#pragma unroll
          for (int q = 0; q < TP; ++q) {
            p[rr][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ft[q].p02), as_bf16x8(w20), f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
            p[rr][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ft[q].p1), as_bf16x8(w01), p[rr][q], 0, 0, 0);
            p[rr][q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(ft[q].p0), as_bf16x8(w01), p[rr][q], 0, 0, 0);
          }
        }
        __builtin_amdgcn_sched_group_barrier(0x008, 3 * RB * TP, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 15 * RB * TP, 0);
#pragma unroll
        for (int rr = 0; rr < RB; ++rr)
#pragma unroll
          for (int q = 0; q < TP; ++q) {
            f32x4& x = p[rr][q];
#pragma unroll
            for (int v = 0; v < 4; ++v) { x[v] = relu(x[v]); z[q][v] += w2[rr] * x[v]; }
            m01[r0 + rr][q] = relu_mask(x[0], x[1]); m23[r0 + rr][q] = relu_mask(x[2], x[3]);
          }
      }
      float s[TP];
#pragma unroll
      for (int q = 0; q < TP; ++q) {
        const float r02 = merge_halves<DPP_ROW_ROR8>(z[q][0], z[q][2], (col & 8) != 0), r13 = merge_halves<DPP_ROW_ROR8>(z[q][1], z[q][3], (col & 8) != 0);
        s[q] = merge_halves<DPP_ROW_HALF_MIRROR>(r02, r13, (col & 4) != 0);       // lanes of bank v: row 4 g + v
      }
      float zz;
      if constexpr (TP == 4) {
        const float s02 = merge_halves<DPP_QUAD_XOR2>(s[0], s[2], (col & 2) != 0), s13 = merge_halves<DPP_QUAD_XOR2>(s[1], s[3], (col & 2) != 0);
        zz = merge_halves<DPP_QUAD_XOR1>(s02, s13, (col & 1) != 0);
      } else {
        if constexpr (TP == 2) zz = merge_halves<DPP_QUAD_XOR1>(s[0], s[1], (col & 1) != 0);
        else zz = s[0] + dpp_f<DPP_QUAD_XOR1, 0xF>(0.f, s[0]);
        zz += dpp_f<DPP_QUAD_XOR2, 0xF>(0.f, zz);
      }
      zz += bias2;
      // sigmoid(z) and log(1 + e^-|z|) from one exponential; the logarithm's argument rounds to u, which is put right by
      // the factor E / (u - 1) (the library's log1pf was a third of the step's instructions)
      const float E = expf(-fabsf(zz)), u = 1.0f + E, ru = 1.0f / u, du = u - 1.0f;
      float dz = ((zz >= 0.f ? ru : E * ru) - y) * inv_n;
      dz = live ? dz : 0.f;
      const float e4[4][4] = {{dpp_f<0x150, 0xF>(0.f, dz), dpp_f<0x154, 0xF>(0.f, dz), dpp_f<0x158, 0xF>(0.f, dz), dpp_f<0x15C, 0xF>(0.f, dz)},
                              {dpp_f<0x151, 0xF>(0.f, dz), dpp_f<0x155, 0xF>(0.f, dz), dpp_f<0x159, 0xF>(0.f, dz), dpp_f<0x15D, 0xF>(0.f, dz)},
                              {dpp_f<0x152, 0xF>(0.f, dz), dpp_f<0x156, 0xF>(0.f, dz), dpp_f<0x15A, 0xF>(0.f, dz), dpp_f<0x15E, 0xF>(0.f, dz)},
                              {dpp_f<0x153, 0xF>(0.f, dz), dpp_f<0x157, 0xF>(0.f, dz), dpp_f<0x15B, 0xF>(0.f, dz), dpp_f<0x15F, 0xF>(0.f, dz)}};
#pragma unroll
      for (int q = 0; q < TP; ++q) {
        Bwd bt;
        if constexpr (ONE) bt = bk[q];
        else bwd_operand(tile_of(base, q), bt);
        const Bf16x3 s0 = split3(e4[q][0] * bt.x[0], e4[q][1] * bt.x[1]), s1 = split3(e4[q][2] * bt.x[2], e4[q][3] * bt.x[3]);
        const u32x4 x01 = {s0.p[0], s1.p[0], s0.p[1], s1.p[1]};
        const u32x4 x2 = {s0.p[2], s1.p[2], 0u, 0u};
        // the third part takes the instruction of the other two, half of it empty.  (That is a choice, not a rule of the chip: 16x16x16 and
        // 16x16x32 products back to back on one accumulator, either first, are exact in 51200 elements checked.  A variant that mixed them here
        // gave wrong sums; it also read matrix results in inline assembly, which gets no wait states, see relu.)
#pragma unroll
        for (int r = 0; r < HT; ++r) {
          const u32x4 mk = {m01[r][q], m23[r][q], m01[r][q], m23[r][q]};
          G[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x2), as_bf16x8(mk), G[r], 0, 0, 0);
          G[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x01), as_bf16x8(mk), G[r], 0, 0, 0);
        }
      }
      // (behind the products, whose results are not read yet)
      const float term = fmaxf(zz, 0.f) - zz * y + (du == 0.f ? E : logf(u) * (E / du));
      gb2 += counts ? dz : 0.f;
      loss += live && counts ? term : 0.f;
    }
    red3[w][lane] = make_float2(gb2, loss);
#pragma unroll
    for (int p = 0; p < NP; ++p) {
      if (p > 0) lds_barrier();                   // the pass before has been read
#pragma unroll
      for (int q = 0; q < PW; ++q) red[w][q][lane] = G[p * PW + q];
      lds_barrier();
      if (w < PW) {
        f32x4 s = red[0][w][lane];
#pragma unroll
        for (int ww = 1; ww < NW; ++ww) s += red[ww][w][lane];
        const float lw2 = a.lr * own2[p];
        const float gw2 = row4_sum((own[p][0] * s[0] + own[p][1] * s[1]) + (own[p][2] * s[2] + own[p][3] * s[3]));
#pragma unroll
        for (int v = 0; v < 4; ++v) own[p][v] -= lw2 * s[v];
        own2[p] -= a.lr * gw2;
        put_w(p);
      }
      if (p == NP - 1 && w == NW - 1) {           // the last wavefront: with fewer unit tiles than wavefronts it owns no weights
        float sb = 0.f, sl = 0.f;
#pragma unroll
        for (int ww = 0; ww < NW; ++ww) { const float2 x = red3[ww][lane]; sb += x.x; sl += x.y; }
        sb = wave_sum(sb); sl = wave_sum(sl);
        b2 -= a.lr * sb;
        if (lane == 0) {
          b2_s = b2;
          if (a.loss) a.loss[ep] = sl * inv_n;
        }
      }
    }
    lds_barrier();
  }
  // fold the standardisation into W1 and b1: the classifier consumes raw features
#pragma unroll
  for (int p = 0; p < NP; ++p) {
    if (w < PW) {
      const int h = unit(p);
      float shift = 0.f;
      if (g < 3) {
#pragma unroll
        for (int v = 0; v < 4; ++v) shift += own[p][v] * isd_s[4 * g + v] * mu_s[4 * g + v];
      }
      shift = row4_sum(shift);
      if (h < H) {
        if (g < 3) {
#pragma unroll
          for (int v = 0; v < 4; ++v) a.params[h * 12 + 4 * g + v] = own[p][v] * isd_s[4 * g + v];
        } else {
          a.params[H * 12 + h] = own[p][0] - shift;
          a.params[H * 13 + h] = own2[p];
        }
      }
    }
  }
  if (t == NW * 64 - 1) a.params[H * 14] = b2;
}

// Shapes by the number of examples, ms for 400 steps.  Up to 64, up to 32 units or above 128: four wavefronts, a tile each (64 examples: 16 units 0.302,
// 0.322 in the next shape; 32 0.362 / 0.366; 200 1.44 / 1.97; but 64 units 0.534 / 0.480 and 128 0.816 / 0.778).  Up to 128: eight wavefronts, a tile each
// (100 examples: 16 units 0.397, 0.497 in the next shape; 64 0.594 / 0.811; 128 0.938 / 1.374).  Up to 256: eight with two tiles each (of 16
// wavefronts with one tile the update waits longer than the shared sigmoids save: 2.07 us a step against 2.32 at 200 examples and 64 units; four
// wavefronts with four tiles 2.33).  Beyond that rounds of 32 tiles (16 with more than 64 units, whose masks take the registers), over
// examples that are split anew in every step.  More than 128 units: four wavefronts, 512 registers each.
template <int HT>
static void launch_clf_train_ht(const TrainArgs& a, hipStream_t s) {
  constexpr int NW = HT > 8 ? 4 : 8, TP = HT > 4 ? 2 : 4, PW = HT > NW ? NW : HT, PWL = HT > 8 ? 1 : (HT > 2 ? 2 : HT), P4 = HT > 4 ? 4 : HT;
  if constexpr (HT <= 2 || HT > 8) {
    if (a.n <= 64) { hipLaunchKernelGGL((k_clf_train<HT, 4, 1, P4, 64>), dim3(1), dim3(256), 0, s, a); return; }
  }
  if constexpr (HT <= 8) {
    if (a.n <= 128) { hipLaunchKernelGGL((k_clf_train<HT, 8, 1, HT, 128>), dim3(1), dim3(512), 0, s, a); return; }
    if (a.n <= 256) { hipLaunchKernelGGL((k_clf_train<HT, 8, 2, HT, 256>), dim3(1), dim3(512), 0, s, a); return; }
  }
  if (a.n <= TRAIN_MAX_N / 2) hipLaunchKernelGGL((k_clf_train<HT, NW, TP, PW, TRAIN_MAX_N / 2>), dim3(1), dim3(NW * 64), 0, s, a);
  else hipLaunchKernelGGL((k_clf_train<HT, NW, TP, PWL, TRAIN_MAX_N>), dim3(1), dim3(NW * 64), 0, s, a);
}

hipError_t launch_clf_train(const TrainArgs& a, hipStream_t s) {
  if (a.n < 1 || a.n > TRAIN_MAX_N || a.hidden < 1 || a.hidden > 256 || a.epochs < 0) return hipErrorInvalidValue;
  if (a.hidden <= 16) launch_clf_train_ht<1>(a, s);
  else if (a.hidden <= 32) launch_clf_train_ht<2>(a, s);
  else if (a.hidden <= 64) launch_clf_train_ht<4>(a, s);
  else if (a.hidden <= 128) launch_clf_train_ht<8>(a, s);
  else launch_clf_train_ht<16>(a, s);
  return hipGetLastError();
}
// Scores of given feature vectors and the confusion counts of "accepted iff C >= tau" against the
// labels: counts[0..3] = true positives, false positives, false negatives, true negatives.
// The parameters go to LDS once per workgroup and four threads share an example's hidden units (a quarter each, added in
// quarter order): a thread that read all the parameters from memory waited for one unit's after another's
// (200 examples, 64 units: 12.8 us, 5.5 us now).
__global__ __launch_bounds__(256) void k_clf_eval(EvalArgs a) {
  __shared__ float ps[256 * 14 + 1];
  __shared__ float part[4][64];
  const int e = threadIdx.x & 63, quarter = threadIdx.x >> 6, H = a.hidden;
  const int n = blockIdx.x * 64 + e;
  for (int i = threadIdx.x; i < H * 14 + 1; i += 256) ps[i] = a.params[i];
  float f[12];
#pragma unroll
  for (int i = 0; i < 12; ++i) f[i] = n < a.n ? a.feats[(size_t)n * 12 + i] : 0.f;
  __syncthreads();
  const int h1 = H * (quarter + 1) / 4;
  float z = 0.f;
  for (int h = H * quarter / 4; h < h1; ++h) {     // fixed order
    float pre = ps[H * 12 + h];
#pragma unroll
    for (int i = 0; i < 12; ++i) pre += ps[h * 12 + i] * f[i];
    z += fmaxf(pre, 0.f) * ps[H * 13 + h];
  }
  part[quarter][e] = z;
  __syncthreads();
  if (quarter != 0 || n >= a.n) return;
  z = (part[0][e] + part[1][e]) + (part[2][e] + part[3][e]);
  const float c = 1.0f / (1.0f + expf(-(z + ps[H * 14])));
  if (a.scores) a.scores[n] = c;
  if (a.counts && a.labels) {
    const int pred = c >= a.tau ? 1 : 0, y = a.labels[n] != 0 ? 1 : 0;
    atomicAdd(a.counts + (pred ? (y ? 0 : 1) : (y ? 2 : 3)), 1);
  }
}

hipError_t launch_clf_eval(const EvalArgs& a, hipStream_t s) {
  if (a.n < 1 || a.hidden < 1 || a.hidden > 256) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_clf_eval, dim3((a.n + 63) / 64), dim3(256), 0, s, a);
  return hipGetLastError();
}

// Training examples of the labelling run (App. D.1): from the classify record of every position, the twelve
// features, the draft's token and the label "the draft's token equals the target's token there".
__global__ __launch_bounds__(256) void k_clf_examples(const ClfOut* __restrict__ rec, int n, const int32_t* __restrict__ ref_tokens,
                                                      float* __restrict__ feats, int32_t* __restrict__ labels, int32_t* __restrict__ tokens) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n) return;
  const ClfOut r = rec[i];
#pragma unroll
  for (int k = 0; k < 12; ++k) feats[(size_t)i * 12 + k] = r.feats[k];
  labels[i] = (r.token == ref_tokens[i]) ? 1 : 0;
  if (tokens != nullptr) tokens[i] = r.token;
}

hipError_t launch_clf_examples(const void* rec, int n, const int32_t* ref_tokens, float* feats, int32_t* labels, int32_t* tokens,
                               hipStream_t s) {
  hipLaunchKernelGGL(k_clf_examples, dim3((n + 255) / 256), dim3(256), 0, s, reinterpret_cast<const ClfOut*>(rec), n, ref_tokens,
                     feats, labels, tokens);
  return hipGetLastError();
}

struct LoopOut { int32_t sl; int32_t block[16]; int32_t halted; };   // mirrors disco_loop_out

__global__ void k_loop_init(uint32_t* gate, int32_t* sl_count, const int32_t* tokens_in, int n_in, LoopOut* out) {
  if (threadIdx.x != 0) return;
  *gate = 0u; sl_count[0] = 0; sl_count[1] = 0;     // second word: the perplexity rule's running sum (0.0f)
  out->sl = 0; out->halted = 0;
  out->block[0] = tokens_in[n_in - 1];
  for (int i = 1; i < 16; ++i) out->block[i] = 0;
}

__global__ void k_loop_finish(const int32_t* sl_count, const uint32_t* gate, LoopOut* out, LoopOut* host_out, const unsigned* abort_word) {
  if (threadIdx.x != 0) return;
  out->sl = (abort_word != nullptr && *abort_word != 0u) ? -1 : *sl_count;
  out->halted = (int32_t)*gate;
  if (host_out) { *host_out = *out; __threadfence_system(); }
}

__global__ __launch_bounds__(256) void k_zero(int* p, int n) {
  for (int i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) p[i] = 0;
}

// Rotary table: (cos, sin) of pos * base^(-2 i / d_head) for every cached position and channel pair
// i; the angle is formed in double precision, the table holds floats.
__global__ __launch_bounds__(256) void k_rope_fill(float* tab, int n_pos, int dh, float base) {
  const int half = dh >> 1;
  const int64_t total = (int64_t)n_pos * half;
  for (int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x; idx < total; idx += (int64_t)gridDim.x * 256) {
    const int pos = (int)(idx / half), i = (int)(idx % half);
    const double inv_freq = exp2(-(2.0 * (double)i / (double)dh) * log2((double)base));
    double sn, cs;
    sincos((double)pos * inv_freq, &sn, &cs);
    tab[idx * 2] = (float)cs;
    tab[idx * 2 + 1] = (float)sn;
  }
}

hipError_t launch_rope_fill(float* tab, int n_pos, int dh, float base, hipStream_t s) {
  const int64_t total = (int64_t)n_pos * (dh / 2);
  int64_t blocks = (total + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(k_rope_fill, dim3((unsigned)blocks), dim3(256), 0, s, tab, n_pos, dh, base);
  return hipGetLastError();
}

hipError_t launch_zero(int* p, int n, hipStream_t s) {
  hipLaunchKernelGGL(k_zero, dim3(n > 4096 ? 16 : 1), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

hipError_t launch_loop_init(uint32_t* gate, int32_t* sl_count, const int32_t* tokens_in, int n_in, void* dev_loop_out,
                            hipStream_t s) {
  hipLaunchKernelGGL(k_loop_init, dim3(1), dim3(64), 0, s, gate, sl_count, tokens_in, n_in,
                     reinterpret_cast<LoopOut*>(dev_loop_out));
  return hipGetLastError();
}

// Host values into device slots: the pending tokens of an iteration (n <= 2) and, for an iteration that
// drafts nothing, the one-token block.
__global__ void k_put_tokens(int32_t* tokens, int t0, int t1, int n, LoopOut* out, LoopOut* host_out) {
  if (threadIdx.x != 0) return;
  if (tokens) { tokens[0] = t0; if (n > 1) tokens[1] = t1; }
  if (out) {
    out->sl = 0; out->halted = 1; out->block[0] = n > 1 ? t1 : t0;
    for (int i = 1; i < 16; ++i) out->block[i] = 0;
    if (host_out) *host_out = *out;
  }
}

hipError_t launch_put_tokens(int32_t* tokens, int t0, int t1, int n, void* dev_loop_out, void* host_loop_out, hipStream_t s) {
  hipLaunchKernelGGL(k_put_tokens, dim3(1), dim3(64), 0, s, tokens, t0, t1, n, reinterpret_cast<LoopOut*>(dev_loop_out),
                     reinterpret_cast<LoopOut*>(host_loop_out));
  return hipGetLastError();
}

hipError_t launch_loop_finish(const int32_t* sl_count, const uint32_t* gate, void* dev_loop_out, void* host_loop_out,
                              const unsigned* abort_word, hipStream_t s) {
  hipLaunchKernelGGL(k_loop_finish, dim3(1), dim3(64), 0, s, sl_count, gate, reinterpret_cast<LoopOut*>(dev_loop_out),
                     reinterpret_cast<LoopOut*>(host_loop_out), abort_word);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// dense prompt pass: the GEMMs of a forward over many groups of 16 tokens at once
// ---------------------------------------------------------------------------------------------
//
// The prompt is processed before the first iteration (Sec. 2: the target model is given a prompt).
// With hundreds of tokens per pass the GEMMs are bound by the matrix unit, not by the weight stream, so the tiling differs from
// the skinny kernel: both operands are shared by the wavefronts of a workgroup through LDS.  Operand layouts, precision (bf16
// hi + lo activations, fp32 accumulation) and epilogue arithmetic are those of the skinny kernel.
//
// A workgroup of 8 wavefronts (WR x WC) owns WR x R2 blocks of 32 rows x WC x C2 blocks of
// 32 panel columns.  With hi + lo panels 64 panel columns are 32 tokens (the lo products are added into the accumulators of
// the hi products), with bf16 activations 64.  What bounds it: the matrix unit, busy in
// 63 - 78 % of the cycles of a launch that fills the chip, at the 1.4 - 1.9 GHz that these launches run at in long passes (counters: W1
// of the multi-query target at 3001 tokens 77 %, 13B gate/up at 2048 in bf16 75 %, QKV 63 %), so
// the loop is built to move little per product: both operands go from memory straight into LDS (no registers), 16 bytes per
// lane in the packed tile order, which is also a conflict-free order of the 128-bit fragment reads, and 32x32x16
// instructions read every fragment once per 128 x 64 wavefront tile.
//
// A stage holds one k-tile (32 columns of K) of the workgroup's row and panel tiles; NST stages form a ring.  Half steps of 16
// columns are software-pipelined through two sets of fragment registers:
//   first half:  matrix instructions of (kt, 0) while the fragments of (kt, 1) are read
//   barrier:     every wavefront has waited for its own copies of stage kt + 1 and for its reads of stage kt
//   second half: matrix instructions of (kt, 1) while the fragments of (kt + 1, 0) are read; the copies of k-tile
//                kt + NST go into the stage that the barrier has just released
//
// Matrices with few tiles (d_model rows at some hundred tokens; every matrix at some tens) are cut along K as well: EPI_SPLIT
// stores a range's sums, k_gemm_sum adds the ranges in order and runs the epilogue.  (Partial sums through write-through
// stores and a ticket in one launch measured slower than no split at all: 110 us against 50 + 16 for 5120 x 5120 at 511 tokens.)

// Sum of four squares.  The roundings are those that the compiler chooses for (x x + y y) + (z z + w w) in an epilogue of one pair of row
// tiles: in its first chunk the first square of a pair is rounded, in the others the second (written out: see split_product).
__device__ __forceinline__ float squares_of_chunk(const bool first, const float4 h) {
#pragma clang fp contract(off)
  const float xx = h.x * h.x, yy = h.y * h.y, zz = h.z * h.z, ww = h.w * h.w;
  return first ? fmaf(h.y, h.y, xx) + fmaf(h.w, h.w, zz) : fmaf(h.x, h.x, yy) + fmaf(h.z, h.z, ww);
}

// What the epilogue of a wavefront with one pair of row tiles reads: requested in front of the products, whose end it would
// otherwise wait behind; k_gemm_sum requests it with the partial sums.  A pass of the 68M shape at 60 tokens 113.9 -> 112.1 us, at 511 142.2 -> 139.0,
// at 600 in bf16 151.5 -> 148.9, of the mid-size grouped-query shape at 100 tokens 401 -> 397.  (The tokens' sums of squares requested there too and
// added up behind the products gained nothing: the first copies take as long.)
template <int EPI, int CA>
struct TileAhead {
  float4 h[EPI == EPI_PARTIAL ? CA : 1][4], gain[4];       // residual values and gains of the four chunks
  float4 rope[EPI == EPI_QKV ? CA : 1][2][2];              // rotary factors of the two 4-row groups
  KvSlot slot[EPI == EPI_QKV ? CA : 1];
  __device__ __forceinline__ void request(const DenseArgs& d, const int g0, const int (&rt)[2]) {
    const GemmArgs& a = d.g;
    const int lane = threadIdx.x & 63, m = lane & 15, gh = lane >> 5;
    if constexpr (EPI == EPI_PARTIAL) {
      if (a.Xout != nullptr)
#pragma unroll
        for (int i = 0; i < 4; ++i) gain[i] = *reinterpret_cast<const float4*>(a.gain + max(rt[i >> 1], 0) * 16 + 8 * (i & 1) + 4 * gh);
    }
    if constexpr (EPI == EPI_PARTIAL || EPI == EPI_QKV) {
#pragma unroll
      for (int c = 0; c < CA; ++c) {
        const int ci = min(g0 + 2 * c + ((lane >> 4) & 1), d.n_groups - 1);
        if constexpr (EPI == EPI_PARTIAL) {
          const float* hrow = a.h + (size_t)ci * d.hs + (size_t)m * a.ld_out;
#pragma unroll
          for (int i = 0; i < 4; ++i) h[c][i] = *reinterpret_cast<const float4*>(hrow + max(rt[i >> 1], 0) * 16 + 8 * (i & 1) + 4 * gh);
        } else {
          const int pos = a.pos0 + 16 * ci + m;
          slot[c] = kv_slot(a, pos);
          if (a.rope_tab != nullptr)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              const int ch = (max(rt[0], 0) * 16 + 4 * (2 * i + gh)) & (a.dh - 1);
              const float4* tab = reinterpret_cast<const float4*>(a.rope_tab + ((size_t)pos * (a.dh >> 1) + ch) * 2);
              rope[c][i][0] = tab[0]; rope[c][i][1] = tab[1];
            }
        }
      }
    }
  }
};

// Epilogue of one wavefront: R2 pairs of row tiles (rt[2 q], rt[2 q + 1]; -1 past the matrix) x CA accumulators of 32 rows x
// 32 tokens.  Lane: token column lane % 32 (two groups of 16), rows 8 i + 4 (lane / 32) .. + 3 of chunk i = 0 .. 3.
// AHEAD: one pair of row tiles, whose inputs `ahead` holds.
template <int EPI, int R2, int CA, bool HI, bool AHEAD = false>
__device__ __forceinline__ void tile_epilogue(const DenseArgs& d, const int g0, const int (&rt)[2 * R2], const f32x16 (&acc)[R2][CA],
                                              const float* rstd_s /* 1 / rms of the tokens from group g0 on, where the launch forms them */,
                                              const TileAhead<EPI, CA>& ahead) {
  static_assert(!AHEAD || R2 == 1, "one pair");
  constexpr bool PAIR = EpiTraits<EPI>::pair;
  const GemmArgs& a = d.g;
  const int lane = threadIdx.x & 63, m = lane & 15, gh = lane >> 5;
#pragma unroll
  for (int c = 0; c < CA; ++c) {
    const int ci = g0 + 2 * c + ((lane >> 4) & 1);
    if (ci >= d.n_groups) continue;               // (half a wavefront at the ragged end)
    const float rstd = EPI == EPI_PARTIAL ? 1.f : (rstd_s != nullptr ? rstd_s[(ci - g0) * 16 + m] : (d.rstd != nullptr ? d.rstd[ci * 16 + m] : 1.f));
    float4 hv[EPI == EPI_PARTIAL ? R2 : 1][4];
    float* hrow = EPI == EPI_PARTIAL ? a.h + (size_t)ci * d.hs + (size_t)m * a.ld_out : nullptr;
    if (EPI == EPI_PARTIAL) {                     // all residual values of the column are requested before the first store
#pragma unroll
      for (int q = 0; q < R2; ++q)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if constexpr (AHEAD) hv[q][i] = ahead.h[c][i];
          else hv[q][i] = *reinterpret_cast<const float4*>(hrow + max(rt[2 * q + (i >> 1)], 0) * 16 + 8 * (i & 1) + 4 * gh);
        }
    }
#pragma unroll
    for (int q = 0; q < R2; ++q) {
      float y[4][4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int v = 0; v < 4; ++v) y[i][v] = acc[q][c][4 * i + v] * rstd;
      if constexpr (PAIR) {
        const int t0 = rt[2 * q];
        if (t0 >= 0) {
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            const int g = 2 * i + gh;             // 4-row group of the 16-row tile
            if constexpr (EPI == EPI_QKV) {
              const int n0 = t0 * 16 + 4 * g, pos = a.pos0 + 16 * ci + m;
              if constexpr (AHEAD) qkv_store<false, true, true>(a, a.q + (size_t)ci * d.qs, n0, m, pos, ahead.slot[c], y[i], y[i + 2], ahead.rope[c][i]);
              else qkv_store(a, a.q + (size_t)ci * d.qs, n0, m, pos, KvSlot{}, y[i], y[i + 2]);
            } else {
              float act[4];
#pragma unroll
              for (int v = 0; v < 4; ++v) act[v] = y[i][v] / (1.0f + expf(-y[i][v])) * y[i + 2][v];
              xpack_store4<false, !HI>(a.Xout + (size_t)ci * d.xouts, a.KT_out, 16, m, (t0 >> 1) * 16 + 4 * g, act);
            }
          }
        }
      } else {
#pragma unroll
        for (int tl = 0; tl < 2; ++tl) {
          const int t0 = rt[2 * q + tl];
          if (t0 < 0) continue;
          float sq = 0.f;
#pragma unroll
          for (int i2 = 0; i2 < 2; ++i2) {
            const int i = 2 * tl + i2, col = t0 * 16 + 8 * i2 + 4 * gh;
            if constexpr (EPI == EPI_PARTIAL) {
              float4 h = hv[q][i];
              h.x += y[i][0]; h.y += y[i][1]; h.z += y[i][2]; h.w += y[i][3];
              *reinterpret_cast<float4*>(hrow + col) = h;
              if (a.Xout != nullptr) {            // deferred RMSNorm of the next GEMM
                const float4 gn = AHEAD ? ahead.gain[i] : *reinterpret_cast<const float4*>(a.gain + col);
                if constexpr (AHEAD) {
                  xpack_put4(a.Xout + (size_t)ci * d.xouts, a.KT_out, 16, m, col, split_product<true>(h.x, gn.x, h.y, gn.y), split_product<true>(h.z, gn.z, h.w, gn.w));
                  sq += squares_of_chunk(i == 0, h);
                } else {
                const float o[4] = {h.x * gn.x, h.y * gn.y, h.z * gn.z, h.w * gn.w};
                xpack_store4(a.Xout + (size_t)ci * d.xouts, a.KT_out, 16, m, col, o);
                sq += (h.x * h.x + h.y * h.y) + (h.z * h.z + h.w * h.w);
                }
              }
            } else {
              float act[4];
#pragma unroll
              for (int v = 0; v < 4; ++v) act[v] = 0.5f * y[i][v] * (1.0f + erff(y[i][v] * 0.70710678118654752f));
              xpack_store4<false, !HI>(a.Xout + (size_t)ci * d.xouts, a.KT_out, 16, m, col, act);
            }
          }
          if constexpr (EPI == EPI_PARTIAL) {
            if (a.Xout != nullptr) {
              sq = half_sum(sq);                  // (lanes l and l + 32 hold the same token: both are here)
              if (gh == 0) a.ssq_out[(size_t)ci * d.ssq_outs + t0 * 16 + m] = sq;      // [slot][token]
            }
          }
        }
      }
    }
  }
}

template <int EPI, int WR, int WC, int R2, int C2, int NST, int OCC, bool HI>
__global__ __launch_bounds__(512, OCC) void k_gemm_tile(const bf16_t* W, const bf16_t* X, size_t xs, int KT_, int n_rows, int n_groups, int grp, int k_split,
                                                        DenseArgs d) {          // (leading arguments: see k_gemm)
  d.g.W = W; d.g.X = X; d.xs = xs; d.g.KT = KT_; d.g.n_rows = n_rows; d.n_groups = n_groups; d.g.grp = grp; d.k_split = k_split;
  constexpr int NW = WR * WC, CA = HI ? C2 : C2 / 2;
  constexpr int NA = 2 * R2 * WR, NBT = 2 * C2 * WC, NT = NA + NBT, PER = NT / NW;
  constexpr int WG_G = HI ? NBT : NBT / 2;        // token groups per workgroup
  static_assert(NW == 8 && NT % NW == 0, "eight wavefronts, equal shares of the copies");
  constexpr bool NORMED = EPI == EPI_QKV || EPI == EPI_SWIGLU;
  __shared__ u32x4 st[NST][NT][64];
  __shared__ float rstd_s[NORMED ? WG_G * 16 : 1];
  const GemmArgs& a = d.g;
  const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = w / WC, wc = w % WC;
  const int n_tiles = a.n_rows >> 4, KT = a.KT;
  const int ncb = (d.n_groups + WG_G - 1) / WG_G, nrb = (n_tiles + NA - 1) / NA;
  // ids go round-robin to the 8 XCDs: XCD x takes a contiguous run of the tiles, which are numbered 8 panel blocks wide, row by row
  const int S = EPI == EPI_SPLIT ? d.k_split : 1, T = nrb * ncb * S, xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int n_x = T / 8 + (xcd < T % 8 ? 1 : 0);
  if (slot >= n_x) return;                        // whole workgroup
  const int unit = xcd * (T / 8) + min(xcd, T % 8) + slot, ti = unit / S, seg = unit - ti * S;
  const int k0 = EPI == EPI_SPLIT ? KT * seg / S : 0, k1 = EPI == EPI_SPLIT ? KT * (seg + 1) / S : KT;
  const int per_pg = nrb * 8, pg = ti / per_pg, in_pg = ti - pg * per_pg;
  const int width = min(8, ncb - pg * 8), rb = in_pg / width, cb = pg * 8 + in_pg - rb * width;
  // row tile of slot s (0 .. NA - 1), -1 past the matrix: pairs (t, t + grp), grp a power of two (1: the tiles in order)
  const int gs = __builtin_ctz(a.grp);
  auto row_tile = [&](const int s) {
    const int bp = (rb * NA + s) >> 1;
    const int t = ((bp >> gs) << (gs + 1)) + (bp & (a.grp - 1)) + ((s & 1) ? a.grp : 0);
    return bp < (n_tiles >> 1) ? t : -1;
  };
  const char* src[PER];
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int s = w + NW * i;
    if (s < NA) {
      src[i] = reinterpret_cast<const char*>(a.W) + (size_t)max(row_tile(s), 0) * KT * 1024;
    } else {
      // panel slots of a wavefront column: hi tiles of its groups, then their lo tiles, or (HI) one tile per group
      const int b = s - NA, wb = b % (2 * C2), gl = HI ? b : b / (2 * C2) * C2 + wb % C2;
      src[i] = reinterpret_cast<const char*>(a.X + (size_t)min(cb * WG_G + gl, d.n_groups - 1) * d.xs) + ((!HI && wb >= C2) ? (size_t)KT * 1024 : 0);
    }
  }
  const uint32_t lds0 = lds_address(&st[0][0][0]);
  auto dma = [&](const int i, const int kt, const int stg) {
    const uint32_t off = (uint32_t)(kt < k1 ? kt : k1 - 1) * 1024u + (uint32_t)lane * 16u;
    lds_dma_16(src[i], off, lds0 + (uint32_t)stg * (NT * 1024u) + (uint32_t)(w + NW * i) * 1024u);
  };
  const int tsel = (lane >> 4) & 1, pos = (lane >> 5) * 16 + (lane & 15);
  auto rd = [&](const int sg, const int t0, const int s) { return st[sg][t0 + tsel][pos + 32 * s]; };
  f32x16 acc[R2][CA];
#pragma unroll
  for (int r = 0; r < R2; ++r)
#pragma unroll
    for (int c = 0; c < CA; ++c)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[r][c][v] = 0.f;
  // (the first stages' copies need only leading arguments and go out while the others arrive.  What is requested between the copies only
  // makes the waits below longer, which count the copies: everything is counted in order)
  constexpr int FIRST = 3;
#pragma unroll
  for (int k = 0; k < FIRST; ++k)
#pragma unroll
    for (int i = 0; i < PER; ++i) dma(i, k0 + k, k);
  // (not the residual update's with bf16 activations, whose tile has twice the tokens: multi-query draft at 63 tokens 685 us a pass against 680)
  constexpr bool AHEAD = EPI != EPI_SPLIT && R2 == 1 && !(EPI == EPI_PARTIAL && HI);
  int rt[2 * R2];
#pragma unroll
  for (int r = 0; r < 2 * R2; ++r) rt[r] = row_tile(wr * 2 * R2 + r);
  TileAhead<EPI, CA> ahead;
  if constexpr (AHEAD) ahead.request(d, cb * WG_G + wc * 2 * CA, rt);
#pragma unroll
  for (int k = FIRST; k < NST; ++k)
#pragma unroll
    for (int i = 0; i < PER; ++i) dma(i, k0 + k, k);
  const bool own_rstd = NORMED && a.ssq != nullptr;
  if (own_rstd) {
    // narrow models (64 sums of squares a row at most): every workgroup adds up its own tokens' while the first copies arrive, in
    // the order of k_rstd_groups
    for (int t = threadIdx.x; t < WG_G * 16; t += 512) {
      const float* sq = a.ssq + (size_t)min(cb * WG_G + (t >> 4), d.n_groups - 1) * a.n_ssq * 16 + (t & 15);
      float tot = 0.f;
#pragma unroll 16
      for (int i = 0; i < a.n_ssq; ++i) tot += sq[i * 16];
      rstd_s[t] = 1.0f / sqrtf(tot / (float)a.d_in + a.eps);
    }
  }
  struct Frag { u32x4 a[R2], b[C2]; };
  Frag f0, f1;
  asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" :: "n"((NST - 1) * PER) : "memory");
#pragma unroll
  for (int c = 0; c < C2; ++c) f0.b[c] = rd(0, NA + (wc * C2 + c) * 2, 0);
#pragma unroll
  for (int r = 0; r < R2; ++r) f0.a[r] = rd(0, (wr * R2 + r) * 2, 0);
  auto half = [&](const Frag& cur, Frag& nxt, const int sg, const int s, const int kt, const int sd, const bool copy) {
#pragma unroll
    for (int q = 0; q < R2; ++q) {
#pragma unroll
      for (int c = q * C2 / R2; c < (q + 1) * C2 / R2; ++c) nxt.b[c] = rd(sg, NA + (wc * C2 + c) * 2, s);
      nxt.a[q] = rd(sg, (wr * R2 + q) * 2, s);
      if (copy)
#pragma unroll
        for (int i = q * PER / R2; i < (q + 1) * PER / R2; ++i) dma(i, kt, sd);
#pragma unroll
      for (int c = 0; c < C2; ++c)
        acc[q][c % CA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(cur.a[q]), as_bf16x8(cur.b[c]), acc[q][c % CA], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);          // keep the reads and copies spread between the matrix instructions
    }
  };
  int sc = 0;                                     // stage of k-tile kt
  for (int kt = k0; kt < k1; ++kt) {
    const int sn = sc == NST - 1 ? 0 : sc + 1;
    half(f0, f1, sc, 1, 0, 0, false);
    // of the copies in flight (k-tiles kt + 1 .. kt + NST - 1) those of kt + 1 must have arrived
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((NST - 2) * PER) : "memory");
    half(f1, f0, sn, 0, kt + NST, sc, true);
    sc = sn;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");   // nothing is in flight into LDS when the workgroup gives it back
  if constexpr (EPI == EPI_SPLIT) {
    // this range's sums, in the lanes' own order: [unit][q][c][chunk][wavefront][lane][4]
    float* plane = a.planes + (size_t)unit * (R2 * CA * 16 * NW * 64) + ((size_t)w * 64 + lane) * 4;
#pragma unroll
    for (int q = 0; q < R2; ++q)
#pragma unroll
      for (int c = 0; c < CA; ++c)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<float4*>(plane + (size_t)((q * CA + c) * 4 + i) * (NW * 256)) =
              make_float4(acc[q][c][4 * i], acc[q][c][4 * i + 1], acc[q][c][4 * i + 2], acc[q][c][4 * i + 3]);
  } else {
    if (own_rstd) __syncthreads();
    tile_epilogue<EPI, R2, CA, HI, AHEAD>(d, cb * WG_G + wc * 2 * CA, rt, acc, own_rstd ? rstd_s + wc * 2 * CA * 16 : nullptr, ahead);
  }
}

// Sum of the K ranges that k_gemm_tile<EPI_SPLIT, 2, 4, 4, 2> left, in range order, and the epilogue: one wavefront per 32 rows
// x 2 token groups.
template <int EPI, bool HI>
__global__ __launch_bounds__(256) void k_gemm_sum(DenseArgs d) {
  constexpr int CA = HI ? 2 : 1, R2 = 4, NW = 8;
  const GemmArgs& a = d.g;
  const int lane = threadIdx.x & 63, n_pairs = a.n_rows >> 5, n_gp = (d.n_groups + 1) >> 1;
  const int id = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (id >= n_pairs * n_gp) return;
  const int pr = id / n_gp, gp = id - pr * n_gp;  // 32-row pair of tiles, pair of token groups
  const int rb = pr / (2 * R2), ps = pr - rb * 2 * R2, wr = ps / R2, q = ps - wr * R2;
  const int cb = gp / (4 * CA), cs = gp - cb * 4 * CA, wc = cs / CA, c = cs - wc * CA;
  const int WG_G = 8 * CA, ncb = (d.n_groups + WG_G - 1) / WG_G, nrb = ((a.n_rows >> 4) + 15) / 16;
  const int per_pg = nrb * 8, pg = cb / 8, width = min(8, ncb - pg * 8), ti = pg * per_pg + rb * width + (cb - pg * 8);
  const size_t PLANE = (size_t)R2 * CA * 16 * NW * 64;
  const float* plane = a.planes + (size_t)ti * d.k_split * PLANE + (size_t)(q * CA + c) * 4 * (NW * 256) + ((size_t)(wr * 4 + wc) * 64 + lane) * 4;
  const int gs = __builtin_ctz(a.grp), t0 = ((pr >> gs) << (gs + 1)) + (pr & (a.grp - 1));
  const int rt[2] = {t0, t0 + a.grp};
  TileAhead<EPI, 1> ahead;
  ahead.request(d, 2 * gp, rt);
  f32x16 acc[1][1];
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[0][0][v] = 0.f;
  for (int s0 = 0; s0 < d.k_split; s0 += 4) {     // sixteen loads in flight
    float4 t[4][4];
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (s0 + s < d.k_split)
#pragma unroll
        for (int i = 0; i < 4; ++i) t[s][i] = *reinterpret_cast<const float4*>(plane + (size_t)(s0 + s) * PLANE + (size_t)i * (NW * 256));
#pragma unroll
    for (int s = 0; s < 4; ++s)
      if (s0 + s < d.k_split)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          acc[0][0][4 * i] += t[s][i].x; acc[0][0][4 * i + 1] += t[s][i].y; acc[0][0][4 * i + 2] += t[s][i].z; acc[0][0][4 * i + 3] += t[s][i].w;
        }
  }
  tile_epilogue<EPI, 1, 1, HI, true>(d, 2 * gp, rt, acc, nullptr, ahead);
}

// Bytes of one workgroup's partial sums of a K range.
static size_t split_unit_bytes(bool hi_only) { return (size_t)256 * 128 * (hi_only ? 2 : 1) * sizeof(float); }

// Workgroup tiles: 128 rows x 256 panel columns, two workgroups per compute unit (c0); 256 x 256, one (c1); 512 x 256, one (c2,
// hi + lo only: 128-token accumulators); 128 x 128 (c3) for grids of up to 256 such tiles, where the
// latency of the k-tiles is most of the time.  Costs in units of half a compute unit's time for a 256 x 256 tile; the
// larger tiles move less per product (c2 6 % faster than c1, c1 5 % than c0 where all fill the chip), the smaller ones
// fill it better: a lone c0 workgroup runs at 1 / 1.4 of its compute unit.  Measured, us (c0 / c1 / c2), hi + lo at
// 511 tokens: 27648 x 5120 274 / 246 / 217, 15360 x 5120 150 / 133 / 185, 5120 x 5120 74 / 101 / -; at 3001:
// 6400 x 6144 396 / 418 / 477.  Cut along K in S ranges: 5120 x 13824 at 511 tokens 214 (c0) against 137 + 17 for its sum.
// c3 against the best of the others, a whole pass: 68M shape at 60 tokens 131 / 142, at 600 in bf16 170 / 196; at a long K, two layers
// of 3072 at 120 tokens 281 / 297, of 4096 at 16 tokens 315 / 326, one 13B layer at 16 tokens in bf16 266 / 271, but in hi + lo
// 255 / 243 (and two layers of 2560 221 / 210): which of them gains there does not follow K, and the rule leaves that open.
DensePlan gemm_dense_plan(int n_rows, int KT, int n_groups, bool hi_only, size_t plane_bytes) {
  const int n_tiles = n_rows / 16;
  auto count = [&](const int na, const int nbt) { const int gg = nbt / (hi_only ? 1 : 2); return (long)((n_tiles + na - 1) / na) * ((n_groups + gg - 1) / gg); };
  const long wgs[4] = {count(8, 16), count(16, 16), count(32, 16), count(8, 8)};
  const long rem = wgs[0] % 512;
  const double c0 = ((double)(wgs[0] / 512) * 2.0 + (rem == 0 ? 0.0 : (rem <= 256 ? 1.4 : 2.0))) / 0.95;
  const double c1 = (double)((wgs[1] + 255) / 256) * 2.0, c2 = hi_only ? 1e30 : (double)((wgs[2] + 255) / 256) * 4.0 / 1.06;
  const double c3 = wgs[3] <= 256 ? 1.35 : 1e30;
  const double unit_us = 0.3 * KT;
  double best = (c0 < c1 ? (c0 < c2 ? c0 : c2) : (c1 < c2 ? c1 : c2));
  if (c3 < best) best = c3;
  best *= unit_us;
  int split = 1;
  for (int S = 2; S <= 16 && wgs[1] * S <= 256 && KT / S >= 8 && (size_t)wgs[1] * S * split_unit_bytes(hi_only) <= plane_bytes; ++S) {
    const double us = 2.0 / S * unit_us + 8.0 + (double)wgs[1] * S * (hi_only ? 0.262 : 0.131) * 2.0 / 4.0;   // two passes over the partial sums at 4 TB/s, a launch
    if (us < best) { best = us; split = S; }
  }
  const int tile = split > 1 ? 1 : (c3 < c0 ? 3 : (c2 < c0 && c2 < c1 ? 2 : (c1 < c0 ? 1 : 0)));
  const int stages = tile == 0 ? (wgs[0] <= 256 && KT >= 64 ? 6 : 3) : (tile == 1 ? 4 : (tile == 2 ? 3 : 8));
  return DensePlan{tile, split, wgs[tile], split > 1 ? (size_t)wgs[1] * split * split_unit_bytes(hi_only) : 0, stages};
}
// A matrix that reads a normalised row forms 1 / rms itself (narrow models: 64 sums of squares a row at most); a wide row's sums are read by
// every workgroup of its tokens, so one launch in front adds them up for all, and so it is where the matrix is cut along K.
bool dense_rms_in_launch(const DensePlan& p, int n_ssq) { return p.split == 1 && n_ssq <= 64; }

template <int EPI, int WR, int WC, int R2, int C2, int NST, int OCC, bool HI>
static void launch_tiles(const DenseArgs& d, const dim3 grid, hipStream_t s) {
  hipLaunchKernelGGL((k_gemm_tile<EPI, WR, WC, R2, C2, NST, OCC, HI>), grid, dim3(512), 0, s, d.g.W, d.g.X, d.xs, d.g.KT, d.g.n_rows, d.n_groups, d.g.grp,
                     d.k_split, d);
}

// Ring depths: a grid of at most a workgroup per compute unit takes the whole LDS: with two resident workgroups one computes while the
// other waits for its copies, a lone one has only its own ring to wait with.  c3 eight stages instead of three (68M shape at 511
// tokens: 2304 and 768 rows, K 768, 12.4 -> 11.0 and 12.7 -> 11.3 us a launch).  c0 six instead of three from K 2048 on, a whole pass: 13B layer
// at 130 tokens 358 -> 350 us, at 300 in bf16 391 -> 386, multi-query target layer at 1000 in bf16 939 -> 928, four layers of 2048 at 511 in bf16
// 545.6 -> 540; with K 768 filling the ring costs more than it hides (68M shape at 511 tokens 142.3 with three, 143.2 with six, at 1000
// 194.0 and 195.3).
template <int EPI, bool HI>
static hipError_t launch_gemm_tile(const DenseArgs& d0, hipStream_t s) {
  DenseArgs d = d0;
  const DensePlan p = gemm_dense_plan(d.g.n_rows, d.g.KT, d.n_groups, HI, d.g.planes != nullptr ? d.plane_bytes : 0);
  const dim3 grid(8u * (unsigned)((p.wgs * p.split + 7) / 8));
  if (d.g.ssq != nullptr && !dense_rms_in_launch(p, d.g.n_ssq)) {
    const hipError_t e = launch_rstd_groups(d.g.ssq, d.g.n_ssq, d.g.d_in, d.g.eps, d.rstd, d.n_groups, s);
    if (e != hipSuccess) return e;
    d.g.ssq = nullptr;
  }
  if (p.split > 1) {
    d.k_split = p.split;
    launch_tiles<EPI_SPLIT, 2, 4, 4, 2, 4, 2, HI>(d, grid, s);
    const long waves = (long)(d.g.n_rows / 32) * ((d.n_groups + 1) / 2);
    hipLaunchKernelGGL((k_gemm_sum<EPI, HI>), dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, d);
    return hipGetLastError();
  }
  switch (p.tile) {
    case 0:
      if (p.stages == 6) launch_tiles<EPI, 2, 4, 2, 2, 6, 2, HI>(d, grid, s);
      else launch_tiles<EPI, 2, 4, 2, 2, 3, 4, HI>(d, grid, s);
      break;
    case 1: launch_tiles<EPI, 2, 4, 4, 2, 4, 2, HI>(d, grid, s); break;
    case 2: if constexpr (!HI) launch_tiles<EPI, 4, 2, 4, 4, 3, 2, HI>(d, grid, s); break;
    default: launch_tiles<EPI, 4, 2, 1, 2, 8, 2, HI>(d, grid, s); break;
  }
  return hipGetLastError();
}

template <int EPI>
static hipError_t launch_gemm_dense_h(const DenseArgs& d, hipStream_t s) {
  return d.hi_only ? launch_gemm_tile<EPI, true>(d, s) : launch_gemm_tile<EPI, false>(d, s);
}

hipError_t launch_gemm_dense(const DenseArgs& d, int epi, hipStream_t s) {
  const GemmArgs& a = d.g;
  if (a.M != 16 || d.n_groups < 1 || a.KT < 1 || a.n_rows < 64 || (a.n_rows % 64) != 0) return hipErrorInvalidValue;
  if ((epi == EPI_QKV || epi == EPI_SWIGLU) && (a.grp < 1 || (a.grp & (a.grp - 1)) != 0 || (a.n_rows / 32) % a.grp != 0)) return hipErrorInvalidValue;
  if (epi == EPI_QKV && a.dh != 64 && a.dh != 128) return hipErrorInvalidValue;
  switch (epi) {
    case EPI_QKV: return launch_gemm_dense_h<EPI_QKV>(d, s);
    case EPI_SWIGLU: return launch_gemm_dense_h<EPI_SWIGLU>(d, s);
    case EPI_PARTIAL: return launch_gemm_dense_h<EPI_PARTIAL>(d, s);
    case EPI_GELU: return launch_gemm_dense_h<EPI_GELU>(d, s);
    default: return hipErrorInvalidValue;
  }
}

// 1 / rms of every row of the prompt pass from its per-tile sums of squares: 64 partial sums per row, added in order (bound by
// the latency of the few loads per thread: four in flight; 7.3 us with 16 partial sums and one load at a time, 4.8 now, d 5120).
__global__ __launch_bounds__(1024) void k_rstd_groups(const float* __restrict__ ssq, int n_ssq, int d, float eps,
                                                      float* __restrict__ rstd) {
  __shared__ float part[64][16];
  const int r = blockIdx.x, m = threadIdx.x & 15, p = threadIdx.x >> 4;
  const float* sq = ssq + (size_t)r * n_ssq * 16;
  float s = 0.f;
  for (int i0 = p; i0 < n_ssq; i0 += 256) {
    float t[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = i0 + 64 * i < n_ssq ? sq[(i0 + 64 * i) * 16 + m] : 0.f;
    s += (t[0] + t[1]) + (t[2] + t[3]);
  }
  part[p][m] = s;
  __syncthreads();
  if (threadIdx.x < 16) {
    float tot = 0.f;
#pragma unroll
    for (int i = 0; i < 64; ++i) tot += part[i][m];
    rstd[r * 16 + m] = 1.0f / sqrtf(tot / (float)d + eps);
  }
}

hipError_t launch_rstd_groups(const float* ssq, int n_ssq, int d, float eps, float* rstd, int n_groups, hipStream_t s) {
  if (n_groups < 1 || n_ssq < 1) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_rstd_groups, dim3(n_groups), dim3(1024), 0, s, ssq, n_ssq, d, eps, rstd);
  return hipGetLastError();
}


// ---------------------------------------------------------------------------------------------
// QKV projection and attention of one layer in ONE launch
// ---------------------------------------------------------------------------------------------
//
// The attention of a head needs only the projection rows of its queries, keys and values, so the dependency
// between the two phases is per head, not grid-wide.  A projection workgroup finishes its
// rows (rotary, query rows, cache entries: write-through stores) and adds 1 to the counter of every head that reads them: its own,
// or all the query heads of a K / V head.  An attention workgroup waits until the counter shows all of its head's
// (bounded: after `limit` polls it sets the
// abort word and goes on with unusable data; the LM head then stores NaN logits and the arg-max and loop-finish
// kernels turn a set abort word into -1 outputs), with its first cache loads already in flight where they cannot touch a 128-byte line that the
// projection is still writing.  The head's ranges are merged by the last one to finish, as in the
// stand-alone attention kernel; that workgroup also zeroes the head's counter for the next launch.  The counters are 256 bytes apart.
//
// OWN: the attention has workgroups of its own, numbered behind the projection's; two steps of their cache entries arrive while the
// projection runs.  Otherwise (the projection's workgroups fill the chip: one per compute unit) the workgroups of a head are neighbours and become
// the ranges of its attention when they have counted themselves in.  Either way nobody waits before it has signalled, so the
// launch completes whenever all its workgroups are resident at once; the launcher checks that they fit.
// us a pass, one launch / two (the draft models' one or two tokens take k_chain since): a 68M draft token 66.8 / 67.8 at 250 positions, 68.1 / 69.3 at 523, 72.3 / 76.6 at 2475; a multi-query draft token
// (12 layers) 300.3 / 309.3 at 250, 314.3 / 324.6 at 640, 329.6 / 366.3 at 2475; two layers of 16 heads on 4 K / V heads, 6 tokens, 122.4 / 125.1
// at 640, 127.3 / 135.8 at 2475; two 13B layers (not OWN: 240 projection workgroups) 298.4 / 301.0 for 6 tokens at 640, 321.6 / 321.9 for 12 at
// 2475, and at 40 the two launches: 291.5 (301 when the projection's workgroups took the attention there too).
constexpr int QA_READY_SLOT = QKV_ATTN_READY_SLOT;   // ints between two heads' counters

struct HeadWaitHook {
  int* ready; int n; unsigned* abort_word; int limit;   // limit: polls (each a memory round trip, about 1 us) before giving up
  uint32_t halted;                                // a halted step's projection counts nobody in
  __device__ __forceinline__ void operator()() const {
    if (threadIdx.x == 0 && !flag_set(halted)) {
      int spins = 0;
      if (limit < 0) __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      while (limit >= 0 && __hip_atomic_load(ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < n) {
        if (++spins > limit) {
          __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
    }
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }
};

// LN: the model's norms are LayerNorms.  The leading arguments: see k_gemm.
template <int P, int RT, int U, int DH, bool LN, bool OWN>
__global__ __launch_bounds__(512) void k_qkv_attn(const bf16_t* W, const bf16_t* X, const uint32_t* gate, const float* ssq, int KT, int n_ssq,
                                                  int M, int nq, int nkv, int pos0, GemmArgs g, AttnArgs a, int* ready, unsigned* abort_word, int safe_end, int limit) {
  g.W = W; g.X = X; g.gate = gate; g.ssq = ssq; g.KT = KT; g.grp = DH / 32; g.n_ssq = n_ssq; g.M = M; a.M = M; g.pos0 = pos0; a.pos0 = pos0;
  g.nq = nq; g.nkv = nkv; a.nq = nq; a.nkv = nkv;
  constexpr int UH = DH / (16 * RT), G = 3 * UH;   // workgroups per q / K / V part of a head; arrivals that a head waits for
  static_assert(UH >= 1 && UH * 16 * RT == DH, "a head part is a whole number of workgroups");
  union Smem { GemmSmem<RT, 8, LN> gemm; AttnSmem<DH, 8> attn; };
  __shared__ Smem sm;
  const int id = blockIdx.x;
  const uint32_t halted = gate_request(g.gate);
  // projection unit `b`; then, its workgroup's stores having completed, it is counted in for heads first .. first + n - 1
  auto project = [&](const int b, const int first, const int n) {
    gemm_unit<P, RT, EPI_QKV, 8, U, true, NoHook, LN>(g, b, 0, g.KT, 0, 1, sm.gemm);
    if (flag_set(halted)) return false;           // uniform over the launch; nothing has been written
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);                // this wavefront's write-through stores have completed
    __syncthreads();                              // ... and those of the whole workgroup
    for (int i = threadIdx.x; i < n; i += 512) __hip_atomic_fetch_add(ready + (first + i) * QA_READY_SLOT, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return true;
  };
  if constexpr (OWN) {
    const int n_gemm = (g.nq + 2 * g.nkv) * UH;
    if (id < n_gemm) {
      const int rep = g.nkv == 1 ? g.nq : (g.nq == g.nkv ? 1 : g.nq / g.nkv), hu = id / UH;
      project(id, hu < g.nq ? hu : (hu - g.nq) % g.nkv * rep, hu < g.nq ? 1 : rep);
      return;
    }
    const int split = (id - n_gemm) / g.nq, head = id - n_gemm - split * g.nq;
    int* rdy = ready + head * QA_READY_SLOT;
    const HeadWaitHook wait{rdy, G, abort_word, limit, halted};
    if (pos0 + M <= ATTN_HEAD_MAX_CTX) {
      AttnWhole<DH, true> at(a, head);
      at.request(safe_end);
      wait();
      at.run(sm.attn, safe_end, halted);
      if (threadIdx.x == 0 && !flag_set(halted)) __hip_atomic_store(rdy, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      attn_range<DH, 8, false, false, true, HeadWaitHook>(a, head, split, sm.attn, halted, wait, safe_end, rdy);
    }
  } else {                                        // a K / V head per query head
    const int head = id / G, j = id % G, part = j / UH, sub = j % UH;
    const int hu = part == 0 ? head : (part == 1 ? g.nq + head : g.nq + g.nkv + head);
    if (!project(hu * UH + sub, head, 1) || j >= a.n_splits) return;
    int* rdy = ready + head * QA_READY_SLOT;
    attn_range<DH, 8, false, false, true, HeadWaitHook>(a, head, j, sm.attn, 0u, HeadWaitHook{rdy, G, abort_word, limit, 0u}, safe_end, rdy);
  }
}

// Workgroups of `kernel` (512 threads, static LDS only) that the device holds at once.
static long resident_capacity(const void* kernel) {
  int per_cu = 0, dev = 0;
  hipDeviceProp_t prop;
  if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 512, 0) != hipSuccess || per_cu < 1) return 0;
  return (long)per_cu * prop.multiProcessorCount;
}

template <int P, int RT, int DH, bool LN, bool OWN>
static long qkv_attn_capacity() {
  static const long c = resident_capacity(reinterpret_cast<const void*>(k_qkv_attn<P, RT, gemm_buffers(RT, P), DH, LN, OWN>));
  return c;
}

// How the context is dealt, and which form the launch takes.  The deal is the one of the workgroups that shared the projection's
// before there were others: a workgroup per G-th of the context, 128 positions at least, where heads have their own K / V; the ranges of
// the stand-alone attention elsewhere.  It decides the order of the sums, so a form is chosen by what fits and the deal is left alone.
QkvAttnPlan qkv_attn_plan(int n_rows, int nq, int nkv, int dh, bool layernorm, int total, int rt, long cap_shared, long cap_own) {
  QkvAttnPlan p{0, 0, 0, 0};
  const long n_gemm = n_rows / (16 * rt);
  const bool whole = total <= ATTN_HEAD_MAX_CTX, sharing = !layernorm && nq == nkv && n_gemm <= cap_shared;
  if (sharing) {
    const int G = 3 * dh / (16 * rt);
    p.split_len = ((total + G - 1) / G + 31) / 32 * 32;
    if (p.split_len < ATTN_SPLIT_LEN) p.split_len = ATTN_SPLIT_LEN;
  } else {
    p.split_len = attn_split_len(total);
  }
  p.n_splits = (total + p.split_len - 1) / p.split_len;
  const long own = n_gemm + (long)nq * (whole ? 1 : p.n_splits);
  // (form 2 for 32-row units only: 64-row units are 200 workgroups or more, which leave room for a few head counts up to 256 positions)
  if (rt == 2 && own <= cap_own) { p.form = 2; p.wgs = own; }     // all resident at once
  else if (sharing && !whole) { p.form = 1; p.wgs = n_gemm; }
  return p;
}
int qkv_attn_rt(int n_rows) { return (n_rows % 64 == 0 && n_rows / 64 >= 200) ? 4 : 2; }      // the row tiles of the stand-alone QKV launch

// Workgroups of the two forms that the GPU holds at once.
template <int P, int RT, int DH>
static void qkv_attn_capacities_rt(bool ln, long* shared, long* own) {
  *shared = qkv_attn_capacity<P, RT, DH, false, false>();
  *own = 0;
  if constexpr (RT == 2) *own = ln ? qkv_attn_capacity<P, RT, DH, true, true>() : qkv_attn_capacity<P, RT, DH, false, true>();
}
#define QKV_ATTN_BY_SHAPE(f, p1, rt, dh, ...) \
  ((dh) == 128 ? ((rt) == 4 ? ((p1) ? f<1, 4, 128>(__VA_ARGS__) : f<2, 4, 128>(__VA_ARGS__)) : ((p1) ? f<1, 2, 128>(__VA_ARGS__) : f<2, 2, 128>(__VA_ARGS__))) \
               : ((rt) == 4 ? ((p1) ? f<1, 4, 64>(__VA_ARGS__) : f<2, 4, 64>(__VA_ARGS__)) : ((p1) ? f<1, 2, 64>(__VA_ARGS__) : f<2, 2, 64>(__VA_ARGS__))))
void qkv_attn_capacities(int M, int rt, int dh, bool layernorm, long* shared, long* own) {
  QKV_ATTN_BY_SHAPE(qkv_attn_capacities_rt, M <= 8, rt, dh, layernorm, shared, own);
}

template <int P, int RT, int DH>
static hipError_t launch_qkv_attn_rt(const GemmArgs& g, AttnArgs& a, int* ready, unsigned* abort_word, int safe_end, int limit, bool may_wait,
                                     bool* launched, hipStream_t s) {
  constexpr int U = gemm_buffers(RT, P);
  const bool ln = g.sum != nullptr;
  long cap_shared, cap_own;
  qkv_attn_capacities_rt<P, RT, DH>(ln, &cap_shared, &cap_own);
  const QkvAttnPlan p = qkv_attn_plan(g.n_rows, g.nq, g.nkv, DH, ln, a.pos0 + a.M, RT, cap_shared, cap_own);
  a.split_len = p.split_len; a.n_splits = p.n_splits;
  if (p.form == 0 || !may_wait) return hipSuccess;
  const dim3 grid((unsigned)p.wgs);
#define QKV_ATTN_ARGS grid, dim3(512), 0, s, g.W, g.X, g.gate, g.ssq, g.KT, g.n_ssq, g.M, g.nq, g.nkv, g.pos0, g, a, ready, abort_word, safe_end, limit
  if (p.form == 1) hipLaunchKernelGGL((k_qkv_attn<P, RT, U, DH, false, false>), QKV_ATTN_ARGS);
  if constexpr (RT == 2) {
    if (p.form == 2 && ln) hipLaunchKernelGGL((k_qkv_attn<P, RT, U, DH, true, true>), QKV_ATTN_ARGS);
    if (p.form == 2 && !ln) hipLaunchKernelGGL((k_qkv_attn<P, RT, U, DH, false, true>), QKV_ATTN_ARGS);
  }
#undef QKV_ATTN_ARGS
  *launched = true;
  return hipGetLastError();
}

// Sets *launched and enqueues the fused launch when the shape allows it and the forward may hold launches that wait; otherwise leaves *launched false and enqueues
// nothing (the caller then launches the QKV projection and the attention separately, the latter over a.split_len / a.n_splits,
// which are chosen here either way).
hipError_t launch_qkv_attn(const GemmArgs& g0, AttnArgs& a, int* ready, unsigned* abort_word, int limit, bool may_wait, bool* launched, hipStream_t s) {
  *launched = false;
  if (ready == nullptr || abort_word == nullptr) return hipSuccess;
  if (g0.nkv < 1 || g0.nq % g0.nkv != 0 || (g0.dh != 64 && g0.dh != 128)) return hipSuccess;
  if (g0.M < 1 || g0.M > 16 || g0.KT < 1 || g0.n_rows != (g0.nq + 2 * g0.nkv) * g0.dh || g0.grp != g0.dh / 32) return hipSuccess;
  if (g0.ssq != nullptr && (g0.n_ssq < 1 || g0.n_ssq > 512)) return hipErrorInvalidValue;
  if (a.M != g0.M || a.nq != g0.nq || a.nkv != g0.nkv || a.dh != g0.dh || a.pos0 != g0.pos0 || a.counters == nullptr) return hipErrorInvalidValue;
  GemmArgs g = g0;
  g.n_split = 1;
  const int pt = a.page_tokens;
  // positions below safe_end share no 128-byte line with the block's own positions: K rows are 128 bytes or more per
  // position; a V^T row holds the positions of one page, 64 to a line
  const int safe_end = (pt % 64 == 0) ? (a.pos0 & ~63) : (a.pos0 / pt) * pt;
  return QKV_ATTN_BY_SHAPE(launch_qkv_attn_rt, g.M <= 8, qkv_attn_rt(g.n_rows), g.dh, g, a, ready, abort_word, safe_end, limit, may_wait, launched, s);
}


// ---------------------------------------------------------------------------------------------
// all layers of a narrow model's forward over one or two tokens in ONE launch
// ---------------------------------------------------------------------------------------------
//
// A forward of a draft model is a chain of small dependent phases.  A launch per phase costs 2.4 us before it does anything and its
// weights arrive a round trip later: 26 us a layer for 9 MB (68M-class draft).  Here the phases of all layers run in workgroups that
// stay, each with a role: QKV projection + MLP input (n_pu of them), attention (n_groups x parts), O-projection + MLP output (16 columns of
// the residual stream each, whose rows live in registers from the first layer to the last).  A workgroup requests the weights of its next
// phase and the cache entries of its next layer while it waits.  13.8 us a layer; a 68M-class draft token with its features at 523
// positions 68.8 -> 49.6 us, four tokens of the 12-layer multi-query draft at 1490 1309 -> 828 us (feature kernel included).  What bounds it: five
// hand-offs of about 1.3 us a layer (six where a head's ranges are spread over workgroups) and, between them, the instructions of the one wavefront
// that finishes a tile.
//
// Hand-off: the data is its own flag.  Every buffer that one workgroup writes and others read inside the launch has an address of its
// own per layer and is filled with CHAIN_EMPTY words by the launch in front (k_chain_begin); a reader polls the words it needs until
// none is empty, so a hand-off is one write-through store and one L2-bypassing load (1.3 us over chains of 200, with 48 to 168 workgroups
// polling; store, drain, counter, poll and load 2.6).  A value that happens to be the empty word (a NaN
// with every bit set) is stored as another NaN.
// The sums are formed in the order of the launches per phase (the wavefronts' k-tiles, the K ranges of the MLP output, the deal of the
// context over ranges and wavefronts), so results do not depend on which of the two runs.
//
// All workgroups are resident at once: they fit the GPU (chain_plan), and no other launch that waits inside is in flight with it (forward_block).  Nobody
// waits without a bound (`limit` polls, then the abort word is set and the launch ends with unusable data, as in k_qkv_attn).
constexpr uint32_t CHAIN_EMPTY = 0xFFFFFFFFu;

__device__ __forceinline__ uint32_t chain_word(uint32_t x) { return x == CHAIN_EMPTY ? 0x7FC07FC0u : x; }
__device__ __forceinline__ void chain_put2(void* p, uint32_t a, uint32_t b) {
  __hip_atomic_store(reinterpret_cast<unsigned long long*>(p), (unsigned long long)chain_word(a) | ((unsigned long long)chain_word(b) << 32),
                     __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void chain_put16(void* base /* uniform */, uint32_t at, u32x4 v) {
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = chain_word(v[i]);
  __builtin_amdgcn_raw_buffer_store_b128(v, __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000), (int)at, 0, 16 /* sc1: write-through, as the atomics */);
}
// Compact panels: a block per 16 columns and token, [hi 16 | lo 16], and S (the panel of a normalised input) the columns' sum of squares and sum
// behind them.  A block leaves its workgroup with one store instruction: a second write-through store of a wavefront becomes
// visible 0.6 us after the first (chains of 200 hand-offs: 1.3 us with one store, 1.6 with hi and lo apart, 2.4 with the statistics in two more).
template <bool S> constexpr int chain_block_bytes() { return S ? 128 : 64; }
// A finishing wavefront has one value a lane: row r = lane % 16 of a tile, token m = lane / 32; lanes 16 .. 31 of a token are its second tile's rows, or
// copies of the first's.  The instructions of that one wavefront are what a phase waits for: with four rows a lane, as the matrix unit
// leaves them, a phase took 0.3 us longer.
__device__ __forceinline__ float chain_neighbour(float v) { return dpp_f<DPP_QUAD_XOR1, 0xF>(0.f, v); }          // lane ^ 1's
// x z of this lane and its neighbour as bf16 hi (lanes 0 .. 15 of a token) or lo (16 .. 31), in the even lanes
__device__ __forceinline__ uint32_t chain_halves(const float x, const float z, const int lane) {
  const HiLo s = split_product<true>(x, z, chain_neighbour(x), chain_neighbour(z));
  return (lane & 16) ? s.lo : s.hi;
}
__device__ __forceinline__ void chain_put4b(char* p, uint32_t v) {
  __hip_atomic_store(reinterpret_cast<uint32_t*>(p), chain_word(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Stores a block: even lanes the words of chain_halves, odd ones (S) the statistics.
template <int M, bool S>
__device__ __forceinline__ void chain_put_block(char* panel, const int slot, const int lane, const uint32_t word, const float sq, const float sx) {
  const int r = lane & 15, hi = (lane & 16) == 0, m = lane >> 5;
  const bool even = (r & 1) == 0;
  const uint32_t v = even ? word : (r == 1 ? __float_as_uint(sq) : (r == 3 ? __float_as_uint(sx) : 0u));
  if (m < M && (even || (S && hi && r < 8))) chain_put4b(panel + (slot * M + m) * chain_block_bytes<S>() + (even ? (hi ? 0 : 32) + r * 2 : 64 + (r >> 1) * 4), v);
}

// What the addresses of a phase are formed from, hidden from the compiler: it would form those of every phase in front of the loop over the
// layers and keep them in registers that the weights in flight need.
__device__ __forceinline__ void chain_opaque(int& lane, int& w) { asm volatile("" : "+v"(lane), "+s"(w)); }

// Polls N 16-byte pieces per lane, at `base` (uniform) + p, until none has an empty word.  A lane without a piece of its own polls one of its
// wavefront's (`on` false): no branches around the loads.
template <int N>
struct ChainWait {
  const char* base; uint32_t p[N]; bool on[N]; u32x4 v[N];
  __device__ __forceinline__ bool attempt() {
    unsigned long long lo[N], hi[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      lo[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(base + p[i]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      hi[i] = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(base + p[i] + 8), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    bool ok = true;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      v[i] = u32x4{(uint32_t)lo[i], (uint32_t)(lo[i] >> 32), (uint32_t)hi[i], (uint32_t)(hi[i] >> 32)};
      ok = ok && v[i][0] != CHAIN_EMPTY && v[i][1] != CHAIN_EMPTY && v[i][2] != CHAIN_EMPTY && v[i][3] != CHAIN_EMPTY;
    }
    return ok;
  }
  __device__ __forceinline__ void run(unsigned* abort_word, const int limit) {
    for (int spins = 0;; ++spins) {
      const bool ok = attempt();
      if (limit >= 0 && __ballot(!ok) == 0ull) return;
      // (once another wavefront has given up, what this one waits for may never come)
      if (spins >= limit || ((spins & 1023) == 1023 && __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u)) {
        __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
      }
    }
  }
};

constexpr int CHAIN_PARTS = 128;       // (range, wavefront, column) sums of a workgroup's share of the attention
struct ChainGemmSmem {
  u32x4 stage[8][64 * 3], stage2[8][64];       // a wavefront's panel pieces on their way to the operand order; zeros where a tile has none
  f32x4 red[2][8][4][8];               // [phase parity][wavefront][tile or K range][4-row group, token]
  alignas(16) float ssq[2][CHAIN_MAX_TOKENS][64], sum[2][CHAIN_MAX_TOKENS][64];      // a row's slots in the order they are added up
};
struct ChainAttnSmem {
  alignas(16) float o[CHAIN_PARTS][64]; float m[CHAIN_PARTS], l[CHAIN_PARTS];
  alignas(16) float ro[32][64]; float rm[32], rl[32];                   // ranges' records, where one workgroup has them all
  u32x4 q[2][2][64];                   // the queries as operands: [hi | lo][32 channels][lane]
  alignas(16) bf16_t kv[CHAIN_MAX_TOKENS][2][64];                       // the block's own keys and values
};

// One matrix phase of a workgroup: RT row tiles (or K ranges: NS of them) x the wavefront's KPW k-tiles per range.
// k-tile i of a range: kb + w + 8 i.
template <int M, int RT, int NS, int KPW>
struct ChainTiles {
  u32x4 A[NS * KPW][RT];
  static __device__ __forceinline__ int seg_begin(const int KT, const int s, const int n_seg) {
    return NS == 1 ? (s == 0 ? 0 : KT) : (int)((unsigned)(KT * s) / (unsigned)n_seg);
  }
  __device__ __forceinline__ void request(const bf16_t* W, const int (&rt)[RT], const int KT, const int n_seg, const int w, const int lane) {
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
      for (int i = 0; i < KPW; ++i) {
        // (past the range: a tile that is multiplied by zeros, without a branch around registers that are in flight)
        const int kt = min(seg_begin(KT, s, n_seg) + w + 8 * i, (s < n_seg ? seg_begin(KT, s + 1, n_seg) : KT) - 1);
#pragma unroll
        for (int r = 0; r < RT; ++r)
          A[s * KPW + i][r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(W) + (size_t)((uint32_t)(rt[r] * KT + kt) * 1024u)) + lane);
      }
  }
  // sets up the wait for this wavefront's pieces of `panel`: piece lane + 64 r of the list [tile][token][two blocks of hi 2 | lo 2 (| statistics)]
  template <bool S, int N>
  __device__ __forceinline__ void pieces(ChainWait<N>& wt, const char* panel, const int KT, const int n_seg, const int w, const int lane) const {
    constexpr int PB = S ? 5 : 4, PT = 2 * PB;
    static_assert(N * 64 >= NS * KPW * PT * M, "a lane per piece");
    wt.base = panel;
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const unsigned c = lane + 64 * r, q = c / (PT * M), of = c - q * (PT * M), sg = q / KPW, i = q - sg * KPW;
      const int kt = seg_begin(KT, sg, n_seg) + w + 8 * (int)i;
      wt.on[r] = q < NS * KPW && (int)sg < n_seg && kt < seg_begin(KT, sg + 1, n_seg);
      const unsigned token = of / PT, pc = of - token * PT, blk = pc / PB;
      wt.p[r] = ((wt.on[r] ? 2u * kt + blk : 2u * min(w, KT - 1)) * M + (wt.on[r] ? token : 0u)) * chain_block_bytes<S>() + (pc - blk * PB) * 16u;
    }
  }
  template <bool S, int N, int NST>
  __device__ __forceinline__ void products(const ChainWait<N>& wt, u32x4 (&stage)[NST], f32x4 (*red)[8] /* [tile or range][8] */, const int lane) const {
    constexpr int PB = S ? 5 : 4, PT = 2 * PB;
    static_assert(NST >= N * 64, "a place per piece");
#pragma unroll
    for (int r = 0; r < N; ++r) if (wt.on[r]) stage[lane + 64 * r] = wt.v[r];
    __builtin_amdgcn_wave_barrier();
    const int n = lane & 15, g = lane >> 4, m = M == 1 ? 0 : n & 1;          // columns without a token repeat one that has
    const u32x4* at = stage + m * PT + (g >> 1) * PB + (n >> 3) * 2 + (g & 1);
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      f32x4 acc[RT];
#pragma unroll
      for (int r = 0; r < RT; ++r) acc[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int i = 0; i < KPW; ++i) {
        const bf16x8 b = as_bf16x8(at[(s * KPW + i) * (PT * M)]);
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(A[s * KPW + i][r]), b, acc[r], 0, 0, 0);
      }
#pragma unroll
      for (int r = 0; r < RT; ++r) {
        f32x4 y;
#pragma unroll
        for (int v = 0; v < 4; ++v) y[v] = acc[r][v] + dpp_f<DPP_ROW_ROR8, 0xF>(0.f, acc[r][v]);     // hi + lo
        if (n < M) red[s * RT + r][g * 2 + n] = y;
      }
    }
  }
};

template <bool LN>
struct ChainNorm {
  // the statistics among this lane's pieces, to where the sum finds them: slots in the order of gemm_unit (wavefront, then row of the
  // wavefront; a second slot 32 further on is added to the first)
  template <int M, int N>
  static __device__ __forceinline__ void share(const ChainWait<N>& wt, float (&ssq)[CHAIN_MAX_TOKENS][64], float (&sum)[CHAIN_MAX_TOKENS][64], const int w, const int lane) {
#pragma unroll
    for (int r = 0; r < N; ++r) {
      const unsigned c = lane + 64 * r, q = c / (10 * M), of = c - q * (10 * M), token = of / 10, pc = of - token * 10;
      if (wt.on[r] && (pc == 4 || pc == 9)) {
        const int s = 2 * (w + 8 * (int)q) + (pc == 9 ? 1 : 0), at = (s & 7) * 4 + ((s & 31) >> 3) + (s & 32);
        ssq[token][at] = __uint_as_float(wt.v[r][0]);
        if (LN) sum[token][at] = __uint_as_float(wt.v[r][1]);
      }
    }
  }
  // Sum of 32 pairs (slot, slot 32 further on) in order: a lane of a 16-lane row reads two pairs, and the additions take them from lane to lane
  // (a lane that reads them all adds twice as often, behind sixteen reads: 0.2 us a phase).
  static __device__ __forceinline__ float total(const float (&x)[64], const int lane) {
    const int i = lane & 15;
    const float u0 = x[i] + x[32 + i], u1 = x[16 + i] + x[48 + i];
    float t = 0.f;
#define CHAIN_ADD(u, k) t += dpp_f<0x150 + k, 0xF>(0.f, u);
#define CHAIN_ADD8(u, k) CHAIN_ADD(u, k) CHAIN_ADD(u, k + 1) CHAIN_ADD(u, k + 2) CHAIN_ADD(u, k + 3) CHAIN_ADD(u, k + 4) CHAIN_ADD(u, k + 5) CHAIN_ADD(u, k + 6) CHAIN_ADD(u, k + 7)
    CHAIN_ADD8(u0, 0) CHAIN_ADD8(u0, 8) CHAIN_ADD8(u1, 0) CHAIN_ADD8(u1, 8)
#undef CHAIN_ADD8
#undef CHAIN_ADD
    return t;
  }
  // y normalised; vg, vb: the LayerNorm's two vectors at this lane's row
  template <int M>
  static __device__ __forceinline__ float apply(const float y, const float (&ssq)[CHAIN_MAX_TOKENS][64], const float (&sum)[CHAIN_MAX_TOKENS][64], const int d, const float eps,
                                                const float vg, const float vb, const int lane) {
    float ss = total(ssq[0], lane);
    if (M == 2) { const float s1 = total(ssq[1], lane); ss = (lane & 32) ? s1 : ss; }
    if (LN) {
      float sx = total(sum[0], lane);
      if (M == 2) { const float s1 = total(sum[1], lane); sx = (lane & 32) ? s1 : sx; }
      const float mean = sx / (float)d;
      const float var = fmaxf(ss / (float)d - mean * mean, 0.f);
      const float rstd = 1.0f / sqrtf(var + eps);
      return rstd * (y - mean * vg) + vb;
    }
    const float rstd = 1.0f / sqrtf(ss / (float)d + eps);
    return y * rstd;
  }
};

// Sum of the wavefronts' partial tiles in wavefront order, this lane's row and token.
template <int M>
__device__ __forceinline__ float chain_sum(const f32x4 (&red)[8][4][8], const int tile, const int lane) {
  const float* p = reinterpret_cast<const float*>(&red[0][tile][((lane & 15) >> 2) * 2 + (M == 1 ? 0 : lane >> 5)]) + (lane & 3);
  float y = p[0];
#pragma unroll
  for (int ww = 1; ww < 8; ++ww) y += p[ww * 4 * 8 * 4];
  return y;
}

// QKV projection and MLP input of every layer.
template <int M, bool LN, int KPW>
__device__ __forceinline__ void chain_projections(const ChainArgs& a, ChainGemmSmem& sm, const int b, const uint32_t halted) {
  constexpr int RU = LN ? 2 : 4, TU = LN ? 1 : 2;         // MLP input: tiles per workgroup, per output unit (32 outputs either way)
  constexpr int N = (KPW * 10 * M + 63) / 64;     // pieces per lane
  int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = M == 1 ? 0 : lane >> 5, r = lane & 15, half = (lane >> 4) & 1;          // of a finishing wavefront: see chain_put_block
  const int KT = a.d >> 5, n_p = (a.nq + 2 * a.nkv) * 2, n_u = a.d_ff >> 5;
  const int rp[2] = {((b >> 1) << 2) + (b & 1), ((b >> 1) << 2) + (b & 1) + 2};      // tiles 32 rows apart: rotary partners
  const int head = rp[0] >> 2, ch = (rp[0] & 3) * 16 + r + 32 * half;          // this workgroup's head part and the lane's channel: tiles 32 apart
  const bool is_q = head < a.nq, is_v = head >= a.nq + a.nkv;
  const int kvh = is_q ? 0 : (is_v ? head - a.nq - a.nkv : head - a.nq);
  int ru[RU];
#pragma unroll
  for (int i = 0; i < RU; ++i) ru[i] = b * RU + i;
  const int pos = a.pos0 + m;
  const int pt = a.page_tokens, lp = pos >> __builtin_ctz(pt), off = pos & (pt - 1);
  const bool p_ep = b < n_p && w == 0, puts = (lane >> 5) < M;
  for (int i = threadIdx.x; i < 2 * CHAIN_MAX_TOKENS * 64; i += 512) { (&sm.ssq[0][0][0])[i] = 0.f; (&sm.sum[0][0][0])[i] = 0.f; }   // slots past the row
  for (int i = threadIdx.x; i < 8 * 64 * 3; i += 512) (&sm.stage[0][0])[i] = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  int page = lp;
  float2 cs = make_float2(1.f, 0.f);              // cos, sin of the channel pair
  if (p_ep) {
    if (!is_q && a.page_table != nullptr) page = a.page_table[lp];
    if (!LN && a.rope != nullptr && !is_v) {
      cs = *reinterpret_cast<const float2*>(a.rope + ((size_t)pos * 32 + (ch & 31)) * 2);
    }
  }
  bool first = true;
  for (int l = 0; l < a.n_layers; ++l) {
    chain_opaque(lane, w);
    const ChainLayer& L = a.layers[l];
    char* hand = a.hand + (size_t)l * a.layer_bytes;
    if (b < n_p) {
      ChainTiles<M, 2, 1, KPW> wq;
      wq.request(L.wqkv, rp, KT, 1, w, lane);
      float vg = 0.f, vb = 0.f;
      if (LN && p_ep) { vg = L.ln[rp[half] * 16 + r]; vb = L.ln[n_p * 32 + rp[half] * 16 + r]; }
      if (first && flag_set(halted)) return;
      first = false;
      ChainWait<N> wt;
      wq.template pieces<true>(wt, hand + a.o_xn, KT, 1, w, lane);
      wt.run(a.abort_word, a.limit);
      wq.template products<true>(wt, sm.stage[w], sm.red[0][w], lane);
      ChainNorm<LN>::template share<M, N>(wt, sm.ssq[0], sm.sum[0], w, lane);
      __syncthreads();
      if (p_ep) {
        int ch_l = ch, off_l = off;
        asm volatile("" : "+v"(ch_l), "+v"(off_l));
        float x = ChainNorm<LN>::template apply<M>(chain_sum<M>(sm.red[0], half, lane), sm.ssq[0], sm.sum[0], a.d, a.eps, vg, vb, lane);
        if (!LN && a.rope != nullptr && !is_v) {  // (the rounding of qkv_store)
          const Pair32 p = swap16(x);             // the channel of the lower half and its partner
          x = half ? fmaf(p.b, cs.x, p.a * cs.y) : fmaf(p.a, cs.x, -(p.b * cs.y));
        }
        if (is_q) {
          if (puts) chain_put4b(reinterpret_cast<char*>(l + 1 == a.n_layers ? a.q_last : reinterpret_cast<float*>(hand + a.o_q)) + (uint32_t)((m * a.nq + head) * 64 + ch_l) * 4u,
                                __float_as_uint(x));
        } else {
          const uint32_t xx = pack_bf16(x, chain_neighbour(x));
          if (puts && (lane & 1) == 0) chain_put4b(hand + a.o_kv + (uint32_t)((((kvh * M + m) * 2 + (is_v ? 1 : 0)) * 64 + ch_l) * 2), xx);
          // the cache entry, for later launches
          bf16_t* blk = a.kv_pages + (size_t)l * a.kv_layer_stride + (((size_t)page * 2 + (is_v ? 1 : 0)) * a.nkv + kvh) * pt * 64;
          if (puts) blk[is_v ? (size_t)ch_l * pt + off_l : (size_t)off_l * 64 + ch_l] = (bf16_t)xx;
        }
      }
    }
    if (b < n_u) {
      chain_opaque(lane, w);
      ChainTiles<M, RU, 1, KPW> wu;
      wu.request(L.w_in, ru, KT, 1, w, lane);
      const bool ep = w < 2;
      float vg = 0.f, vb = 0.f;
      if (LN && ep) { vg = L.ln[2 * n_p * 32 + (b * 2 + w) * 16 + r]; vb = L.ln[2 * n_p * 32 + a.d_ff + (b * 2 + w) * 16 + r]; }
      if (first && flag_set(halted)) return;
      first = false;
      ChainWait<N> wt;
      wu.template pieces<true>(wt, hand + a.o_xn2, KT, 1, w, lane);
      wt.run(a.abort_word, a.limit);
      wu.template products<true>(wt, sm.stage[w], sm.red[1][w], lane);
      ChainNorm<LN>::template share<M, N>(wt, sm.ssq[1], sm.sum[1], w, lane);
      __syncthreads();
      if (ep) {
        const float y = ChainNorm<LN>::template apply<M>(chain_sum<M>(sm.red[1], w * TU + (TU == 2 ? half : 0), lane), sm.ssq[1], sm.sum[1], a.d, a.eps, vg, vb, lane);
        const Pair32 p = swap16(y);               // TU 2: the row's gate and up
        const float u = LN ? 0.5f * y : p.a / (1.0f + expf(-p.a)), z = LN ? 1.0f + erff(y * 0.70710678118654752f) : p.b;       // the activation is u z
        chain_put_block<M, false>(hand + a.o_act, b * 2 + w, lane, chain_halves(u, z, lane), 0.f, 0.f);
      }
    }
  }
}

// O-projection and MLP output of every layer for 16 columns of the residual stream.
template <int M, bool LN, int KPW, int NSEG>
__device__ __forceinline__ void chain_residual(const ChainArgs& a, ChainGemmSmem& sm, const int b, const uint32_t halted) {
  int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int m = M == 1 ? 0 : lane >> 5, r = lane & 15;          // of the finishing wavefront: see chain_put_block
  const int KTQ = a.nq * 2, KTF = a.d_ff >> 5, col = b * 16 + r;
  const bool ep = w == 0;
  float h = ep ? a.h[(size_t)m * a.d + col] : 0.f;
  const int rt[1] = {b};
  for (int i = threadIdx.x; i < 8 * 64 * 4; i += 512) (i < 8 * 64 * 3 ? (&sm.stage[0][0])[i] : (&sm.stage2[0][0])[i - 8 * 64 * 3]) = u32x4{0u, 0u, 0u, 0u};
  __syncthreads();
  // sums over a token's 16 columns, in the order of gemm_unit: four at a time, then the four in pairs
  auto columns_sum = [](float v) { v += dpp_f<DPP_ROW_HALF_MIRROR, 0xF>(0.f, v); return v + dpp_f<DPP_ROW_MIRROR, 0xF>(0.f, v); };
  auto squares = [&] {
    const float e = fmaf(h, h, chain_neighbour(h * h));            // (even lanes)
    const float q = e + dpp_f<DPP_QUAD_XOR2, 0xF>(0.f, e);
    return columns_sum(dpp_f<0x00, 0xF>(0.f, q));                  // (lane 0 of four to all of them)
  };
  auto values = [&] {
    float q = h + chain_neighbour(h);
    q += dpp_f<DPP_QUAD_XOR2, 0xF>(0.f, q);
    return columns_sum(q);
  };
  auto next_input = [&](const float y, const float gn, char* panel) {
    h += y;
    chain_put_block<M, true>(panel, b, lane, chain_halves(h, gn, lane), squares(), LN ? values() : 0.f);
  };
  for (int l = 0; l < a.n_layers; ++l) {
    chain_opaque(lane, w);
    const ChainLayer& L = a.layers[l];
    char* hand = a.hand + (size_t)l * a.layer_bytes;
    const bool last = l + 1 == a.n_layers;
    ChainTiles<M, 1, 1, KPW> wo;
    wo.request(L.wo, rt, KTQ, 1, w, lane);
    ChainTiles<M, 1, NSEG, KPW> wd;
    wd.request(L.w_out, rt, KTF, a.n_seg, w, lane);
    float g2 = 0.f, g1 = 0.f;
    if (ep) { g2 = L.norm2_g[col]; g1 = L.next_g[col]; }
    if (l == 0 && flag_set(halted)) return;
    {
      ChainWait<1> wt;
      wo.template pieces<false>(wt, hand + a.o_xattn, KTQ, 1, w, lane);
      wt.run(a.abort_word, a.limit);
      wo.template products<false>(wt, sm.stage2[w], sm.red[0][w], lane);
      __syncthreads();
      if (w == 0) next_input(chain_sum<M>(sm.red[0], 0, lane), g2, hand + a.o_xn2);
    }
    {
      ChainWait<(NSEG * KPW * 8 * M + 63) / 64> wt;
      wd.template pieces<false>(wt, hand + a.o_act, KTF, a.n_seg, w, lane);
      wt.run(a.abort_word, a.limit);
      wd.template products<false>(wt, sm.stage[w], sm.red[1][w], lane);
      __syncthreads();
      if (w == 0) {
        float y = chain_sum<M>(sm.red[1], 0, lane);
#pragma unroll
        for (int s = 1; s < NSEG; ++s) {
          const float z = chain_sum<M>(sm.red[1], s, lane);
          if (s < a.n_seg) y += z;
        }
        if (!last) {
          next_input(y, g1, hand + a.layer_bytes + a.o_xn);
        } else {                                  // the LM head's launch reads the ordinary panels
          h += y;
          const uint32_t word = chain_halves(h, g1, lane);
          const float sq = squares(), sx = LN ? values() : 0.f;
          if ((lane >> 5) < M) {
            if ((lane & 1) == 0)
              *reinterpret_cast<uint32_t*>(a.x_out + ((size_t)(col >> 5) * 64 + ((col & 31) >> 3) * 16 + m + ((lane & 16) ? 8 : 0)) * 8 + (col & 7)) = word;
            if ((lane & 31) == 0) a.ssq_out[b * 16 + m] = sq;
            if (LN && (lane & 31) == 0) a.sum_out[b * 16 + m] = sx;
          }
        }
      }
    }
  }
}

// Lane i of a 16-lane row's v to all of the row, i = 0 .. 7.
__device__ __forceinline__ void row_bcast8(const float v, float (&o)[8]) {
  o[0] = dpp_f<0x150, 0xF>(0.f, v); o[1] = dpp_f<0x151, 0xF>(0.f, v); o[2] = dpp_f<0x152, 0xF>(0.f, v); o[3] = dpp_f<0x153, 0xF>(0.f, v);
  o[4] = dpp_f<0x154, 0xF>(0.f, v); o[5] = dpp_f<0x155, 0xF>(0.f, v); o[6] = dpp_f<0x156, 0xF>(0.f, v); o[7] = dpp_f<0x157, 0xF>(0.f, v);
}

// Attention of a group of query heads that read one K / V head, in every layer: part `part` of the ranges of their deal.  A column of
// the products is a (head, token).  What one of the eight wavefronts of the launch per phase takes of a range (32 positions, and every
// 256th after) is a sum of its own here too; those sums are dealt to the wavefronts and merged as there.  Where a group's ranges
// are spread over workgroups, each hands its ranges' records round, and a column is merged by one of them.
template <int M>
__device__ __forceinline__ void chain_attention(const ChainArgs& a, ChainAttnSmem& sm, const int group, const int part, const uint32_t halted) {
  const int total = a.pos0 + M, SL = a.split_len, n_r = a.n_splits;
  int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r0 = n_r * part / a.parts, r1 = n_r * (part + 1) / a.parts;
  const int rep = a.nq / a.nkv, per_kv = a.n_groups / a.nkv, kvh = group / per_kv, h_in = (group - kvh * per_kv) * a.heads;
  const int head0 = kvh * rep + h_in, n_col = min(a.heads, rep - h_in) * M;
  const int per = min(8, SL >> 5);                // sums of a whole range
  const int tail = min(per, (min(r1 * SL, total) - (r1 - 1) * SL + 31) >> 5), n_items = (r1 - 1 - r0) * per + tail;
  const int pt = a.page_tokens, pshift = __builtin_ctz(pt);             // pages of a power of two
  const uint32_t page_bytes = 256u * (uint32_t)(a.nkv * pt), k_off = 128u * (uint32_t)(kvh * pt), v_off = 128u * (uint32_t)((a.nkv + kvh) * pt);
  const int per_inv = (65536 + per - 1) / per;    // item / per = item per_inv >> 16 for the few items there are
  struct Cur { int item, base, s1, more; };       // a step of 32 positions, of a sum that has had steps (more) or not; s1 0: none
  auto open = [&](const int item) {
    Cur c{item, 0, 0, 0};
    if (item < n_items) {
      const int q = item * per_inv >> 16, r = r0 + q;
      c.base = r * SL + (item - q * per) * 32; c.s1 = min((r + 1) * SL, total);
    }
    return c;
  };
  auto next = [&](const Cur& c) { return c.item < n_items && c.base + 256 < c.s1 ? Cur{c.item, c.base + 256, c.s1, 1} : open(c.item + 8); };
  struct Raw { u32x4 k[2][2]; uint2 v[2][4]; } x0, x1;       // K rows of two 16-position tiles, V^T tiles of the same positions
  // Entries in front of the block (a position at or behind it reads the last one's, whatever the step: no branch around registers in flight).
  auto request = [&](Raw& x, const Cur& c, const int l) {
    const char* kv = reinterpret_cast<const char*>(a.kv_pages + (size_t)l * a.kv_layer_stride);
    const int j = lane & 15, g = lane >> 4, last = max(a.pos0 - 1, 0);
    int p[2], q[2];                               // a K row's position; the first of the four positions of a V^T piece
    uint32_t pp[2], qp[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      p[t] = min(c.base + 16 * t + j, last); q[t] = min(c.base + 16 * t + 4 * g, last & ~3);
      pp[t] = (uint32_t)p[t] >> pshift; qp[t] = (uint32_t)q[t] >> pshift;
    }
    if (a.page_table != nullptr) {
#pragma unroll
      for (int t = 0; t < 2; ++t) { pp[t] = (uint32_t)a.page_table[pp[t]]; qp[t] = (uint32_t)a.page_table[qp[t]]; }
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const uint32_t at = pp[t] * page_bytes + k_off + (uint32_t)(p[t] & (pt - 1)) * 128u + 16u * g;
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) x.k[t][ks] = *reinterpret_cast<const u32x4*>(kv + at + ks * 64);
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {                 // channel row = lane % 16 of each 16-channel tile, 4 consecutive positions
      const uint32_t at = qp[t] * page_bytes + v_off + 2u * (uint32_t)(j * pt + (q[t] & (pt - 1)));
#pragma unroll
      for (int ch = 0; ch < 4; ++ch) x.v[t][ch] = *reinterpret_cast<const uint2*>(kv + at + (uint32_t)(ch * pt) * 32u);
    }
  };
  const Cur c0 = open(w), c1 = next(c0);
  request(x0, c0, 0);
  request(x1, c1, 0);
  if (flag_set(halted)) return;
  for (int l = 0; l < a.n_layers; ++l) {
    chain_opaque(lane, w);
    const int j = lane & 15, g = lane >> 4;
    char* hand = a.hand + (size_t)l * a.layer_bytes;
    {
      // the group's queries (16 pieces a column, two columns a wavefront), and the block's own keys and values (16 pieces a token, the first wavefront's)
      ChainWait<1> wt;
      const int pc = lane & 15, col = 2 * w + (lane >> 4), kvm = (lane >> 4) - 2;
      const bool is_q = lane < 32 && col < n_col, is_kv = w == 0 && lane >= 32 && kvm < M;
      const uint32_t h_at = (uint32_t)(hand - reinterpret_cast<const char*>(a.q_last)), q_at = l + 1 == a.n_layers ? 0u : h_at + a.o_q;      // (the distance fits: launch_chain)
      wt.on[0] = is_q || is_kv;
      wt.base = reinterpret_cast<const char*>(a.q_last);
      wt.p[0] = (is_kv ? h_at + a.o_kv + (kvh * M + kvm) * 256u : q_at + ((min(col, n_col - 1) % M) * a.nq + head0 + min(col, n_col - 1) / M) * 256u) + pc * 16u;
      wt.run(a.abort_word, a.limit);
      if (is_q) {
        const HiLo s0 = split_bf16(__uint_as_float(wt.v[0][0]), __uint_as_float(wt.v[0][1])), s1 = split_bf16(__uint_as_float(wt.v[0][2]), __uint_as_float(wt.v[0][3]));
        reinterpret_cast<uint2*>(&sm.q[0][pc >> 3][((pc & 7) >> 1) * 16 + col])[pc & 1] = make_uint2(s0.hi, s1.hi);
        reinterpret_cast<uint2*>(&sm.q[1][pc >> 3][((pc & 7) >> 1) * 16 + col])[pc & 1] = make_uint2(s0.lo, s1.lo);
      }
      if (is_kv) reinterpret_cast<u32x4*>(&sm.kv[kvm][0][0])[pc] = wt.v[0];
      __syncthreads();
    }
    // AttnWave::step, in its order; what a sum has so far waits for its next step in LDS, not in registers that loads in flight need
    auto take = [&](Raw& x, const Cur& c) {
      if (c.base + 32 > a.pos0) {                 // the block's own entries come from the hand-off, not from the cache
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int mk = c.base + 16 * t + j - a.pos0;
          if (mk >= 0 && mk < M) {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) x.k[t][ks] = *reinterpret_cast<const u32x4*>(&sm.kv[mk][0][ks * 32 + 8 * g]);
          }
#pragma unroll
          for (int m = 0; m < M; ++m) {
            const int e = a.pos0 + m - (c.base + 16 * t + 4 * g);
            if (e >= 0 && e < 4) {
              const uint32_t keep = (e & 1) ? 0x0000FFFFu : 0xFFFF0000u;
#pragma unroll
              for (int ch = 0; ch < 4; ++ch) {
                const uint32_t nv = (uint32_t)sm.kv[m][1][ch * 16 + j] << (16 * (e & 1));
                if (e < 2) x.v[t][ch].x = (x.v[t][ch].x & keep) | nv;
                else x.v[t][ch].y = (x.v[t][ch].y & keep) | nv;
              }
            }
          }
        }
      }
      if (c.base + 32 > c.s1) {                   // beyond the range: zeros (0 * NaN would poison the sum)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const int p0 = c.base + 16 * t + 4 * g;
          const uint2 keep = make_uint2((p0 < c.s1 ? 0x0000FFFFu : 0u) | (p0 + 1 < c.s1 ? 0xFFFF0000u : 0u),
                                        (p0 + 2 < c.s1 ? 0x0000FFFFu : 0u) | (p0 + 3 < c.s1 ? 0xFFFF0000u : 0u));
#pragma unroll
          for (int i = 0; i < 4; ++i) { x.v[t][i].x &= keep.x; x.v[t][i].y &= keep.y; }
        }
      }
      f32x4 S[2];
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        S[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
          S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x.k[t][ks]), as_bf16x8(sm.q[0][ks][lane]), S[t], 0, 0, 0);
          S[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(x.k[t][ks]), as_bf16x8(sm.q[1][ks][lane]), S[t], 0, 0, 0);
        }
        S[t] *= a.scale;
      }
      if (c.base + 32 > min(c.s1, a.pos0 + 1)) {  // some column does not see all of it
        const int lim = min(c.s1 - 1, a.pos0 + (M == 1 ? 0 : j & 1));           // last position of the range that column j sees
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
          for (int v = 0; v < 4; ++v) S[t][v] = c.base + 16 * t + 4 * g + v <= lim ? S[t][v] : NEG_BIG;
      }
      float mx = fmaxf(fmaxf(fmaxf(S[0][0], S[0][1]), fmaxf(S[0][2], S[0][3])), fmaxf(fmaxf(S[1][0], S[1][1]), fmaxf(S[1][2], S[1][3])));
      mx = row4_max(mx);
      const int at = c.item * n_col + j;
      float m_run = NEG_BIG, l_run = 0.f;
      if (c.more && j < n_col) { m_run = sm.m[at]; l_run = sm.l[at]; }
      const float m_new = fmaxf(m_run, mx), alpha = __expf(m_run - m_new);
      float sum = 0.f;
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const float e = (S[t][v] > 0.5f * NEG_BIG) ? __expf(S[t][v] - m_new) : 0.f;
          S[t][v] = e;
          sum += e;
        }
      sum = row4_sum(sum);
      l_run = l_run * alpha + sum;
      f32x4 O[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        O[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (c.more && j < n_col) O[i] = *reinterpret_cast<const f32x4*>(&sm.o[at][i * 16 + 4 * g]) * alpha;
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        union { uint32_t u[2]; s16x4 v; } ph, pl;
#pragma unroll
        for (int v = 0; v < 2; ++v) { const HiLo y = split_bf16(S[t][2 * v], S[t][2 * v + 1]); ph.u[v] = y.hi; pl.u[v] = y.lo; }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          union { uint2 u; s16x4 v; } vv;
          vv.u = x.v[t][i];
          O[i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vv.v, ph.v, O[i], 0, 0, 0);
          O[i] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(vv.v, pl.v, O[i], 0, 0, 0);
        }
      }
      if (j < n_col) {
#pragma unroll
        for (int i = 0; i < 4; ++i) *reinterpret_cast<f32x4*>(&sm.o[at][i * 16 + 4 * g]) = O[i];
        if (g == 0) { sm.m[at] = m_new; sm.l[at] = l_run; }
      }
    };
    Cur ca = c0, cb = c1;
    while (ca.item < n_items) {
      take(x0, ca);
      ca = next(cb);
      if (ca.item < n_items) request(x0, ca, l);
      if (cb.item >= n_items) break;
      take(x1, cb);
      cb = next(ca);
      if (cb.item < n_items) request(x1, cb, l);
    }
    __syncthreads();
    // ranges: a row of 16 lanes (four channels each) per range and column; lane i of a row knows sum i, and hands it round
    chain_opaque(lane, w);
    const int c4 = (lane & 15) * 4, own = lane & 7;
    const bool plain = SL >= 256 && total <= ATTN_HEAD_MAX_CTX;      // (the order of a head in one workgroup)
    float* recs = reinterpret_cast<float*>(hand + a.o_rec) + (size_t)group * n_r * a.heads * M * CHAIN_REC;
    // (32 lanes where the record goes to another workgroup: the second row of lanes stores its maximum and sum with the same instruction)
    const int rows = a.parts == 1 ? 4 : 2;
    for (int rc = w * rows + (lane >> (a.parts == 1 ? 4 : 5)); rc < (r1 - r0) * n_col; rc += 8 * rows) {
      const int r = rc / n_col, col = rc - r * n_col, n = r0 + r == r1 - 1 ? tail : per;
      const float* o_r = &sm.o[r * per * n_col + col][c4];
      f32x4 piece[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        piece[i] = *reinterpret_cast<const f32x4*>(o_r + min(i, n - 1) * n_col * 64);
#pragma unroll
        for (int v = 0; v < 4; ++v) piece[i][v] = i < n ? piece[i][v] : 0.f;
      }
      const int at = (r * per + min(own, n - 1)) * n_col + col;
      const float mi = own < n ? sm.m[at] : NEG_BIG, li = own < n ? sm.l[at] : 0.f;
      float mm = fmaxf(mi, dpp_f<DPP_QUAD_XOR1, 0xF>(mi, mi));
      mm = fmaxf(mm, dpp_f<DPP_QUAD_XOR2, 0xF>(mm, mm));
      mm = fmaxf(mm, dpp_f<DPP_ROW_HALF_MIRROR, 0xF>(mm, mm));
      float f[8], ls[8], ll = 0.f;
      row_bcast8(expf(mi - mm), f);               // 0 past the range's sums
      row_bcast8(li, ls);
#pragma unroll
      for (int i = 0; i < 8; ++i) ll = fmaf(ls[i], f[i], ll);
      f32x4 o;
      if (plain) {
        o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
          for (int v = 0; v < 4; ++v) o[v] = fmaf(piece[i][v], f[i], o[v]);
      } else {
        o = range_sum<8>([&](int i) { return piece[i]; }, [&](int i) { return f[i]; });
      }
      if (a.parts == 1) {
        *reinterpret_cast<f32x4*>(&sm.ro[rc][c4]) = o;
        if (c4 == 0) { sm.rm[rc] = mm; sm.rl[rc] = ll; }
      } else {
        const bool second = (lane & 16) != 0;
        if (!second || c4 == 0)
          chain_put16(recs, (uint32_t)(((r0 + r) * n_col + col) * CHAIN_REC + (second ? 64 : c4)) * 4u,
                      second ? u32x4{__float_as_uint(mm), __float_as_uint(ll), 0u, 0u}
                             : u32x4{__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])});
      }
    }
    if (a.parts == 1) __syncthreads();
    // columns: a row of lanes each; column t is merged by the workgroup of part parts - 1 - t % parts
    const int col = a.parts - 1 - part + (w * 4 + (lane >> 4)) * a.parts;
    if (__ballot(col < n_col) != 0ull) {
      const bool on = col < n_col;
      const int cc = on ? col : 0;
      f32x4 ro[CHAIN_MAX_RANGES];
      float mi = NEG_BIG, li = 0.f;
      if (a.parts == 1) {
#pragma unroll
        for (int r = 0; r < CHAIN_MAX_RANGES; ++r) ro[r] = *reinterpret_cast<const f32x4*>(&sm.ro[min(r, n_r - 1) * n_col + cc][c4]);
        if (own < n_r) { mi = sm.rm[own * n_col + cc]; li = sm.rl[own * n_col + cc]; }
      } else {
        ChainWait<CHAIN_MAX_RANGES + 1> wt;
        wt.base = reinterpret_cast<const char*>(recs);
        const uint32_t rec = (uint32_t)(cc * CHAIN_REC * 4), next_range = (uint32_t)(n_col * CHAIN_REC * 4);
#pragma unroll
        for (int r = 0; r < CHAIN_MAX_RANGES; ++r) wt.p[r] = rec + (uint32_t)min(r, n_r - 1) * next_range + c4 * 4;
        wt.p[CHAIN_MAX_RANGES] = rec + (uint32_t)min(own, n_r - 1) * next_range + 256;
        wt.run(a.abort_word, a.limit);
#pragma unroll
        for (int r = 0; r < CHAIN_MAX_RANGES; ++r)
          ro[r] = f32x4{__uint_as_float(wt.v[r][0]), __uint_as_float(wt.v[r][1]), __uint_as_float(wt.v[r][2]), __uint_as_float(wt.v[r][3])};
        if (own < n_r) { mi = __uint_as_float(wt.v[CHAIN_MAX_RANGES][0]); li = __uint_as_float(wt.v[CHAIN_MAX_RANGES][1]); }
      }
      // lane i of a row: the running maximum in front of range i and with it
      float ms[8], ls[8], fo[8], fn[8], mx = NEG_BIG, before = NEG_BIG, with = NEG_BIG;
      row_bcast8(mi, ms);
      row_bcast8(li, ls);
#pragma unroll
      for (int r = 0; r < 8; ++r) {
        if (own == r) before = mx;
        mx = fmaxf(mx, ms[r]);
        if (own == r) with = mx;
      }
      row_bcast8(expf(before - with), fo);
      row_bcast8(expf(mi - with), fn);
      float Ls = 0.f, o[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < CHAIN_MAX_RANGES; ++r)
        if (r < n_r) {
          Ls = merged(Ls, fo[r], ls[r], fn[r]);
#pragma unroll
          for (int v = 0; v < 4; ++v) o[v] = merged(o[v], fo[r], ro[r][v], fn[r]);
        }
      const float inv = 1.0f / Ls;
      const HiLo s0 = split_product<RANGES_LO_EXACT>(o[0], inv, o[1], inv), s1 = split_product<RANGES_LO_EXACT>(o[2], inv, o[3], inv);
      // four lanes hold a block of 16 channels: lanes 0, 1 store its hi, lanes 2, 3 its lo, 16 bytes each, gathered from two lanes
      auto quad = [&](const uint32_t h, const uint32_t l) {
        const uint32_t h0 = (uint32_t)dpp_i<0x88, 0xF>(0, (int)h), l0 = (uint32_t)dpp_i<0x88, 0xF>(0, (int)l);       // lanes 0, 2, 0, 2 of the four
        return (lane & 2) ? l0 : h0;
      };
      auto quad1 = [&](const uint32_t h, const uint32_t l) {
        const uint32_t h1 = (uint32_t)dpp_i<0xDD, 0xF>(0, (int)h), l1 = (uint32_t)dpp_i<0xDD, 0xF>(0, (int)l);       // lanes 1, 3, 1, 3
        return (lane & 2) ? l1 : h1;
      };
      const u32x4 out = {quad(s0.hi, s0.lo), quad(s1.hi, s1.lo), quad1(s0.hi, s0.lo), quad1(s1.hi, s1.lo)};
      if (on) chain_put16(hand + a.o_xattn, (uint32_t)((((head0 + col / M) * 4 + ((lane & 15) >> 2)) * M + col % M) * 64 + (lane & 3) * 16), out);
    }
    if (l + 1 < a.n_layers) {                     // the next layer's entries arrive while its queries are being formed
      request(x0, c0, l + 1);
      request(x1, c1, l + 1);
    }
  }
}

template <int M, bool LN, int KPW, int NSEG>
__global__ __launch_bounds__(512, 4) void k_chain(ChainArgs a) {
  union Smem { ChainGemmSmem gemm; ChainAttnSmem attn; };
  __shared__ Smem sm;
  const uint32_t halted = gate_request(a.gate);
  const int id = blockIdx.x, n_attn = a.n_groups * a.parts;
  if (id < a.n_pu) chain_projections<M, LN, KPW>(a, sm.gemm, id, halted);
  else if (id < a.n_pu + n_attn) chain_attention<M>(a, sm.attn, (id - a.n_pu) % a.n_groups, (id - a.n_pu) / a.n_groups, halted);
  else chain_residual<M, LN, KPW, NSEG>(a, sm.gemm, id - a.n_pu - n_attn, halted);
}

// (plain 16-byte stores: the launch's end makes them visible)
__device__ __forceinline__ void chain_empty16(char* p, uint32_t at) { *reinterpret_cast<u32x4*>(p + at) = u32x4{CHAIN_EMPTY, CHAIN_EMPTY, CHAIN_EMPTY, CHAIN_EMPTY}; }
struct ChainBegin {
  const float* g; float* h; int64_t tok_stride; int pos0, vocab, max_pos;
  uint32_t fill_from, fill, fill_q;    // empty words: from byte fill_from behind the first input panel, 16-byte pieces there and in the last layer's queries
};
// In front of k_chain: the embedding rows with the first layer's input (one workgroup per token, the arithmetic of norm_row), and empty
// words into everything that k_chain hands over.
__global__ __launch_bounds__(256) void k_chain_begin(const int32_t* tokens, const bf16_t* tok_emb, const bf16_t* pos_emb, const uint32_t* gate, char* xn, float* q_last,
                                                     int d, int M, ChainBegin n) {
  __shared__ float red[5];
  const uint32_t halted = gate_request(gate);
  const int t = threadIdx.x;
  if ((int)blockIdx.x >= M) {
    if (flag_set(halted)) return;
    const uint32_t i = (blockIdx.x - M) * 256u + t;              // 16 bytes a thread
    if (i < n.fill + n.fill_q)
      chain_empty16(i < n.fill ? xn + n.fill_from : reinterpret_cast<char*>(q_last), (i < n.fill ? i : i - n.fill) * 16u);
    return;
  }
  const int m = blockIdx.x, k = t * 4;
  int tok = tokens[m];
  tok = tok < 0 ? 0 : (tok >= n.vocab ? n.vocab - 1 : tok);
  int pos = n.pos0 + m;
  if (pos >= n.max_pos) pos = n.max_pos - 1;
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f), gn = v;
  if (k < d) {
    const uint2 u = *reinterpret_cast<const uint2*>(tok_emb + (size_t)tok * n.tok_stride + k);
    gn = *reinterpret_cast<const float4*>(n.g + k);
    v = make_float4(bf16_to_f32(u.x & 0xFFFF), bf16_to_f32(u.x >> 16), bf16_to_f32(u.y & 0xFFFF), bf16_to_f32(u.y >> 16));
    if (pos_emb) {
      const uint2 p = *reinterpret_cast<const uint2*>(pos_emb + (size_t)pos * d + k);
      v.x += bf16_to_f32(p.x & 0xFFFF); v.y += bf16_to_f32(p.x >> 16);
      v.z += bf16_to_f32(p.y & 0xFFFF); v.w += bf16_to_f32(p.y >> 16);
    }
  }
  if (flag_set(halted)) return;
  if (k < d) {
    *reinterpret_cast<float4*>(n.h + (size_t)m * d + k) = v;
    const HiLo x0 = split_product<true>(v.x, gn.x, v.y, gn.y), x1 = split_product<true>(v.z, gn.z, v.w, gn.w);
    char* blk = xn + ((k >> 4) * M + m) * chain_block_bytes<true>() + (k & 12) * 2;
    chain_put2(blk, x0.hi, x1.hi);
    chain_put2(blk + 32, x0.lo, x1.lo);
  }
  const float ss = block_sum<256>((v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w), red);
  const float sx = block_sum<256>((v.x + v.y) + (v.z + v.w), red);
  if (t < d / 16) {
    char* stats = xn + (t * M + m) * chain_block_bytes<true>() + 64;
    chain_put2(stats, t == 0 ? __float_as_uint(ss) : 0u, t == 0 ? __float_as_uint(sx) : 0u);
    chain_put2(stats + 8, 0u, 0u);
  }
}

// The instance for a model and a block: f<M, LN, KPW, NSEG>.
#define CHAIN_BY_SHAPE(f, M, ln, kpw, ...) \
  ((M) == 1 ? ((ln) ? ((kpw) == 3 ? f<1, true, 3, 4>(__VA_ARGS__) : f<1, true, 4, 3>(__VA_ARGS__)) \
                    : ((kpw) == 3 ? f<1, false, 3, 4>(__VA_ARGS__) : f<1, false, 4, 3>(__VA_ARGS__))) \
            : ((ln) ? ((kpw) == 3 ? f<2, true, 3, 4>(__VA_ARGS__) : f<2, true, 4, 3>(__VA_ARGS__)) \
                    : ((kpw) == 3 ? f<2, false, 3, 4>(__VA_ARGS__) : f<2, false, 4, 3>(__VA_ARGS__))))
template <int M, bool LN, int KPW, int NSEG>
static long chain_capacity() {
  static const long c = resident_capacity(reinterpret_cast<const void*>(k_chain<M, LN, KPW, NSEG>));
  return c;
}
template <int M, bool LN, int KPW, int NSEG>
static hipError_t chain_start(const ChainArgs& a, hipStream_t s) {
  hipLaunchKernelGGL((k_chain<M, LN, KPW, NSEG>), dim3((unsigned)a.wgs), dim3(512), 0, s, a);
  return hipGetLastError();
}

// Whether a forward of M tokens behind pos0 positions takes k_chain, and how.  Heads of 64 channels in a model of at most 1024 columns whose layers fit the
// kernel's registers: k-tiles of a wavefront per matrix (three, or four with fewer K ranges of the MLP output).  `room`: bytes at a.hand.
bool chain_plan(ChainArgs& a, int d_qkv, int dh, bool layernorm, size_t room, long capacity) {
  const int d = a.d, d_q = a.nq * 64, KTF = a.d_ff >> 5, total = a.pos0 + a.M;
  if (a.kv_layer_stride >= (size_t)1 << 30 || (a.page_tokens & (a.page_tokens - 1)) != 0) return false;      // 32-bit offsets into a layer's cache, shifts
  if (dh != 64 || a.M > CHAIN_MAX_TOKENS || a.n_layers > CHAIN_MAX_LAYERS || d > 1024 || d_q > 1024 || d_qkv != (a.nq + 2 * a.nkv) * 64) return false;
  a.n_seg = gemm_split_for(d, KTF, a.M);
  const int wide = d > d_q ? d : d_q, per_seg = (KTF + a.n_seg - 1) / a.n_seg;
  const int kpw = (wide > 768 || per_seg > 24) ? 4 : 3;
  if (per_seg > 8 * kpw || a.n_seg > (kpw == 3 ? 4 : 3)) return false;
  if (gemm_split_for(d, d_q >> 5, a.M) != 1) return false;
  long cap_shared = capacity, cap_own = capacity;
  const int rt = qkv_attn_rt(d_qkv);
  if (rt != 2) return false;
  if (capacity == 0) qkv_attn_capacities(a.M, rt, dh, layernorm, &cap_shared, &cap_own);
  const QkvAttnPlan p = qkv_attn_plan(d_qkv, a.nq, a.nkv, dh, layernorm, total, rt, cap_shared, cap_own);
  if (p.form != 2 || p.n_splits > CHAIN_MAX_RANGES) return false;
  a.split_len = p.split_len; a.n_splits = p.n_splits;
  // The heads of a K / V head share its keys and values as columns of the same products, as far as sixteen columns go; a group's ranges go to
  // as many workgroups as make up 24, or 36 where the launch keeps within CHAIN_MAX_WGS: a step of 32 positions costs a wavefront about half a
  // microsecond.  68M-class token, 24 / 36 / 48: at 523 positions 49.8 / 48.5 / 48.7 us, at 1024 50.5 / 49.5 / 49.4, at 2048 58.4 / 54.1 / 54.0.
  // Thirteen groups and more have two of the 36: there, and where ranges are long, a workgroup gets two ranges at most (from 512 positions on
  // one) as far as there is room.  One layer of 16 heads of their own, 128 columns, 3071 positions, two tokens: a launch per phase 26.6 us, two workgroups a
  // group 29.1, now 24.9; six LayerNorm layers at 2400, one token: 136.6, 124.9, 93.5.  Over 1224 models and blocks that take it (64 to 1024 columns,
  // 1 to 16 heads, 1 to 6 layers, 20 to 3071 positions) this launch is 1.03 (one layer of 16 heads at 3071) to 1.7 times as fast as a launch per phase,
  // 1.34 at the median.
  const int rep = a.nq / a.nkv, per_kv = (rep * a.M + 15) / 16;
  a.heads = (rep + per_kv - 1) / per_kv;
  a.n_groups = a.nkv * per_kv;
  const int n_p = d_qkv / 32, n_u = a.d_ff / 32;
  a.n_pu = n_p > n_u ? n_p : n_u;
  const int room_for = (CHAIN_MAX_WGS - a.n_pu - d / 16) / a.n_groups, few = 24 / a.n_groups < 1 ? 1 : 24 / a.n_groups;
  const int two = a.split_len < 512 ? 2 : 1, want = 36 / a.n_groups > (a.n_splits + two - 1) / two ? 36 / a.n_groups : (a.n_splits + two - 1) / two;
  a.parts = want < room_for ? want : room_for;
  if (a.parts < few) a.parts = few;
  if (a.parts > a.n_splits) a.parts = a.n_splits;
  const int most = (a.n_splits + a.parts - 1) / a.parts;          // ranges of a workgroup
  const int part_len = a.split_len / 32 < 8 ? a.split_len / 32 : 8;
  if (most * part_len * a.heads * a.M > CHAIN_PARTS || most * a.heads * a.M > 32) return false;
  a.kpw = kpw;
  a.wgs = a.n_pu + a.n_groups * a.parts + d / 16;
  if (a.wgs > CHAIN_MAX_WGS || a.wgs > (capacity != 0 ? capacity : CHAIN_BY_SHAPE(chain_capacity, a.M, layernorm, kpw))) return false;
  // the hand-off buffers of a layer, each on a line of its own
  size_t off = 0;
  auto take = [&](size_t bytes) { const size_t o = off; off += (bytes + 127) / 128 * 128; return (unsigned)o; };
  const size_t M = (size_t)a.M;
  a.o_xn = take(M * 8 * d);
  a.o_q = take(M * 4 * d_q); a.o_kv = take(M * 256 * a.nkv); a.o_xattn = take(M * 4 * d_q); a.o_xn2 = take(M * 8 * d);
  a.o_act = take(M * 4 * a.d_ff);
  a.o_rec = take(a.parts > 1 ? M * 4 * CHAIN_REC * a.n_splits * a.heads * a.n_groups : 0);
  a.layer_bytes = off;
  return off * (size_t)a.n_layers <= room;
}

hipError_t launch_chain(const NormArgs& n, const ChainArgs& a, bool layernorm, hipStream_t s) {
  if (n.tokens == nullptr || n.M != a.M || n.d != a.d || a.hand == nullptr || a.q_last == nullptr) return hipErrorInvalidValue;
  if (a.hand < reinterpret_cast<const char*>(a.q_last) || (size_t)(a.hand - reinterpret_cast<const char*>(a.q_last)) + a.layer_bytes * a.n_layers >= (size_t)1 << 32)
    return hipErrorInvalidValue;                  // 32-bit offsets
  const ChainBegin b{n.g, n.h, n.tok_stride, n.pos0, n.vocab, n.max_pos, a.o_q - a.o_xn, (uint32_t)((a.layer_bytes * a.n_layers - a.o_q) / 16), (uint32_t)(a.M * a.nq * 16)};
  hipLaunchKernelGGL(k_chain_begin, dim3((unsigned)a.M + (b.fill + b.fill_q + 255) / 256), dim3(256), 0, s, n.tokens, n.tok_emb, n.pos_emb, n.gate, a.hand + a.o_xn, a.q_last,
                     n.d, a.M, b);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return CHAIN_BY_SHAPE(chain_start, a.M, layernorm, a.kpw, a, s);
}

// ---------------------------------------------------------------------------------------------
// one launch per forward or per draft loop: persistent workgroups, phases separated by a grid barrier
// ---------------------------------------------------------------------------------------------
//
// A forward of the RMSNorm / rotary / SwiGLU family is a chain of phases (per layer: QKV projection, attention,
// O-projection, gate/up, down; then the LM head), each of which needs everything the phase before it wrote.
// Launched one kernel per phase, every boundary costs a ramp (first weight bytes arrive 2 - 3 us after the
// launch) on top of the phase's own tail.  Here one cooperative launch of one workgroup per compute unit runs
// all phases; a workgroup's share of a phase is fixed by its index, so at the end of a phase it knows which
// weight tiles it will need first in the next one and requests them BEFORE it waits at the grid barrier: the
// weight stream of phase i + 1 is in flight while phase i drains and the barrier's round trips pass.
//
// Coherence inside the launch: the eight XCDs have separate L2s, and an L2-wide write-back / invalidate at
// every barrier costs more than the barrier (measured: 8 - 13 us).  Instead (a) every store that another
// workgroup will read is a write-through store and small hand-off data is read with L2-bypassing loads
// (COH accesses above); (b) what MANY workgroups of a phase read (the activation panels with their sums of
// squares, the queries) is given a fresh address per phase ("versions"), so no L2 can hold an older copy
// and plain loads are safe and hit in the reader's own L2 after the first touch: L2-bypassing loads of the
// same few lines from every workgroup queue up on a few memory channels.
//
// Grid barrier, two levels: workgroup i adds 1 to the counter of its group i % 16; the workgroup that completes
// a group adds 1 to the top counter; the one that completes the top counter writes the barrier's number into
// the 16 release words, and every workgroup polls only the release word of its own group (16 pollers per
// word: with every workgroup polling every counter, the polls of 256 workgroups queue up on a few memory
// channels and the workgroups leave the barrier microseconds apart).  All words are 256 bytes apart.  The
// host zeroes them before the launch.  Every wait is bounded: after BAR_SPIN_LIMIT polls the workgroup
// sets the abort word, every later barrier falls through at once, and the launch drains with unusable
// results (the arg-max and loop-finish kernels turn a set abort word into -1 outputs).

constexpr int BAR_GROUPS = 16;
constexpr int BAR_SLOT = 64;                 // ints between two words (256 bytes)
constexpr int BAR_TOP = BAR_GROUPS;          // word index (in slots) of the top counter
constexpr int BAR_RELEASE = BAR_GROUPS + 1;  // first release word
constexpr int BAR_ABORT = 2 * BAR_GROUPS + 1;
constexpr int BAR_SPIN_LIMIT = 1 << 20;      // polls (each a memory round trip, about 1 us) before giving up

// n = number of this barrier (1, 2, ..), per_group = workgroups per group
__device__ __forceinline__ void bar_arrive(unsigned* bar, const unsigned n, const unsigned per_group) {
  __builtin_amdgcn_s_waitcnt(0);             // this wavefront's hand-off stores have completed
  __builtin_amdgcn_s_barrier();              // ... and those of the whole workgroup
  if (threadIdx.x == 0) {
    const unsigned old = __hip_atomic_fetch_add(bar + (blockIdx.x % BAR_GROUPS) * BAR_SLOT, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (old + 1 == n * per_group) {
      const unsigned old_top = __hip_atomic_fetch_add(bar + BAR_TOP * BAR_SLOT, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (old_top + 1 == n * BAR_GROUPS) {
#pragma unroll
        for (int g = 0; g < BAR_GROUPS; ++g)
          __hip_atomic_store(bar + (BAR_RELEASE + g) * BAR_SLOT, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  asm volatile("" ::: "memory");
}

__device__ __forceinline__ void bar_wait(unsigned* bar, const unsigned n) {
  if (threadIdx.x == 0) {
    unsigned* rel = bar + (BAR_RELEASE + blockIdx.x % BAR_GROUPS) * BAR_SLOT;
    unsigned* abort_word = bar + BAR_ABORT * BAR_SLOT;
    int spins = 0;
    while ((int)(__hip_atomic_load(rel, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) - n) < 0) {
      ++spins;
      if ((spins & 255) == 0 && __hip_atomic_load(abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) break;
      if (spins > BAR_SPIN_LIMIT) {
        __hip_atomic_store(abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Row tiles per work unit of the four GEMM kinds, by model class (chosen so that a phase has about one unit
// per compute unit): wide models and narrow ones.
struct FwdBig { static constexpr int QKV = 4, PART = 4, UP = 8, LM = 8; };
struct FwdSmall { static constexpr int QKV = 2, PART = 1, UP = 2, LM = 8; };

// LDS of the persistent kernel: one arena, every phase lays its own structure over it (the phases are
// separate functions, so that each gets its own register allocation).
constexpr int FWD_SMEM_BYTES = 68 * 1024;
__shared__ __align__(16) unsigned char g_fwd_smem[FWD_SMEM_BYTES];
template <typename T> __device__ __forceinline__ T& fwd_smem() {
  static_assert(sizeof(T) <= FWD_SMEM_BYTES, "phase structure larger than the arena");
  return *reinterpret_cast<T*>(g_fwd_smem);
}

// The launch's arguments stay in the kernel-argument segment; the phase functions read them through this
// pointer (scalar loads).
typedef const FwdArgs __attribute__((address_space(4)))* FwdArgsPtr;

// What a phase function needs beyond the launch's arguments.
struct FwdCtx { FwdArgsPtr f; int step, l, M, pos0; unsigned bar_n; };   // bar_n: number of the barrier that ends the phase before (0: none)

struct FwdWaitHook {
  unsigned* bar; unsigned n;
  __device__ __forceinline__ void operator()() const { if (n != 0u) bar_wait(bar, n); }
};

__device__ __forceinline__ GemmArgs fwd_base_args(FwdArgsPtr f, const int M) {
  GemmArgs g{};
  g.M = M; g.n_split = 1; g.grp = 1; g.planes = f->planes; g.counters = f->gemm_counters; g.only_row = -1;
  return g;
}
// the sums of squares of a panel version follow its two panels
__device__ __forceinline__ float* fwd_ssq_of(FwdArgsPtr f, const bf16_t* xn_version) {
  return reinterpret_cast<float*>(const_cast<bf16_t*>(xn_version) + (size_t)32 * f->d);
}
__device__ __forceinline__ void fwd_normed_input(FwdArgsPtr f, GemmArgs& g, const bf16_t* x) {
  g.X = x; g.KT = f->d >> 5; g.ssq = fwd_ssq_of(f, x); g.n_ssq = f->d >> 4; g.d_in = f->d; g.eps = f->eps;
}
__device__ __forceinline__ void fwd_residual(FwdArgsPtr f, GemmArgs& g, const bf16_t* w, const bf16_t* x, const int k, const int split,
                                             const float* next_gain, bf16_t* xout) {
  g.W = w; g.X = x; g.KT = k >> 5; g.n_rows = f->d; g.h = f->h; g.ld_out = f->d; g.n_split = split;
  g.Xout = xout; g.KT_out = f->d >> 5; g.gain = next_gain; g.ssq_out = fwd_ssq_of(f, xout); g.n_ssq_out = f->d >> 4;
}
// panel versions of a step: xn has 2 L + 1 per step, xattn and xact L each
__device__ __forceinline__ bf16_t* fwd_xn(FwdArgsPtr f, const int step, const int v) {
  return f->xn + ((size_t)step * (2 * f->n_layers + 1) + v) * f->xn_stride;
}
__device__ __forceinline__ float* fwd_q(FwdArgsPtr f, const int step, const int l) {
  return f->q + ((size_t)step * f->n_layers + l) * 16 * f->d_q;
}
__device__ __forceinline__ bf16_t* fwd_xattn(FwdArgsPtr f, const int step, const int l) {
  return f->xattn + ((size_t)step * f->n_layers + l) * f->xattn_stride;
}
__device__ __forceinline__ bf16_t* fwd_xact(FwdArgsPtr f, const int step, const int l) {
  return f->xact + ((size_t)step * f->n_layers + l) * f->xact_stride;
}

// One GEMM phase: unit u = (row group u % groups, K range u / groups); workgroup i takes units i, i + G, ...
// Its first unit waits for the phase before (after requesting its first weight tiles); a workgroup without a
// unit just waits.  Ends with the arrival at the phase's own barrier.
template <int P, int RT, int EPI>
__device__ __forceinline__ void fwd_gemm_phase(const FwdCtx& c, const GemmArgs& ga, const int groups) {
  GemmSmem<RT, 8>& sm = fwd_smem<GemmSmem<RT, 8>>();
  const FwdWaitHook hook{c.f->bar, c.bar_n};
  const int n_units = groups * ga.n_split;
  int u = blockIdx.x;
  if (u >= n_units) {
    hook();
  } else {
    bool first = true;
    for (; u < n_units; u += gridDim.x) {
      const int b = u % groups, seg = u / groups;
      const int kt_begin = (int)((int64_t)ga.KT * seg / ga.n_split), kt_end = (int)((int64_t)ga.KT * (seg + 1) / ga.n_split);
      // (inside one launch the buffers filled before the barrier are the only prefetch across it: deeper buffers than the
      //  per-phase launches take with two panels)
      constexpr int U = RT >= 8 ? (P >= 2 ? 2 : 3) : 4;
      if (first) gemm_unit<P, RT, EPI, 8, U, true, FwdWaitHook>(ga, b, kt_begin, kt_end, seg, ga.n_split, sm, hook);
      else gemm_unit<P, RT, EPI, 8, U, true, FwdWaitHook>(ga, b, kt_begin, kt_end, seg, ga.n_split, sm, FwdWaitHook{nullptr, 0u});
      first = false;
    }
  }
  bar_arrive(c.f->bar, c.bar_n + 1, gridDim.x / BAR_GROUPS);
}

#define FWD_PHASE_FN __forceinline__

template <int P, typename C>
__device__ FWD_PHASE_FN void fwd_qkv(const FwdCtx c) {
  FwdArgsPtr f = c.f;
  GemmArgs g = fwd_base_args(f, c.M);
  g.W = f->layers[c.l].wqkv; fwd_normed_input(f, g, fwd_xn(f, c.step, 2 * c.l)); g.n_rows = f->d_qkv;
  g.grp = f->dh >> 5; g.q = fwd_q(f, c.step, c.l); g.ldq = f->d_q; g.nq = f->nq; g.nkv = f->nkv; g.dh = f->dh; g.pos0 = c.pos0;
  g.rope_tab = f->rope; g.kv_layer = f->kv_pages + (size_t)c.l * f->kv_layer_stride; g.page_table = f->page_table;
  g.page_tokens = f->page_tokens;
  fwd_gemm_phase<P, C::QKV, EPI_QKV>(c, g, f->d_qkv / (16 * C::QKV));
}

template <bool LOOP>
__device__ FWD_PHASE_FN void fwd_attn(const FwdCtx c) {
  FwdArgsPtr f = c.f;
  AttnArgs at{};
  at.q = fwd_q(f, c.step, c.l); at.ldq = f->d_q; at.kv_layer = f->kv_pages + (size_t)c.l * f->kv_layer_stride; at.page_table = f->page_table;
  at.page_tokens = f->page_tokens; at.nq = f->nq; at.nkv = f->nkv; at.dh = f->dh; at.M = c.M; at.pos0 = c.pos0;
  at.scale = f->attn_scale; at.part = f->part; at.split_len = f->attn_split_len;
  at.n_splits = (c.pos0 + c.M + f->attn_split_len - 1) / f->attn_split_len;
  at.Xout = fwd_xattn(f, c.step, c.l); at.counters = f->attn_counters;
  FwdWaitHook{f->bar, c.bar_n}();
  const int n_units = f->nq * at.n_splits;
  for (int u = blockIdx.x; u < n_units; u += gridDim.x) {
    const int head = u % f->nq, split = u / f->nq;
    if (f->dh == 128) attn_range<128, 8, true, LOOP>(at, head, split, fwd_smem<AttnSmem<128, 8>>(), 0u);
    else attn_range<64, 8, true, LOOP>(at, head, split, fwd_smem<AttnSmem<64, 8>>(), 0u);
  }
  bar_arrive(f->bar, c.bar_n + 1, gridDim.x / BAR_GROUPS);
}

template <int P, typename C>
__device__ FWD_PHASE_FN void fwd_o(const FwdCtx c) {
  FwdArgsPtr f = c.f;
  GemmArgs g = fwd_base_args(f, c.M);
  fwd_residual(f, g, f->layers[c.l].wo, fwd_xattn(f, c.step, c.l), f->d_q, f->split_o, f->layers[c.l].norm2_g,
               fwd_xn(f, c.step, 2 * c.l + 1));
  fwd_gemm_phase<P, C::PART, EPI_PARTIAL>(c, g, f->d / (16 * C::PART));
}

template <int P, typename C>
__device__ FWD_PHASE_FN void fwd_up(const FwdCtx c) {
  FwdArgsPtr f = c.f;
  GemmArgs g = fwd_base_args(f, c.M);
  g.W = f->layers[c.l].w_in; fwd_normed_input(f, g, fwd_xn(f, c.step, 2 * c.l + 1)); g.n_rows = 2 * f->d_ff;
  g.Xout = fwd_xact(f, c.step, c.l); g.KT_out = f->d_ff >> 5;
  fwd_gemm_phase<P, C::UP, EPI_SWIGLU>(c, g, 2 * f->d_ff / (16 * C::UP));
}

template <int P, typename C>
__device__ FWD_PHASE_FN void fwd_down(const FwdCtx c) {
  FwdArgsPtr f = c.f;
  GemmArgs g = fwd_base_args(f, c.M);
  const bool last = (c.l + 1 == f->n_layers);
  fwd_residual(f, g, f->layers[c.l].w_out, fwd_xact(f, c.step, c.l), f->d_ff, f->split_dn,
               last ? f->normf_g : f->layers[last ? c.l : c.l + 1].norm1_g, fwd_xn(f, c.step, 2 * c.l + 2));
  fwd_gemm_phase<P, C::PART, EPI_PARTIAL>(c, g, f->d / (16 * C::PART));
}

template <int P, typename C>
__device__ FWD_PHASE_FN void fwd_lm(const FwdCtx c) {
  FwdArgsPtr f = c.f;
  GemmArgs g = fwd_base_args(f, c.M);
  g.W = f->wlm; fwd_normed_input(f, g, fwd_xn(f, c.step, 2 * f->n_layers)); g.n_rows = f->vocab;
  g.out = f->logits; g.ld_out = f->vocab; g.only_row = f->only_last ? c.M - 1 : -1;
  fwd_gemm_phase<P, C::LM, EPI_STORE>(c, g, f->vocab / (16 * C::LM));
}

// Draft loop: Eq. 2 features and classifier on the step's logits; the workgroup that finishes them embeds the
// next step's token (row 0 of the residual stream, the first panel version of that step, the sums of squares).
__device__ FWD_PHASE_FN void fwd_classify(const FwdCtx c) {
  FwdArgsPtr f = c.f;
  FwdWaitHook{f->bar, c.bar_n}();
  ClassifyArgs ca{};
  ca.logits = f->clf.logits; ca.vocab = f->clf.vocab; ca.clf_params = f->clf.clf_params; ca.hidden = f->clf.hidden;
  ca.tau = f->clf.tau; ca.token_next = f->clf.token_next; ca.gate = f->clf.gate; ca.sl_count = f->clf.sl_count;
  ca.ppl_threshold = f->clf.ppl_threshold; ca.scratch = f->clf.scratch;
  ca.pos_feature = f->clf.pos_feature + (float)c.step;
  ca.force_halt = (c.step + 1 == f->n_steps && !f->open_end) ? 1 : 0;
  ca.out = reinterpret_cast<ClfOut*>(f->clf.out) + c.step;
  ca.block_slot = f->clf.block_slot + c.step;
  ca.force_token = f->clf.force_token ? f->clf.force_token + c.step : nullptr;
  ca.ref_token = f->clf.ref_token ? f->clf.ref_token + c.step : nullptr;
  const int nb = (f->vocab + 4 * CM_NT - 1) / (4 * CM_NT);
  if ((int)blockIdx.x < nb) {
    const int tok = classify_unit<CM_NT>(ca, blockIdx.x, nb, 0u);
    if (tok >= 0 && c.step + 1 < f->n_steps) {
      NormArgs na{};
      na.h = f->h; na.d = f->d; na.M = 1; na.layernorm = 0; na.eps = f->eps; na.g = f->layers[0].norm1_g;
      na.Xout = fwd_xn(f, c.step + 1, 0);
      na.ssq_out = fwd_ssq_of(f, na.Xout); na.n_ssq_out = f->d >> 4; na.tok_emb = f->tok_emb; na.tok_stride = f->tok_stride;
      na.vocab = f->vocab; na.max_pos = 1 << 30;
      __syncthreads();
      norm_row<CM_NT, true>(na, 0, tok, reinterpret_cast<float*>(g_fwd_smem), 0u);
    }
  }
  bar_arrive(f->bar, c.bar_n + 1, gridDim.x / BAR_GROUPS);
}

template <int P, typename C, bool LOOP>
__global__ __launch_bounds__(512) void k_forward(FwdArgs f_by_value) {
  (void)f_by_value;                           // read through the kernel-argument segment (first argument, offset 0)
  FwdArgsPtr f = (FwdArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  unsigned epoch = 0;                         // barriers this workgroup has arrived at
  const int n_steps = LOOP ? f->n_steps : 1, n_layers = f->n_layers;
  for (int step = 0; step < n_steps; ++step) {
    FwdCtx c;
    c.f = f; c.step = step;
    c.M = (LOOP && step > 0) ? 1 : f->M;
    c.pos0 = (LOOP && step > 0) ? f->pos0 + f->M + (step - 1) : f->pos0;
    for (int l = 0; l < n_layers; ++l) {
      c.l = l;
      c.bar_n = epoch++; fwd_qkv<P, C>(c);
      c.bar_n = epoch++; fwd_attn<LOOP>(c);
      c.bar_n = epoch++; fwd_o<P, C>(c);
      c.bar_n = epoch++; fwd_up<P, C>(c);
      c.bar_n = epoch++; fwd_down<P, C>(c);
    }
    c.l = 0;
    c.bar_n = epoch++; fwd_lm<P, C>(c);
    if (!LOOP) break;
    c.bar_n = epoch++; fwd_classify(c);
    // every workgroup learns the verdict of the step (the wait also orders the next step behind the embedding)
    bar_wait(f->bar, epoch);
    if (__hip_atomic_load(f->clf.gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) break;
  }
}

// Workgroups of the persistent launch: one per compute unit, a multiple of the barrier's counter count; 0 if
// the device cannot hold them all at once (then there is no persistent launch).
template <typename K>
static int forward_grid_for(K kernel) {
  int dev = 0, cus = 0, per_cu = 0, coop = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev) != hipSuccess || !coop) return 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 512, 0) != hipSuccess || per_cu < 1) return 0;
  return cus / BAR_GROUPS * BAR_GROUPS;
}

template <int P, typename C, bool LOOP>
static hipError_t launch_forward_cfg(const FwdArgs& f0, hipStream_t s) {
  static int grid = -1;                        // per process: the library serves the devices of one kind
  if (grid < 0) grid = forward_grid_for(k_forward<P, C, LOOP>);
  if (grid < BAR_GROUPS) return hipErrorCooperativeLaunchTooLarge;
  FwdArgs f = f0;
  // K ranges of the two residual-update GEMMs: about one work unit per workgroup, at least one k-tile per wavefront
  auto split_for = [&](int k) {
    const int groups = f.d / (16 * C::PART), kt = k >> 5;
    int sp = grid / groups;
    if (sp > kt / 8) sp = kt / 8;
    return sp < 1 ? 1 : (sp > GEMM_MAX_SPLIT ? GEMM_MAX_SPLIT : sp);
  };
  f.split_o = split_for(f.d_q);
  f.split_dn = split_for(f.d_ff);
  // attention ranges: about one (head, range) unit per workgroup, never shorter than the records were sized for
  const int total = f.pos0 + f.M + (LOOP ? f.n_steps - 1 : 0);
  const int target = grid / f.nq < 1 ? 1 : grid / f.nq;
  int len = ((total + target - 1) / target + 31) / 32 * 32;
  f.attn_split_len = len < ATTN_SPLIT_LEN ? ATTN_SPLIT_LEN : len;
  void* params[] = {&f};
  return hipLaunchCooperativeKernel(reinterpret_cast<void*>(k_forward<P, C, LOOP>), dim3(grid), dim3(512), params, 0, s);
}

bool forward_shape_ok(int d, int d_q, int d_qkv, int d_ff, int dh, int vocab, bool big) {
  const int rq = big ? FwdBig::QKV : FwdSmall::QKV, rp = big ? FwdBig::PART : FwdSmall::PART, ru = big ? FwdBig::UP : FwdSmall::UP;
  if (d % (16 * rp) || d_qkv % (16 * rq) || (2 * d_ff) % (16 * ru) || vocab % 128) return false;
  if (d % 32 || d_q % 32 || d_ff % 32) return false;
  if (dh != 64 && dh != 128) return false;
  return true;
}

hipError_t launch_forward(const FwdArgs& f, bool big, bool loop, hipStream_t s) {
  if (f.M < 1 || f.M > 16 || !forward_shape_ok(f.d, f.d_q, f.d_qkv, f.d_ff, f.dh, f.vocab, big)) return hipErrorInvalidValue;
  if (f.layers == nullptr || f.bar == nullptr) return hipErrorInvalidValue;
  if (loop) {
    if (f.M > 8 || f.n_steps < 1 || f.d > 4096 || f.clf.scratch == nullptr || f.clf.gate == nullptr) return hipErrorInvalidValue;
    return big ? launch_forward_cfg<1, FwdBig, true>(f, s) : launch_forward_cfg<1, FwdSmall, true>(f, s);
  }
  if (f.M <= 8) return big ? launch_forward_cfg<1, FwdBig, false>(f, s) : launch_forward_cfg<1, FwdSmall, false>(f, s);
  return big ? launch_forward_cfg<2, FwdBig, false>(f, s) : launch_forward_cfg<2, FwdSmall, false>(f, s);
}

}  // namespace disco
