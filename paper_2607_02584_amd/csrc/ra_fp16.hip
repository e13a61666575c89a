// ra_fp16.hip -- BF16/FP16 fallback attention for gfx950 (the 16-bit path the
// paper keeps for accuracy-sensitive DiT blocks and denoising steps).
//
// Producer: plain 3D RoPE (Sec. 3) of Q and K in binary32, rounded to the
// 16-bit input type, written in a tiled layout that makes every 32-token chunk
// a ready matrix-core operand; V is re-laid out the same way, transposed.
//
// Attention: S^T = K Q^T on v_mfma_f32_32x32x16_{bf16,f16} (fp32 accumulate),
// blockwise online softmax over blocks of kv_block (64 or 128) keys in
// ascending order,
//   m = max(m, rowmax(S * Kc)),  P = 2^(S*Kc - m),  l = alpha*l + sum P,
// P rounded to the 16-bit type as the A operand of O += P V, and O = O / l.
// Each lane holds the scores of one query, so row reductions stay inside the
// lane plus one exchange between the two wave halves.
//
// 16-bit tiled layouts (elements), token n = 32*c + r:
//   Q, K: (((c*8 + ch/16)*2 + (ch/8)%2)*32 + r)*8 + ch%8
//   V:    (((c*2 + s)*2 + h)*128 + ch)*8 + e  holds V[32c + 16s + 8(e/4) + 4h + e%4][ch]
#include <type_traits>
#include <utility>

#include "ra_internal.h"
#include "ra_plan.h"
#include "ra_xcd.h"

namespace ra {
namespace {

typedef float v16f __attribute__((ext_vector_type(16)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));
typedef _Float16 v8h __attribute__((ext_vector_type(8)));


__device__ __forceinline__ float h2f(uint16_t b, int is_fp16) {
  if (is_fp16) return __half2float(__ushort_as_half(b));
  return __uint_as_float(static_cast<uint32_t>(b) << 16);
}

__device__ __forceinline__ uint16_t f2h(float v, int is_fp16) {
  if (is_fp16) return __half_as_ushort(__float2half(v));
  return __bfloat16_as_ushort(__float2bfloat16(v));
}

__device__ __forceinline__ int fdiv(int n, int d, float inv_d) {
  int q = static_cast<int>(static_cast<float>(n) * inv_d);
  if (q * d > n) --q;
  if ((q + 1) * d <= n) ++q;
  return q;
}

// One workgroup per 32-token chunk and group of heads: plain RoPE of Q and K in
// binary32, rounded to 16 bits, written to the tiled layout.  A thread holds two
// 16-byte pieces of the chunk (8 channels of one token each) and the cosines and
// sines of their pairs, which do not depend on the head: it reads them once and
// turns the same piece of every head's Q and K with them (read per head, as one
// 16-byte table entry per pair, the tables were four times the bytes of the
// data, from the L2).  The plain RoPE block is [c s; -s c], so the first half of
// a table entry is all of it.  Global accesses are whole 256-byte rows on one
// side and the chunk's 8 KB in order on the other; the piece (token r, channels
// 8 u ..) passes through LDS slot 32 u + (r ^ u), which spreads the 16 pieces of
// a row over the banks.  32760 tokens, 12 heads, Q and K together: 133 -> 67 us
// (6 TB/s).
__global__ __launch_bounds__(256) void k_rope16(RopeTables t, const uint16_t* q, const uint16_t* k, uint16_t* qo,
                                                uint16_t* ko, int BH, int N, int Npad, int is_fp16, int heads) {
  __shared__ __align__(16) uint4 tile[2][512];
  const int c = blockIdx.x, tid = threadIdx.x;
  const int h0 = blockIdx.y * heads, nh = BH - h0 < heads ? BH - h0 : heads;
  const int u = tid & 15;          // channels 8 u .. 8 u + 7 of rows tid / 16 and 16 + tid / 16
  const int W = t.grid[2], Hg = t.grid[1];
  const int np0 = t.split[0] / 2, np1 = t.split[1] / 2, np2 = t.split[2] / 2;
  float2 cs[2][4];
  size_t src[2];
  bool in[2];
  int slot[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = 16 * i + (tid >> 4), n = 32 * c + r;
    in[i] = n < N;
    const int nn = in[i] ? n : N - 1;
    src[i] = static_cast<size_t>(nn) * kD + 8 * u;
    slot[i] = 32 * u + (r ^ u);
    const int tq = fdiv(nn, W * Hg, 1.0f / static_cast<float>(W * Hg));
    const int rem = nn - tq * W * Hg;
    const int hq = fdiv(rem, W, 1.0f / static_cast<float>(W));
    const int wq = rem - hq * W;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int p = 4 * u + e;
      const float4* g = p < np0 ? t.axis[0] + tq * np0 + p
                                : (p < np0 + np1 ? t.axis[1] + hq * np1 + (p - np0)
                                                 : t.axis[2] + wq * np2 + (p - np0 - np1));
      cs[i][e] = *reinterpret_cast<const float2*>(g);
    }
  }
  auto base = [&](int job) {   // job 2 h + (0 for Q, 1 for K)
    return ((job & 1) ? k : q) + static_cast<size_t>(h0 + (job >> 1)) * N * kD;
  };
  uint4 raw[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) raw[i] = *reinterpret_cast<const uint4*>(base(0) + src[i]);
  for (int job = 0; job < 2 * nh; ++job) {
    uint4* tl = tile[job & 1];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const uint32_t w[4] = {raw[i].x, raw[i].y, raw[i].z, raw[i].w};
      uint32_t o[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float x0 = h2f(w[e] & 0xffff, is_fp16), x1 = h2f(w[e] >> 16, is_fp16);
        const float y0 = __fmaf_rn(x1, -cs[i][e].y, __fmul_rn(x0, cs[i][e].x));
        const float y1 = __fmaf_rn(x1, cs[i][e].x, __fmul_rn(x0, cs[i][e].y));
        o[e] = in[i] ? f2h(y0, is_fp16) | (static_cast<uint32_t>(f2h(y1, is_fp16)) << 16) : 0u;
      }
      tl[slot[i]] = make_uint4(o[0], o[1], o[2], o[3]);
    }
    if (job + 1 < 2 * nh) {
#pragma unroll
      for (int i = 0; i < 2; ++i) raw[i] = *reinterpret_cast<const uint4*>(base(job + 1) + src[i]);
    }
    __syncthreads();   // two tiles: the next write goes to the other one
    uint4* dst = reinterpret_cast<uint4*>(((job & 1) ? ko : qo) +
                                          (static_cast<size_t>(h0 + (job >> 1)) * Npad + 32 * c) * kD);
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int x = 256 * i + tid;   // slot 32 u' + r'
      dst[x] = tl[(x & ~31) + ((x & 31) ^ (x >> 5))];
    }
  }
}

// The table copy (the first `copy_blocks` workgroups; src may be pinned host
// memory read through its device mapping) and the V relayout, which needs no
// tables: one workgroup per 32-token chunk and head, the chunk through LDS.
__global__ __launch_bounds__(256) void k_v16_relayout(const uint32_t* tsrc, uint32_t* tdst, int nwords,
                                                      int copy_blocks, const uint16_t* v, uint16_t* out, int N,
                                                      int Npad) {
  __shared__ uint16_t tile[32][kD + 2];
  const int tid = threadIdx.x;
  if (static_cast<int>(blockIdx.x) < copy_blocks) {
    const int i = blockIdx.x * 256 + tid;
    if (i < nwords) tdst[i] = tsrc[i];
    return;
  }
  const int nc = Npad / 32, x = blockIdx.x - copy_blocks;
  const int bh = x / nc, c = x - bh * nc;
  for (int i = tid; i < 32 * 32; i += 256) {
    const int r = i >> 5, cl = i & 31;
    const int n = c * 32 + r;
    uint2 w = make_uint2(0u, 0u);
    if (n < N) w = *reinterpret_cast<const uint2*>(v + (static_cast<size_t>(bh) * N + n) * kD + 4 * cl);
    tile[r][4 * cl + 0] = w.x & 0xffff;
    tile[r][4 * cl + 1] = w.x >> 16;
    tile[r][4 * cl + 2] = w.y & 0xffff;
    tile[r][4 * cl + 3] = w.y >> 16;
  }
  __syncthreads();
  // 512 output vectors of 8 elements: (s, h, ch)
  for (int i = tid; i < 512; i += 256) {
    const int ch = i & 127, h = (i >> 7) & 1, s = i >> 8;
    uint32_t e[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int e0 = 2 * q, e1 = 2 * q + 1;
      const int k0 = 16 * s + 8 * (e0 >> 2) + 4 * h + (e0 & 3);
      const int k1 = 16 * s + 8 * (e1 >> 2) + 4 * h + (e1 & 3);
      e[q] = tile[k0][ch] | (static_cast<uint32_t>(tile[k1][ch]) << 16);
    }
    const size_t off = static_cast<size_t>(bh) * Npad * kD + ((static_cast<size_t>(c * 2 + s) * 2 + h) * 128 + ch) * 8;
    *reinterpret_cast<uint4*>(out + off) = make_uint4(e[0], e[1], e[2], e[3]);
  }
}

template <bool F16>
struct MF;
template <>
struct MF<false> {
  typedef v8bf vec;
  typedef __bf16 v2t __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ v16f mfma(vec a, vec b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  }
};
template <>
struct MF<true> {
  typedef v8h vec;
  typedef _Float16 v2t __attribute__((ext_vector_type(2)));
  static __device__ __forceinline__ v16f mfma(vec a, vec b, v16f c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
  }
};

typedef float v2f __attribute__((ext_vector_type(2)));

// two binary32 values -> one dword of two 16-bit values (round to nearest even)
template <bool F16>
__device__ __forceinline__ uint32_t pack2(float x, float y) {
  const typename MF<F16>::v2t t = __builtin_convertvector(v2f{x, y}, typename MF<F16>::v2t);
  return __builtin_bit_cast(uint32_t, t);
}

// f(0) .. f(15), each index a compile-time constant
template <typename F, int... R>
__device__ __forceinline__ void each16_(F&& f, std::integer_sequence<int, R...>) {
  (f(std::integral_constant<int, R>()), ...);
}
template <typename F>
__device__ __forceinline__ void each16(F&& f) {
  each16_(f, std::make_integer_sequence<int, 16>());
}

template <typename V>
__device__ __forceinline__ V as_vec(uint4 u) {
  return __builtin_bit_cast(V, u);
}

// A tile of KV keys (K or V: KV * 256 bytes) from global memory straight into
// LDS, in pieces of 1 KB (16 bytes per lane), every wave its share.  Issued from
// asm, so the compiler does not wait for it at unrelated LDS accesses; dma_wait
// and a barrier make the data visible.
template <int KV, int NW>
__device__ __forceinline__ void dma_tile(const uint16_t* src, uint16_t* dst, int wave, int lane) {
#pragma unroll
  for (int i = 0; i < KV / (4 * NW); ++i) {
    const int o = (i * NW + wave) * 512;   // elements
    const void* g = src + o + 8 * lane;
#if defined(__HIP_DEVICE_COMPILE__)
    const unsigned l =
        static_cast<unsigned>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint16_t*)(dst + o)));
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off"
                 :
                 : "v"(g), "s"(__builtin_amdgcn_readfirstlane(l))
                 : "m0", "memory");
#else
    (void)g;
#endif
  }
}
__device__ __forceinline__ void dma_wait() {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}

// Output rows of a wave (register r of a tile: query 8 (r / 4) + 4 hh + r % 4 of
// the 32 from q0 on), tiles T0 .. T0 + NT - 1, times inv[r], in the output type;
// the type is chosen once, not per element.
template <int T0, int NT, typename T, typename F>
__device__ __forceinline__ void store_rows(T* o, const v16f (&of)[4], const float (&inv)[16], int N, int q0, int hh, F conv) {
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int qi = 8 * (r >> 2) + 4 * hh + (r & 3);
    if (q0 + qi < N) {
#pragma unroll
      for (int mt = T0; mt < T0 + NT; ++mt) o[qi * kD + mt * 32] = conv(of[mt][r] * inv[r]);
    }
  }
}
template <int T0, int NT>
__device__ __forceinline__ void finish_rows(const Fp16Args& a, const v16f (&of)[4], float ltot, int bh, int q0, int hh,
                                            int j) {
  float inv[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) inv[r] = 1.0f / __shfl(ltot, 8 * (r >> 2) + 4 * hh + (r & 3));
  const size_t ob = (static_cast<size_t>(bh) * a.N + q0) * kD + j;
  if (a.out_dtype == 2)
    store_rows<T0, NT>(static_cast<float*>(a.o) + ob, of, inv, a.N, q0, hh, [](float v) { return v; });
  else if (a.out_dtype == 1)
    store_rows<T0, NT>(static_cast<uint16_t*>(a.o) + ob, of, inv, a.N, q0, hh, [](float v) { return f2h(v, 1); });
  else
    store_rows<T0, NT>(static_cast<uint16_t*>(a.o) + ob, of, inv, a.N, q0, hh, [](float v) { return f2h(v, 0); });
}

// One wave = 32 queries; S^T = K Q^T puts the scores of one query in one lane
// (register r of chunk ch is key 32 ch + 8 (r / 4) + 4 hh + r % 4).  The 16-bit
// P values of register pairs are directly the A operand of O = P V (A and B
// operands share one lane layout), with V read as the B operand in the key
// order of its relayout, so a lane of the output tile holds one channel of 16
// queries (query 8 (r / 4) + 4 hh + r % 4 in register r).
//
// Software pipeline over blocks: once a 32-key chunk's probabilities are
// rounded to 16 bits, its score registers take the next block's scores of
// the same chunk; those products and the chunk's PV products run on the
// matrix core beside the next chunk's probabilities, with their LDS operands
// read four products ahead, and a block starts with its scores in registers.
// K tiles are staged two blocks ahead and V tiles one block ahead, so two LDS
// buffers of each suffice (block j + 2's K goes where block j's K was, whose
// scores were taken during block j - 1).
// NW waves share the K/V tiles.  8 (256 queries) put two waves on every SIMD of a
// compute unit with one copy of the tiles: at kv_block 128 the tiles fill the
// LDS, and 4 waves were alone with it (32760 tokens 7.40 -> 5.88 ms); at
// kv_block 64 the unit's tile traffic halves (6.17 -> 5.95 ms; the kernel runs at
// the power limit there, 1.93-2.05 GHz of 2.4).  4 (128 queries) are for a last round that
// would leave units idle, and for heads that 256-query tiles fit badly.  The launch
// covers a list of tiles of 32 NW queries, per_head of them a head, from tile u0 on.
template <bool F16, int kKV, int NW>
__global__ __launch_bounds__(64 * NW, NW == 8 ? 1 : (kKV == 64 ? 2 : 1)) void k_attn16(Fp16Args a, int u0, int per_head) {
  typedef typename MF<F16>::vec vec;
  constexpr int NCH = kKV / 32;
  constexpr int TILE = kKV * kD;  // elements of K (and of V) per block
  __shared__ __align__(16) uint16_t sK[2][TILE];
  __shared__ __align__(16) uint16_t sV[2][TILE];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5, j = lane & 31;
  const int U = u0 + xcd_order(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x));
  const int bh = U / per_head;
  const int wq0 = (U - bh * per_head) * (32 * NW);
  if (wq0 >= a.N) return;   // the last tile of a head may reach past its tokens
  const int q0 = wq0 + wave * 32;
  const int qrow = q0 + j;
  const int N = a.N;
  const int nblocks = (N + kKV - 1) / kKV;
  const size_t hoff = static_cast<size_t>(bh) * a.Npad * kD;
  const uint16_t* kbase = a.k + hoff;
  const uint16_t* vbase = a.v + hoff;
  const float Kc = a.Kc;
  auto load_k = [&](int b) { dma_tile<kKV, NW>(kbase + static_cast<size_t>(b) * TILE, sK[b & 1], wave, lane); };
  auto load_v = [&](int b) { dma_tile<kKV, NW>(vbase + static_cast<size_t>(b) * TILE, sV[b & 1], wave, lane); };

  vec qop[8];
  {
    // (waves past the padded length, in the last workgroup, take the last rows
    // and store nothing)
    const int qr = qrow < a.Npad ? qrow : a.Npad - 32 + j;
    const uint16_t* qp = a.q + hoff + static_cast<size_t>(qr >> 5) * 4096 + (qr & 31) * 8;
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) qop[kc] = as_vec<vec>(*reinterpret_cast<const uint4*>(qp + (kc * 2 + hh) * 256));
  }

  v16f of[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) of[mt][r] = 0.f;
  float m = -INFINITY, l = 0.f;

  auto kop = [&](const uint16_t* kt, int ch, int kc) {
    return as_vec<vec>(*reinterpret_cast<const uint4*>(&kt[(((ch * 8 + kc) * 2 + hh) * 32 + j) * 8]));
  };
  v16f s[NCH];

  // prologue: K and V of block 0 and K of block 1 in LDS, block 0's scores
  load_k(0);
  load_v(0);
  if (nblocks > 1) load_k(1);
  dma_wait();
  __syncthreads();
#pragma unroll
  for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
    for (int r = 0; r < 16; ++r) s[ch][r] = 0.f;
#pragma unroll
  for (int kc = 0; kc < 8; ++kc)
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) s[ch] = MF<F16>::mfma(kop(sK[0], ch, kc), qop[kc], s[ch]);
  __syncthreads();   // every wave has read block 0's K before it is overwritten

  auto step = [&](int jb, auto masked_tag, auto more_tag) {
    constexpr bool MASKED = decltype(masked_tag)::value;
    constexpr bool more = decltype(more_tag)::value;
    // Issue priority: the block's dependent chain of vector work (maximum,
    // alpha, the first chunk's probabilities) and the first chunk's products
    // run at the higher priority, the remaining products at the lower one,
    // so the waves of a SIMD alternate halves (about 2 % faster than one
    // priority throughout).
    __builtin_amdgcn_s_setprio(1);
    const int buf = jb & 1;
    const int key0 = jb * kKV;
    // block j + 2's K where block j's was, block j + 1's V where block j - 1's
    // was: requested at the block's start, waited for at its end
    if (more) {
      if (jb + 2 < nblocks) load_k(jb + 2);
      load_v(jb + 1);
    }
    if (MASKED) {
#pragma unroll
      for (int ch = 0; ch < NCH; ++ch)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (key0 + ch * 32 + 8 * (r >> 2) + 4 * hh + (r & 3) >= N) s[ch][r] = -INFINITY;
    }

    // ---- row maximum of S * Kc (Kc > 0: the product of the maximum) ----
    // (a chain of three-input maxima per chunk, seeded below every score)
    float mx = -3.40282347e38f;
#pragma unroll
    for (int ch = 0; ch < NCH; ++ch) {
      float cx = -3.40282347e38f;
#pragma unroll
      for (int r = 0; r < 16; r += 2) cx = fmaxf(fmaxf(cx, s[ch][r]), s[ch][r + 1]);
      mx = fmaxf(mx, cx);
    }
    const float tmax = max_halves(__fmul_rn(mx, Kc));
    const float mnew = fmaxf(m, tmax);
    const float alpha = __builtin_amdgcn_exp2f(m - mnew);
    m = mnew;
    if (__any(alpha != 1.0f)) {
      const RowFactors ab = row_factors(alpha);
      auto row = [&](auto rc) {
        constexpr int r = decltype(rc)::value;
        const float ar = row_factor<r>(ab);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) of[mt][r] = __fmul_rn(of[mt][r], ar);
      };
      each16(row);
    }

    // ---- P = 2^(S Kc - m) in 16 bits, row sums of the unrounded P, O += P V ----
    float ls[4];
    uint32_t pw[NCH][8];
    auto probs = [&](int ch, int r2) {   // registers 2 r2, 2 r2 + 1 of chunk ch
      float P[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int r = 2 * r2 + u;
        float p = __builtin_amdgcn_exp2f(__fmaf_rn(s[ch][r], Kc, -mnew));
        if (MASKED && s[ch][r] == -INFINITY) p = 0.f;
        if (ch == 0 && r < 4) ls[r] = p;
        else ls[r & 3] += p;
        P[u] = p;
      }
      pw[ch][r2] = pack2<F16>(P[0], P[1]);
    };
    // the products of chunk c (group c): 8 PV products (k-step stp = i / 4,
    // tile mt = i % 4), then, with a next block, its 8 score products of chunk
    // c (channel step kc = i - 8); operand of product i of group c
    const uint16_t* kn = sK[buf ^ 1];
    auto opB = [&](int c, int i) {
      if (i < 8)
        return as_vec<vec>(
            *reinterpret_cast<const uint4*>(&sV[buf][(((c * 2 + (i >> 2)) * 2 + hh) * 128 + (i & 3) * 32 + j) * 8]));
      return kop(kn, c, i - 8);
    };
    constexpr int NPR = more ? 16 : 8;   // products per chunk
    auto product = [&](int c, int i, vec op) {
      if (i < 8) {
        const int stp = i >> 2, mt = i & 3;
        const vec A = as_vec<vec>(
            make_uint4(pw[c][4 * stp], pw[c][4 * stp + 1], pw[c][4 * stp + 2], pw[c][4 * stp + 3]));
        of[mt] = MF<F16>::mfma(A, op, of[mt]);
      } else {
        const int kc = i - 8;
        if (kc == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) s[c][r] = 0.f;
        }
        s[c] = MF<F16>::mfma(op, qop[kc], s[c]);
      }
    };
#pragma unroll
    for (int r2 = 0; r2 < 8; ++r2) probs(0, r2);
    // Operands are read from LDS kAhead products ahead, and every product is a
    // scheduling region of its own: left alone, the compiler moved the reads
    // back to one product before their use, and the matrix core waited for
    // them (1560 tokens, 12 heads 52.1 -> 50.2 us, 4680 tokens, 5 heads 109 ->
    // 104 us, 32760 tokens 6.09 -> 5.91 ms; 3, 6 or 8 ahead, or regions of two
    // products: 0.3 to 1.5 % slower).
    constexpr int kAhead = 4;
    vec ops[kAhead];
#pragma unroll
    for (int i = 0; i < kAhead; ++i) ops[i] = opB(0, i);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      // chunk c's products, beside chunk c + 1's probabilities
#pragma unroll
      for (int i = 0; i < NPR; ++i) {
        // the operand kAhead products ahead (into the next chunk's products)
        const int n2 = i + kAhead;
        const int c2 = n2 < NPR ? c : c + 1, i2 = n2 < NPR ? n2 : n2 - NPR;
        vec& op = ops[(c * NPR + i) % kAhead];
        product(c, i, op);
        if (c2 < NCH) op = opB(c2, i2);
        constexpr int PER = NPR / 8;   // products per pair of probabilities
        if (c + 1 < NCH && i % PER == PER - 1) probs(c + 1, i / PER);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (c == 0) __builtin_amdgcn_s_setprio(0);
    }
    l = __fmaf_rn(l, alpha, (ls[0] + ls[1]) + (ls[2] + ls[3]));
    if (more) dma_wait();
    __syncthreads();
  };

  using kNo = std::integral_constant<bool, false>;
  using kYes = std::integral_constant<bool, true>;
  for (int jb = 0; jb + 1 < nblocks; ++jb) step(jb, kNo(), kYes());
  step(nblocks - 1, kYes(), kNo());

  // ---- epilogue: O / l ----
  finish_rows<0, 4>(a, of, l + __shfl_xor(l, 32), bh, q0, hh, j);
}

// --------------------------------------------------- key-split variant --
// The same rows by workgroups of 4 waves and 64 queries: wave (qs, kh) takes
// queries 32 qs .. 32 qs + 31 and the half kh of every block's keys, so a
// block's chain (maximum, alpha, probabilities, products) is half as long and a
// 256-query tile becomes four workgroups.  The two waves of a row exchange the
// maxima of their halves across the block barrier, each keeps its own row sums
// and O over its keys, and both are added at the end.  The next block's scores
// go to registers of their own and are taken beside the maximum's chain.
template <bool F16, int kKV>
__global__ __launch_bounds__(256, kKV == 64 ? 2 : 1) void k_attn16_split(Fp16Args a, int tile0) {
  typedef typename MF<F16>::vec vec;
  constexpr int NCW = kKV / 64;   // 32-key chunks per wave
  constexpr int TILE = kKV * kD;
  __shared__ __align__(16) uint16_t sT[4 * TILE];   // K tiles of blocks j, j + 1 (j mod 2), then V
  __shared__ float sM[2][4][32];
  __shared__ float sL[4][64];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int hh = lane >> 5, j = lane & 31;
  const int qs = wave & 1, kh = wave >> 1;
  const int ntile = (a.Npad + 255) / 256;
  const int U = 4 * tile0 + xcd_order(static_cast<int>(blockIdx.x), static_cast<int>(gridDim.x));
  const int bh = (U >> 2) / ntile;
  const int wq0 = ((U >> 2) - bh * ntile) * 256 + (U & 3) * 64;
  if (wq0 >= a.N) return;   // the last tile of a head may reach past its tokens
  const int q0 = wq0 + 32 * qs, qrow = q0 + j;
  const int N = a.N;
  const int nblocks = (N + kKV - 1) / kKV;
  const size_t hoff = static_cast<size_t>(bh) * a.Npad * kD;
  const uint16_t* kbase = a.k + hoff;
  const uint16_t* vbase = a.v + hoff;
  const float Kc = a.Kc;
  uint16_t* const sK = sT;
  uint16_t* const sV = sT + 2 * TILE;
  auto load_k = [&](int b) { dma_tile<kKV, 4>(kbase + static_cast<size_t>(b) * TILE, sK + (b & 1) * TILE, wave, lane); };
  auto load_v = [&](int b) { dma_tile<kKV, 4>(vbase + static_cast<size_t>(b) * TILE, sV + (b & 1) * TILE, wave, lane); };

  load_k(0);
  load_v(0);
  if (nblocks > 1) load_k(1);
  vec qop[8];
  {
    const uint16_t* qp = a.q + hoff + static_cast<size_t>(qrow >> 5) * 4096 + (qrow & 31) * 8;
#pragma unroll
    for (int kc = 0; kc < 8; ++kc) qop[kc] = as_vec<vec>(*reinterpret_cast<const uint4*>(qp + (kc * 2 + hh) * 256));
  }
  v16f of[4];
#pragma unroll
  for (int mt = 0; mt < 4; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) of[mt][r] = 0.f;
  float m = -INFINITY, l = 0.f, gmax = -INFINITY;
  dma_wait();
  __syncthreads();

  v16f sa[NCW], sb[NCW];
  auto scores = [&](const uint16_t* kt, v16f (&s)[NCW]) {
#pragma unroll
    for (int c = 0; c < NCW; ++c) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[c][r] = 0.f;
#pragma unroll
      for (int kc = 0; kc < 8; ++kc) {
        const vec op = as_vec<vec>(
            *reinterpret_cast<const uint4*>(&kt[((((kh * NCW + c) * 8 + kc) * 2 + hh) * 32 + j) * 8]));
        s[c] = MF<F16>::mfma(op, qop[kc], s[c]);
      }
    }
  };
  // the scores of block jn are in s: keys past N masked, the half's row maximum
  // left for the row's other wave
  auto finish_scores = [&](int jn, v16f (&s)[NCW]) {
    if (jn == nblocks - 1 && N % kKV != 0) {
#pragma unroll
      for (int c = 0; c < NCW; ++c)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (jn * kKV + (kh * NCW + c) * 32 + 8 * (r >> 2) + 4 * hh + (r & 3) >= N) s[c][r] = -INFINITY;
    }
    // (seeded as in the plain kernel: the seed stays for a half whose scores are
    // all -inf, masked or not, and is below every other score of the row; -inf in
    // its place would make alpha of a first block without a finite score 2^NaN)
    float mx = -3.40282347e38f;
#pragma unroll
    for (int c = 0; c < NCW; ++c) {
      float cx = -3.40282347e38f;
#pragma unroll
      for (int r = 0; r < 16; r += 2) cx = fmaxf(fmaxf(cx, s[c][r]), s[c][r + 1]);
      mx = fmaxf(mx, cx);
    }
    gmax = max_halves(__fmul_rn(mx, Kc));
    if (hh == 0) sM[jn & 1][wave][j] = gmax;
  };
  scores(sK, sa);
  finish_scores(0, sa);
  __syncthreads();   // the maxima are visible; block 0's K has been read

  auto step = [&](int jb, v16f (&s)[NCW], v16f (&sn)[NCW], auto last_tag) {
    constexpr bool LAST = decltype(last_tag)::value;
    if (!LAST) {
      if (jb + 2 < nblocks) load_k(jb + 2);
      load_v(jb + 1);
      scores(sK + ((jb + 1) & 1) * TILE, sn);
    }
    const float mnew = fmaxf(m, fmaxf(gmax, sM[jb & 1][wave ^ 2][j]));
    const float alpha = __builtin_amdgcn_exp2f(m - mnew);
    m = mnew;
    if (__any(alpha != 1.0f)) {
      const RowFactors ab = row_factors(alpha);
      each16([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        const float ar = row_factor<r>(ab);
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) of[mt][r] = __fmul_rn(of[mt][r], ar);
      });
    }
    float ls[4];
    const uint16_t* vt = sV + (jb & 1) * TILE;
#pragma unroll
    for (int c = 0; c < NCW; ++c) {
      uint32_t pw[8];
#pragma unroll
      for (int r2 = 0; r2 < 8; ++r2) {
        float P[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int r = 2 * r2 + u;
          float p = __builtin_amdgcn_exp2f(__fmaf_rn(s[c][r], Kc, -mnew));
          if (LAST && s[c][r] == -INFINITY) p = 0.f;
          if (c == 0 && r < 4) ls[r] = p;
          else ls[r & 3] += p;
          P[u] = p;
        }
        pw[r2] = pack2<F16>(P[0], P[1]);
      }
#pragma unroll
      for (int stp = 0; stp < 2; ++stp) {
        const vec A = as_vec<vec>(make_uint4(pw[4 * stp], pw[4 * stp + 1], pw[4 * stp + 2], pw[4 * stp + 3]));
#pragma unroll
        for (int mt = 0; mt < 4; ++mt) {
          const vec op = as_vec<vec>(*reinterpret_cast<const uint4*>(
              &vt[((((kh * NCW + c) * 2 + stp) * 2 + hh) * 128 + mt * 32 + j) * 8]));
          of[mt] = MF<F16>::mfma(A, op, of[mt]);
        }
      }
    }
    l = __fmaf_rn(l, alpha, (ls[0] + ls[1]) + (ls[2] + ls[3]));
    if (!LAST) {
      finish_scores(jb + 1, sn);
      dma_wait();
    }
    __syncthreads();
  };
  using kNo = std::integral_constant<bool, false>;
  int jb = 0;
  for (; jb + 2 < nblocks; jb += 2) {
    step(jb, sa, sb, kNo());
    step(jb + 1, sb, sa, kNo());
  }
  if (jb + 1 < nblocks) {
    step(jb, sa, sb, kNo());
#pragma unroll
    for (int c = 0; c < NCW; ++c) sa[c] = sb[c];
  }
  step(nblocks - 1, sa, sb, std::integral_constant<bool, true>());

  // each wave finishes two of the row's four output tiles: it hands the other
  // two to its partner (the tiles have all been read)
  float* ox = reinterpret_cast<float*>(sT);
  float* mine = ox + wave * 32 * 64 + lane;
  const float* theirs = ox + (wave ^ 2) * 32 * 64 + lane;
  sL[wave][lane] = l;
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) mine[(mt * 16 + r) * 64] = kh == 0 ? of[2 + mt][r] : of[mt][r];
  __syncthreads();
  l += sL[wave ^ 2][lane];
  const float ltot = l + __shfl_xor(l, 32);
  auto take = [&](int t0) {
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int r = 0; r < 16; ++r) of[t0 + mt][r] += theirs[(mt * 16 + r) * 64];
  };
  if (kh == 0) {
    take(0);
    finish_rows<0, 2>(a, of, ltot, bh, q0, hh, j);
  } else {
    take(2);
    finish_rows<2, 2>(a, of, ltot, bh, q0, hh, j);
  }
}

}  // namespace

hipError_t launch_prepare16(const RopeTables& t, const uint32_t* tsrc, uint32_t* tdst, int64_t nwords,
                            const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* qo, uint16_t* ko,
                            uint16_t* vo, int BH, int N, int Npad, int is_fp16, hipStream_t s) {
  const int copy_blocks = static_cast<int>((nwords + 255) / 256);
  hipLaunchKernelGGL(k_v16_relayout, dim3(copy_blocks + Npad / 32 * BH), dim3(256), 0, s, tsrc, tdst,
                     static_cast<int>(nwords), copy_blocks, v, vo, N, Npad);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // 4 heads per workgroup, or fewer while that leaves under 4 workgroups per
  // compute unit, where a workgroup's chain of heads is what takes the time
  int heads = 4;
  while (heads > 1 && static_cast<int64_t>(Npad / 32) * ((BH + heads - 1) / heads) < 1024) heads /= 2;
  hipLaunchKernelGGL(k_rope16, dim3(Npad / 32, (BH + heads - 1) / heads), dim3(256), 0, s, t, q, k, qo, ko, BH, N,
                     Npad, is_fp16, heads);
  return hipGetLastError();
}

template <bool F16, int KV>
hipError_t launch_attn16(const Fp16Args& a, hipStream_t s) {
  const TilePlan p = plan_fallback(a.Npad, a.BH, KV, a.units);
  const int n256 = (a.Npad + 255) / 256;   // 256-query tiles of a head
  if (p.tiles128)
    hipLaunchKernelGGL((k_attn16<F16, KV, 4>), dim3(p.tiles128), dim3(256), 0, s, a, 0, a.Npad / 128);
  if (p.whole) hipLaunchKernelGGL((k_attn16<F16, KV, 8>), dim3(p.whole), dim3(512), 0, s, a, 0, n256);
  if (p.halves)
    hipLaunchKernelGGL((k_attn16<F16, KV, 4>), dim3(2 * p.halves), dim3(256), 0, s, a, 2 * p.whole, 2 * n256);
  if (p.quarters)
    hipLaunchKernelGGL((k_attn16_split<F16, KV>), dim3(4 * p.quarters), dim3(256), 0, s, a, p.whole);
  return hipGetLastError();
}

hipError_t launch_attn_fp16(const Fp16Args& a, int kv_block, hipStream_t s) {
  if (kv_block == 128) return a.is_fp16 ? launch_attn16<true, 128>(a, s) : launch_attn16<false, 128>(a, s);
  return a.is_fp16 ? launch_attn16<true, 64>(a, s) : launch_attn16<false, 64>(a, s);
}

}  // namespace ra
