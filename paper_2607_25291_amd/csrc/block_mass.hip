// Exact attention block mass per KV group for gfx950: the ground truth of the proxy-fidelity
// comparison (Sec. 3.2, Property 1: full attention's block mass defines the oracle mask).
//
// One workgroup per (batch n, KV head g, query block i) takes H query heads of the group at a time:
// b/32 waves per head, 32 query rows per wave. It walks the keys c <= the block's last row twice, in
// stages of 64 keys that every wave reads from LDS (double-buffered direct loads, the K layout of the
// attention kernel, S^T = K Q^T, one query row per lane pair): pass 1 keeps each row's running maximum
// (over its two lanes, tile by tile) and each lane's sum of exp over its keys (the two are added after
// the walk), pass 2 adds each block's probability sum, exp(s - m) / l over the wave's rows and the
// block's causal keys. The waves' sums of a block meet in LDS and are added in a fixed order, so the
// result is deterministic.
//
// Bound: vector ALU. A 32x32 tile of logits costs 256 MFMA cycles per SIMD and a little more of
// maximum, fma, exp2 and add, so four waves per SIMD (128 VGPRs) run one tile's MFMAs beside the
// arithmetic on the tile before. 32 / 8 heads, 8K tokens: 571 us, matrix cores busy 45 % and vector
// ALUs 74 % of 1.19 M cycles; 591 us without the pipeline; 3860 us with the keys read from global
// memory by every wave (32 scattered rows per load, one wave's tile at a time).
#include <mutex>

#include "cosa_device.h"
#include "cosa_internal.h"

namespace cosa {
namespace {

struct MassParams {
  const uint16_t* q;
  const uint16_t* k;
  float* mass;
  int Hq, Hkv, L, nb, G, n_units;
  float scale_log2;
};

// Sum of v over the wave as a wave-uniform value, in a fixed order (DPP within rows of 16 lanes,
// then the four row sums).
__device__ __forceinline__ float wave_sum(float v) {
  v += dpp_mov<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp_mov<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp_mov<0x141>(v);  // row_half_mirror
  v += dpp_mov<0x140>(v);  // row_mirror
  const float r0 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 0));
  const float r1 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 16));
  const float r2 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 32));
  const float r3 = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 48));
  return (r0 + r1) + (r2 + r3);
}

// v, or -inf where d (query minus key) is negative.
__device__ __forceinline__ float mask_above(float v, int d) {
  asm volatile("" : "+v"(d));
  const uint32_t masked = (uint32_t)(d >> 31);
  return __builtin_bit_cast(float, (__builtin_bit_cast(uint32_t, v) & ~masked) | (0xFF800000u & masked));
}

constexpr int kStageKeys = 64;
constexpr int kStageBytes = kStageKeys * kHeadDim * 2;
// The key stages, the waves' sums and a mass for every block fit the LDS of a CU.
static_assert(2 * kStageBytes + 2 * 16 * 4 + kMaxBlocks * 4 <= 160 * 1024, "LDS of block_mass_kernel");

template <int BLOCK, int H>
__global__ __attribute__((amdgpu_flat_work_group_size(BLOCK * 2 * H, BLOCK * 2 * H)))
__attribute__((amdgpu_waves_per_eu(4)))
void block_mass_kernel(const MassParams P) {
  constexpr int WPH = BLOCK / 32;              // waves per head
  constexpr int NW = WPH * H;
  constexpr int SPB = BLOCK / kStageKeys;      // stages per key block
  __shared__ __attribute__((aligned(1024))) char stage[2][kStageBytes];
  __shared__ float part[2][NW];  // each wave's sum of a block, by block parity
  extern __shared__ float slots[];             // [nb], the masses so far

  // Heaviest query blocks of every head first.
  const int heads = P.n_units / P.nb;
  const int ng = blockIdx.x % heads, i = P.nb - 1 - blockIdx.x / heads;
  const int g = ng % P.Hkv, n = ng / P.Hkv;
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int half = lane >> 5, l32 = lane & 31;
  const int hw = w / WPH, wl = w % WPH;
  for (int j = threadIdx.x; j <= i; j += NW * 64) slots[j] = 0.f;

  const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(P.k + (size_t)ng * P.L * kHeadDim), (short)0, P.L * kHeadDim * 2, 0x00020000);
  const int row0 = i * BLOCK + wl * 32;  // the wave's first query row
  const int n_stages = (i + 1) * SPB;
  int k_rd[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) k_rd[c] = l32 * 256 + (((2 * c + half) ^ (l32 & 15)) << 4);

  // The next stage's keys go into the buffer that was read last; `end` publishes them: every wave's
  // copies have landed and every wave is done with the other buffer.
  int buf = 0;
  auto fetch = [&](int ks, int to) __attribute__((always_inline)) {
    copy_page<kStageKeys, NW, true>(krs, stage[to], ks * kStageBytes, w, lane);
  };
  auto end = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_s_waitcnt(kVmcntLgkm0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // S^T tile t (0, 1) of the stage in the current buffer: register r holds key 64 ks + 32 t + 8 (r / 4) +
  // 4 half + r % 4 of the lane's query row.
  auto tile = [&](const bf16x8_t (&qf)[8], int t, f32x16_t& s) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c)
      s = mfma32x32x16(
          as_bf16x8(*reinterpret_cast<const u32x4_t*>(stage[0] + k_rd[c] + t * 32 * 256)), qf[c], s);
  };
  auto mask_tile = [&](int ks, int t, f32x16_t& s) __attribute__((always_inline)) {
    int qh = row0 + l32 - 4 * half - ks * kStageKeys - 32 * t;
    asm volatile("" : "+v"(qh));
#pragma unroll
    for (int r = 0; r < 16; ++r)  // the sign of (query - key) selects -inf, without compare masks
      s[r] = mask_above(s[r], qh - (8 * (r >> 2) + (r & 3)));
  };
  // One tile's MFMAs with the arithmetic on the tile before it in their shadow.
  auto interleave = [] __attribute__((always_inline)) {
    __builtin_amdgcn_sched_group_barrier(0x100, 3, 0);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      if (c < 5) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
    }
  };
  // One walk over the stages: use(s) takes each tile's logits. The tiles below the wave's diagonal are
  // pipelined one deep, across the stages and their barriers: in lock-step behind a barrier, the four
  // waves of a SIMD would otherwise all run their MFMAs first and all their arithmetic after them.
  // step(ks) runs once per stage, when `use` has taken every tile before stage ks.
  auto walk = [&](const bf16x8_t (&qf)[8], bool last, auto&& use, auto&& step)
      __attribute__((always_inline)) {
    const int n_full = row0 / kStageKeys;  // stages whose keys precede the wave's first row
    f32x16_t a, b;
#pragma unroll
    for (int r = 0; r < 16; ++r) b[r] = -INFINITY;  // adds nothing: the pipeline starts without a branch
    for (int ks = 0; ks < n_stages; ++ks) {
      if (ks + 1 < n_stages || !last) fetch(ks + 1 < n_stages ? ks + 1 : 0, buf ^ 1);
      if (ks < n_full) {
        tile(qf, 0, a);
        use(b);
        interleave();
        step(ks);
        tile(qf, 1, b);
        use(a);
        interleave();
      } else {
        if (ks == n_full) use(b);
        step(ks);
        if (ks * kStageKeys <= row0 + 31) {
          tile(qf, 0, a);
          tile(qf, 1, b);
          mask_tile(ks, 0, a);
          mask_tile(ks, 1, b);
          use(a);
          use(b);
        }
      }
      end();
      // The read offsets move to the other buffer once per stage.
      const int to_next = buf ? -kStageBytes : kStageBytes;
#pragma unroll
      for (int c = 0; c < 8; ++c) k_rd[c] += to_next;
      buf ^= 1;
    }
  };

  fetch(0, 0);
  end();
  for (int h0 = 0; h0 < P.G; h0 += H) {
    bf16x8_t qf[8];
    const uint16_t* qp =
        P.q + ((size_t)(n * P.Hq + g * P.G + h0 + hw) * P.L + row0 + l32) * kHeadDim + 8 * half;
#pragma unroll
    for (int c = 0; c < 8; ++c) qf[c] = as_bf16x8(ldg16(qp + 16 * c));

    // Pass 1: the row's maximum mb (logit * scale * log2 e), the same in its two lanes, and this lane's
    // sum of 2^(x - mb). Until the first finite logit mb is the lowest finite value, against which a masked
    // key (-inf) adds 0. The sum moves to a new maximum by 2^(mb - mbn) of the rounded maxima, which is
    // what its terms were formed with.
    // What each addition rounds off is carried along (Kahan): a row that one key dominates would
    // otherwise lose every tile of tiny terms, and its masses come out large by as much.
    float mb = -__FLT_MAX__, l = 0.f, lost = 0.f;
    walk(qf, false, [&](const f32x16_t& s) __attribute__((always_inline)) {
      float mx[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) mx[r] = vmax(vmax(s[r], s[r + 4]), vmax(s[r + 8], s[r + 12]));
      const float mbn = vmax(mb, half_max(vmax(vmax(mx[0], mx[1]), vmax(mx[2], mx[3]))) * P.scale_log2);
      float rs[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int r = 0; r < 16; ++r)
        rs[r & 3] += __builtin_amdgcn_exp2f(fmaf(s[r], P.scale_log2, -mbn));
      const float alpha = __builtin_amdgcn_exp2f(mb - mbn);
      const float base = l * alpha, y = ((rs[0] + rs[1]) + (rs[2] + rs[3])) - lost * alpha;
      l = base + y;
      lost = (l - base) - y;
      mb = mbn;
    }, [](int) {});
    // mrow is mb and the factor 1: both lanes hold the row's maximum. Written as plainly as that, pass 1's
    // loop is scheduled differently and the kernel takes 2 % longer (32 / 8 heads, 8K tokens 561 / 565 us,
    // 7 / 1 heads, 60 blocks of 128 1285 / 1314).
    const float mrow = half_max(mb);
    const float inv = 1.f / half_sum((l - lost) * __builtin_amdgcn_exp2f(mb - mrow));

    // Pass 2: probability mass of every key block over the wave's rows. A block's sums are posted in
    // the stage after its last one, published by that stage's barrier and added by one thread in the
    // stage after that; part[j & 1] is written again a barrier later at the earliest.
    float ps[4] = {0.f, 0.f, 0.f, 0.f};
    auto post = [&](int j) __attribute__((always_inline)) {
      const float wsum = wave_sum(((ps[0] + ps[1]) + (ps[2] + ps[3])) * inv);
      if (lane == 0) part[j & 1][w] = wsum;
#pragma unroll
      for (int r = 0; r < 4; ++r) ps[r] = 0.f;
    };
    auto add_block = [&](int j) __attribute__((always_inline)) {
      float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int x = 0; x < NW; ++x) a[x & 3] += part[j & 1][x];
      slots[j] += (a[0] + a[1]) + (a[2] + a[3]);
    };
    walk(qf, h0 + H >= P.G, [&](const f32x16_t& s) __attribute__((always_inline)) {
#pragma unroll
      for (int r = 0; r < 16; ++r)
        ps[r & 3] += __builtin_amdgcn_exp2f(fmaf(s[r], P.scale_log2, -mrow));
    }, [&](int ks) __attribute__((always_inline)) {
      if (ks > 0 && ks % SPB == 0) post(ks / SPB - 1);
      if (ks > SPB && (ks - 1) % SPB == 0 && threadIdx.x == (unsigned)(ks % NW) * 64)
        add_block((ks - 1) / SPB - 1);
    });
    post(i);
    __syncthreads();
    if (threadIdx.x == 0) {
      if (SPB == 1 && i > 0) add_block(i - 1);
      add_block(i);
    }
    __syncthreads();  // slots and part are used again
  }
  float* out = P.mass + ((size_t)ng * P.nb + i) * P.nb;
  for (int j = threadIdx.x; j <= i; j += NW * 64) out[j] = slots[j];
}

template <int BLOCK, int H>
hipError_t launch_t(const MassParams& P, size_t lds, hipStream_t stream) {
  static std::mutex mu;
  static size_t granted = 0;
  if (lds > 16 * 1024) {
    std::lock_guard<std::mutex> lock(mu);
    if (lds > granted) {
      const hipError_t e =
          hipFuncSetAttribute(reinterpret_cast<const void*>(&block_mass_kernel<BLOCK, H>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      granted = lds;
    }
  }
  hipLaunchKernelGGL((block_mass_kernel<BLOCK, H>), dim3(P.n_units), dim3(BLOCK * 2 * H), lds, stream,
                     P);
  return hipGetLastError();
}

// Query heads that share a workgroup's staged keys: as many of four as divide the group.
template <int BLOCK>
hipError_t launch_heads(const MassParams& P, size_t lds, hipStream_t stream) {
  if (P.G % 4 == 0) return launch_t<BLOCK, 4>(P, lds, stream);
  if (P.G % 2 == 0) return launch_t<BLOCK, 2>(P, lds, stream);
  return launch_t<BLOCK, 1>(P, lds, stream);
}

}  // namespace

hipError_t launch_block_mass(const Shape& sh, const uint16_t* q, const uint16_t* k, float* mass,
                             hipStream_t stream) {
  MassParams P{q, k, mass, sh.Hq, sh.Hkv, sh.L, sh.nb, sh.G, sh.B * sh.Hkv * sh.nb,
               sh.scale * 1.4426950408889634f};
  const size_t lds = (size_t)sh.nb * sizeof(float);
  return sh.b == 128 ? launch_heads<128>(P, lds, stream) : launch_heads<64>(P, lds, stream);
}

}  // namespace cosa
