// Ordered-skipping attention (OSK) and the dense causal flash baseline for gfx950.
//
// A workgroup computes HPW query heads of one KV group for one query block of b rows: b/32
// wavefronts per head, 32 query rows per wavefront. The K and V pages of each visited key block are
// fetched once into LDS and serve every head of the workgroup. Logits are formed transposed,
// S^T = K Q^T, with bf16 MFMA 32x32x16 so that every lane owns one query row; the online softmax
// runs in fp32 (Sec. 3.1). OSK walks the KAP list (Algorithm A, attention loop) and after Q K^T
// decides, for each head's whole b-row tile at once, whether the value side can be skipped
// (Eq. (skip)); the dense kernel visits j = 0..i in order and never skips.
//
// Pages move from HBM straight into LDS (buffer loads with an LDS destination: no registers are
// spent on staging), double-buffered. Each wave works through its pages in two halves,
//   QK(m): Q K^T of page m, the diagonal mask, the new running max and the wave's skip vote;
//   PV(m): the skip decision from the votes, softmax, P V of page m;
// with a workgroup barrier after each half. With two heads of 128-row tiles (and in some grids of
// 64-row tiles, launch_t) the waves of the second head start one barrier later, so phase 2m runs
// QK(m) of head 0 beside PV(m-1) of head 1 and phase
// 2m+1 runs PV(m) of head 0 beside QK(m) of head 1. Waves w and w + 4 share a SIMD: while one
// issues the Q K^T MFMAs the other runs its softmax VALU work and P V MFMAs. The waves of head 0
// fetch K pages (page m+1 at the end of QK(m), after its vote), those of head 1 V pages (page m+1
// at the end of their QK(m)); a single head fetches both. Issuing a page copy stalls the issuing
// wave for about as long as the load path takes to accept it, so it comes after the Q K^T MFMAs:
// in a phase whose P V half computes, the copy then overlaps the partner wave's P V work instead
// of delaying the Q K^T chain. A wave waits for its own copies at the end of its PV half, so every
// copy has the rest of its phase and the next one to land before the barrier that publishes it.
//
// With one head in a workgroup (an odd number of query heads per KV head, or few tiles) nothing inside
// the workgroup fills the other's waits, so it keeps one page buffer per tensor instead of two and several
// workgroups share a CU (two of b = 128, four of b = 64: two waves per SIMD again), each at its own
// point of the walk. The next K page is fetched during PV(m) and the next V page during QK(m+1).
// Against double-buffered pages at one wave per SIMD: dense 28 / 4 heads, 9,856 tokens 867 -> 630 us;
// prefill 16 / 16 heads, 12,416 tokens 328 -> 271 us. Head pairs stay where they can be formed: they
// fetch each page once for both heads (32 / 8 heads, 32K tokens: 5 % faster than single heads).
//
// The grid is either one workgroup per tile (query block, head pair) or, when the caller supplies
// work-queue counters and the tiles outnumber what the CUs hold at once, persistent: as many workgroups
// as the CUs hold take tiles from per-XCD queues in the order the hardware would run them (see the
// tile loop below). The order of the tiles is unit_tile's, the choice of heads launch_shape's.
// With a paged KV cache (Sec. 4.3 "Physical jumping over pages"; appendix D.1) the copies gather a
// block's rows through the page table; everything from the LDS layouts on is shared.
//
// LDS layouts (one 16-byte slot of 8 values at a time; a direct load writes 64 consecutive slots,
// each lane picks the global slot that belongs there):
//   K [key][d]  256-byte rows, slot s of row r stored at slot s ^ (r % 16). The MFMA A-operand reads
//               (lane = key, 16 bytes of d) of 16 consecutive keys hit 16 different slots.
//   V [key][d]  256-byte rows, slot s of row r stored at slot s ^ 4 (r % 4). P V takes V through
//               transposing LDS reads (ds_read_b64_tr_b16): in each 16-lane group the lane i receives,
//               for k = 0..3, element i % 4 of the 8 bytes addressed by lane 4k + i / 4. Lane i
//               addressing V[key0 + i/4][d0 + 4 (i%4)] therefore receives keys key0..key0+3 of
//               column d0 + i, which is the P^T key set that lane holds from the S^T accumulators.
#include <limits.h>

#include <algorithm>
#include <type_traits>

#include "cosa_device.h"
#include "cosa_internal.h"

namespace cosa {
namespace {

typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef int i32x4_t __attribute__((ext_vector_type(4)));

// A wave-uniform read of data this kernel never writes (the count and first list entries in a
// tile's prologue), through the constant address space: a scalar load, counted apart from the
// vector memory operations (the Q fragments) already in flight. Inside the page loop the list is
// read with vector loads instead: an outstanding scalar load would make every LDS wait a full one.
__device__ __forceinline__ int32_t ld_uniform(const int32_t* p) {
  return *(const __attribute__((address_space(4))) int32_t*)(size_t)p;
}

// A packed sequence as the attention walks it (16 bytes: a lane reads two).
struct PackSeq {
  int start;       // first rank of its piece, INT_MAX past the last sequence
  int first, len;  // first block, blocks
  float tau;       // skip threshold
};

// The walking order of a pack (order_of): the sequences by falling length. Those before `tail` go one
// after the other, each from its last block down; the others go together, by falling position in their
// sequence. A piece is a range of ranks: piece k < tail is sequence k, piece k >= tail the positions that
// exactly the sequences tail .. k have.
struct PackOrder {
  int n, tail;  // n == 0: not packed
  alignas(16) PackSeq seq[kMaxPackedSeqs];
};

struct AttnParams {
  AttnArgs a;
  int Hq, Hkv, L, nb, G, n_units;
  // The (batch, KV head) pairs whose query blocks are walked together (unit_tile): n_front groups of
  // group_heads, then one of last_heads.
  int group_heads, n_front, last_heads;
  int fold;  // resident grids of more than one workgroup a CU: CUs of an XCD, otherwise 0
  float scale, scale_log2;
  PackOrder pack;
};

// The query block i of (batch, KV head) ng that unit u stands for, with the first block F and the skip
// threshold tau of the packed sequence that holds it (0 and the call's threshold without packing). The
// heads go in groups (group_heads_of); in a group the heaviest query blocks of every head come first, so
// that its last tiles are the lightest ones and the CUs finish together. With whole heads one after the
// other, the last head's heaviest blocks started when the others were done (dense, 32 / 8 heads, 4K
// tokens 190 -> 131 us, 8K 577 -> 478 us).
// Packs: lane l holds the sequences 2 l (pa) and 2 l + 1 (pb) of P.pack.seq, and a count of the pieces that
// start at or before the rank finds its own. The queries' loads wait for the block, so no memory is read
// on the way: a search through the kernel arguments took 0.4 us of every tile (16 / 8 heads, 60 sequences
// of 10 blocks of 128: 390 -> 385 us).
__device__ __forceinline__ void unit_tile(const AttnParams& P, i32x4_t pa, i32x4_t pb, int u, int& ng,
                                          int& i, int& F, float& tau) {
  const int gsz = P.group_heads * P.nb;
  const int grp = min(u / gsz, P.n_front), r = u - grp * gsz;
  int rank;  // two divisions by values the compiler keeps the reciprocals of
  if (grp < P.n_front) {
    rank = r / P.group_heads;
    ng = r - rank * P.group_heads;
  } else {
    rank = r / P.last_heads;
    ng = r - rank * P.last_heads;
  }
  ng += grp * P.group_heads;
  i = P.nb - 1 - rank;
  F = 0;
  tau = P.a.tau;
  if (P.pack.n > 0) {
    const int k = __popcll(__ballot(pa.x <= rank)) + __popcll(__ballot(pb.x <= rank)) - 1;
    auto of = [](int even, int odd, int q) {  // the value of sequence q
      const int e = __builtin_amdgcn_readlane(even, q >> 1), o = __builtin_amdgcn_readlane(odd, q >> 1);
      return (q & 1) ? o : e;
    };
    const int len = of(pa.z, pb.z, k);  // in the tail: of the shortest sequence that reaches the piece
    int down = rank - of(pa.x, pb.x, k), q = k;
    if (k > P.pack.tail) {
      const int together = k - P.pack.tail + 1, off = down;
      down = off / together;
      q = P.pack.tail + off - down * together;
    }
    F = of(pa.y, pb.y, q);
    tau = __builtin_bit_cast(float, of(pa.w, pb.w, q));
    i = F + len - down - 1;
  }
}

template <int BLOCK, int HPW>
struct TileCfg {
  static constexpr int kWavesPerHead = BLOCK / 32;
  static constexpr int kWaves = HPW * kWavesPerHead;
  static constexpr int kThreads = kWaves * 64;
  static constexpr int kKeyTiles = BLOCK / 32;
  static constexpr int kPage = BLOCK * kHeadDim * 2;         // bytes of one K or V page
  // Page buffers per tensor: two, or one where a workgroup holds a single head (see the file comment).
  static constexpr int kStages = HPW == 1 ? 1 : 2;
  static constexpr int kLdsBytes = 2 * kStages * kPage;
  static constexpr int kWgPerCu = (160 * 1024) / (kLdsBytes + 256);
  static constexpr int kWavesPerEu = (kWgPerCu * kWaves) / 4 > 1 ? (kWgPerCu * kWaves) / 4 : 1;
};

// Paged variant (Sec. 4.3 "Physical jumping over pages"): the block's rows live in physical pages of
// 2^log2p >= 16 tokens of a [n_pages, Hkv, page, d] cache. Wave w moves the consecutive chunks
// w * CPW .. w * CPW + CPW - 1 in runs of four (16 rows): a run starts 16-aligned, so it lies inside
// one physical page whatever the page size, and each run takes one buffer resource, its chunks
// immediate offsets from it (no per-chunk test for a page boundary). Lane k of `tbl` holds the raw
// table entry of the block's k-th page-sized segment (segment 0 when a page holds the block). A run
// reads its entry into a scalar register and forms the page address there (the range clamp, a
// 64-bit multiply by the page stride `pstride` and the add to the head's cache base `cache`), so
// that the copy adds no vector instructions to the wave that issues it; entries outside
// [0, n_pages) read page 0.
template <int BLOCK, int NW, bool IS_K, bool WHOLE>
__device__ __forceinline__ void copy_page_paged(int tbl, uint64_t cache, uint64_t pstride,
                                                unsigned n_pages, int first_row, int log2p,
                                                char* dst, int w, int lane) {
  constexpr int kChunks = BLOCK * kHeadDim * 2 / 1024;
  constexpr int CPW = kChunks / NW;
  static_assert(kChunks % NW == 0 && CPW % 4 == 0, "each wave moves a multiple of 16 rows");
  const int page_mask = (1 << log2p) - 1;
  // Opaque wave index: the per-chunk offsets are formed here instead of being hoisted out of the
  // page loop into scalar registers.
  asm volatile("" : "+s"(w));
  if constexpr (WHOLE) {
    // The block lies inside one physical page (page size >= block): one resource for the wave's
    // chunks, as for a contiguous cache.
    const uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane(tbl);
    const uint64_t base = cache + (uint64_t)(e < n_pages ? e : 0u) * pstride;
    const int in_page = first_row & page_mask;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(base + (uint64_t)in_page * (kHeadDim * 2)), (short)0, BLOCK * kHeadDim * 2,
        0x00020000);
    int lds0 = (int)(size_t)COSA_LDS(dst) + w * CPW * 1024;
    int src0 = w * CPW * 1024;
    asm volatile("" : "+s"(lds0), "+s"(src0));
#pragma unroll
    for (int u = 0; u < CPW; ++u) {
      // Row 4 (w CPW + u) + lane / 16 of the block; only its residue mod 16 enters the swizzle,
      // and w CPW is a multiple of 4.
      const int row = 4 * (u & 3) + (lane >> 4);
      const int stored = lane & 15;
      const int slot = IS_K ? (stored ^ (row & 15)) : (stored ^ ((row & 3) << 2));
      const int voff = (lane >> 4) * (kHeadDim * 2) + slot * 16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (__attribute__((address_space(3))) void*)(size_t)(lds0 + u * 1024), 16, voff,
          src0 + u * 1024, 0, 0);
    }
    return;
  }
#pragma unroll
  for (int run = 0; run < CPW / 4; ++run) {
    const int row0 = (w * CPW + 4 * run) * 4;  // first row of the run within the block
    const int in_page = (first_row + row0) & page_mask;
    const int seg = row0 >> log2p;
    const uint32_t e = (uint32_t)__builtin_amdgcn_readlane(tbl, seg);
    const uint64_t base = cache + (uint64_t)(e < n_pages ? e : 0u) * pstride;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(base + (uint64_t)in_page * (kHeadDim * 2)), (short)0, 16 * kHeadDim * 2,
        0x00020000);
#pragma unroll
    for (int u4 = 0; u4 < 4; ++u4) {
      const int u = 4 * run + u4;
      // Row 4 (w CPW + u) + lane / 16 of the block; only its residue mod 16 enters the swizzle,
      // and w CPW is a multiple of 4.
      const int row = 4 * (u & 3) + (lane >> 4);
      const int stored = lane & 15;
      const int slot = IS_K ? (stored ^ (row & 15)) : (stored ^ ((row & 3) << 2));
      const int voff = (lane >> 4) * (kHeadDim * 2) + slot * 16;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, COSA_LDS(dst + (w * CPW + u) * 1024), 16, voff,
                                               u4 * 1024, 0, 0);
    }
  }
}

// Where the keys and values live: contiguous [B, Hkv, L, d], or a paged cache whose pages are
// smaller than a block (a block spans several pages) or at least a block (one page holds it).
constexpr int kPgNone = 0;
constexpr int kPgSplit = 1;
constexpr int kPgWhole = 2;

// How the key blocks of a query block are walked.
constexpr int kWalkDense = 0;  // j = 0 .. i ascending, every block computed
constexpr int kWalkList = 1;   // OSK: the KAP list in list order, rowmax skip vote
constexpr int kWalkMask = 2;   // j = 0 .. i ascending, blocks whose mask byte is 0 skipped in-loop

// Mask byte of block j of a row whose last causal block is i (0 past it).
__device__ __forceinline__ int mask_byte(const uint8_t* mrow, int j, int i) {
  return j <= i ? mrow[j] : 0;
}

// Zeroes the work-queue counters of a persistent OSK launch (one per XCD, 128 bytes apart).
__global__ void queue_reset(uint32_t* queue) {
  if (threadIdx.x < kNumXcd) queue[threadIdx.x * kOskQueueStep] = 0u;
}

template <int BLOCK, int HPW, int WALK, int PG, bool PERSIST, bool STAGGER>
__global__ __attribute__((amdgpu_flat_work_group_size(TileCfg<BLOCK, HPW>::kThreads,
                                                      TileCfg<BLOCK, HPW>::kThreads)))
__attribute__((amdgpu_waves_per_eu(TileCfg<BLOCK, HPW>::kWavesPerEu,
                                   TileCfg<BLOCK, HPW>::kWavesPerEu)))
void attention_kernel(const AttnParams P) {
  using Cfg = TileCfg<BLOCK, HPW>;
  constexpr bool PAGED = PG != kPgNone;
  constexpr bool OSK = WALK == kWalkList;
  constexpr bool MASKED = WALK == kWalkMask;
  constexpr int KT = Cfg::kKeyTiles;
  constexpr int WPH = Cfg::kWavesPerHead;
  constexpr int PAGE = Cfg::kPage;
  // V buffers first: they get the low 64 KiB, where every transposing read's buffer and key offsets
  // fit the instruction's immediate (the K reads add their buffer base once per d chunk).
  __shared__ __attribute__((aligned(1024))) char v_lds0[PAGE];
  __shared__ __attribute__((aligned(1024))) char v_lds1[Cfg::kStages == 2 ? PAGE : 16];
  __shared__ __attribute__((aligned(1024))) char k_lds0[PAGE];
  __shared__ __attribute__((aligned(1024))) char k_lds1[Cfg::kStages == 2 ? PAGE : 16];
  __shared__ float vote[2][Cfg::kWaves];
  __shared__ int tile_slot;

  // Persistent grid (OSK with a work queue): a grid that fills the CUs takes tiles until none are left.
  // Slot p is the tile the hardware would run as workgroup p; queue x hands out the slots
  // p = x + 8 k, which the hardware would deal to XCD x, heaviest first. A workgroup starts on its
  // own XCD's queue and moves on to the next one when that is empty, so every tile is taken exactly
  // once and every workgroup leaves once all eight queues are empty. Thread 0 claims the next slot
  // during the last page of the current tile, which hides the atomic's latency without holding a
  // slot for long, and broadcasts it through LDS.
  const int n_slots = (P.n_units + kNumXcd - 1) / kNumXcd * kNumXcd * (P.G / HPW);
  int qx = PERSIST ? (int)(__builtin_amdgcn_s_getreg(0xF814) & (kNumXcd - 1)) : 0;  // XCC_ID
  int qtried = 0;
  unsigned k_next = 0u;
  bool have_next = false;
  auto claim = [&]() -> int {
    while (qtried < kNumXcd) {
      const int p = qx + kNumXcd * (int)atomicAdd(&P.a.queue[qx * kOskQueueStep], 1u);
      if (p < n_slots) return p;
      qx = (qx + 1) & (kNumXcd - 1);
      ++qtried;
    }
    return -1;
  };
  // The pack's sequences, two a lane (unit_tile); read once, not behind each tile's stores.
  i32x4_t pack_even = {0, 0, 0, 0}, pack_odd = {0, 0, 0, 0};
  if (P.pack.n > 0) {
    const i32x4_t* seq = reinterpret_cast<const i32x4_t*>(P.pack.seq) + 2 * (threadIdx.x & 63);
    pack_even = seq[0];
    pack_odd = seq[1];
  }
  for (;;) {
  int unit, pair;
  if constexpr (PERSIST) {
    if (threadIdx.x == 0) {
      int p = -1;
      if (have_next) {
        p = qx + kNumXcd * (int)k_next;
        if (p >= n_slots) {
          qx = (qx + 1) & (kNumXcd - 1);
          ++qtried;
          p = claim();
        }
      } else {
        p = claim();
      }
      have_next = false;
      tile_slot = p;
    }
    __syncthreads();
    const int ps = __builtin_amdgcn_readfirstlane(tile_slot);
    __syncthreads();
    if (ps < 0) return;
    if (!map_tile(ps, P.G / HPW, P.n_units, unit, pair)) continue;
  } else {
    int p = blockIdx.x;
    if (P.fold > 0) {  // rounds of P.fold workgroups an XCD, every second one backwards (launch_t)
      const int k = p >> 3, round = k / P.fold, first = round * P.fold;
      const int last = min(first + P.fold, (int)gridDim.x >> 3) - 1;
      if (round & 1) p = ((first + last - k) << 3) | (p & 7);
    }
    if (!map_tile(p, P.G / HPW, P.n_units, unit, pair)) return;
  }
  // Packed sequences: block i only sees the blocks F .. i of its own sequence, whose skip threshold
  // is its own (the masked walk is never packed).
  int ng, i, F;  // ng = n * Hkv + g
  float tau;
  unit_tile(P, pack_even, pack_odd, unit, ng, i, F, tau);
  const int g = ng % P.Hkv, n = ng / P.Hkv;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave index, scalar
  const int half = lane >> 5, l32 = lane & 31;
  const int hw = w / WPH, wl = w % WPH;  // head slot in the workgroup, wave within the head
  const int h = g * P.G + pair * HPW + hw;

  const size_t kv_off = (size_t)ng * P.L * kHeadDim;
  const size_t qo_off = (size_t)(n * P.Hq + h) * P.L * kHeadDim;
  const int qrow = i * BLOCK + wl * 32 + l32;
  const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(P.a.k + kv_off), (short)0, P.L * kHeadDim * 2, 0x00020000);
  const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(P.a.v + kv_off), (short)0, P.L * kHeadDim * 2, 0x00020000);

  // Q^T as the MFMA B operand: lane owns query row qrow, 8 chunks of 16 d (8 per lane half). Loaded
  // first: it does not depend on the list, so its latency overlaps the list reads below.
  bf16x8_t qf[8];
  {
    const uint16_t* qp = P.a.q + qo_off + (size_t)qrow * kHeadDim + 8 * half;
#pragma unroll
    for (int c = 0; c < 8; ++c) qf[c] = as_bf16x8(ldg16(qp + 16 * c));
  }

  int cnt;
  const int32_t* lst = nullptr;
  const uint8_t* mrow = nullptr;
  if constexpr (OSK) {
    cnt = ld_uniform(P.a.count + (size_t)ng * P.nb + i);
    cnt = cnt < P.nb ? cnt : P.nb;
    lst = P.a.order + ((size_t)ng * P.nb + i) * P.nb;
  } else if constexpr (MASKED) {
    mrow = P.a.mask + ((size_t)ng * P.nb + i) * P.nb;
    cnt = 0;
    for (int b0 = 0; b0 <= i; b0 += 64) cnt += __popcll(__ballot(mask_byte(mrow, b0 + lane, i) != 0));
  } else {
    cnt = i - F + 1;
  }
  // The mask walk: the bits of the 64 blocks from mbase on that are still ahead, and the mask bytes of
  // the 64 blocks after those, in flight. A run of masked blocks costs the walk a bit scan (and a
  // load per 64 blocks), nothing is fetched or computed for it. When every masked block was a step
  // with the walk's two barriers, 32 / 8 heads, 16K tokens, 27 % of the blocks took 703 us; now 601.
  uint64_t mbits = 0;
  int mbase = -64, mahead = 0;
  if constexpr (MASKED) mahead = mask_byte(mrow, lane, i);
  auto next_masked = [&]() -> int {
    while (mbits == 0 && mbase + 64 <= i) {
      mbase += 64;
      mbits = __ballot(mahead != 0);
      mahead = mask_byte(mrow, mbase + 64 + lane, i);
    }
    if (mbits == 0) return -1;
    const int j = mbase + __builtin_ctzll(mbits);
    mbits &= mbits - 1;
    return j;
  };
  // List entries, read ahead of their use. A malformed entry (outside [F, i]) is fetched as block
  // i but contributes nothing.
  auto raw_entry = [&](int kk) -> int {
    if constexpr (OSK) return kk < cnt ? lst[kk] : 0;
    else return F + kk;
  };
  auto listed = [&](int raw) -> bool { return (unsigned)(raw - F) <= (unsigned)(i - F); };
  auto page_of = [&](int raw) -> int { return listed(raw) ? raw : i; };

  // Physical pages of a listed block (paged caches): lane k loads the table entry of the block's k-th
  // page-sized segment (the lanes past the block's segments load entries they do not use, those past
  // the sequence's row read 0), through a buffer resource over the row of sequence n. The entry is
  // checked only where it is used, a page later: a check right after the load would wait for it.
  const int log2p = PAGED ? P.a.pg.log2_page : 0;
  const unsigned n_pages = PAGED ? (unsigned)min(P.a.pg.n_pages, 1LL << 31) : 0u;
  const __amdgpu_buffer_rsrc_t trs = __builtin_amdgcn_make_buffer_rsrc(
      PAGED ? (void*)(P.a.pg.table + (size_t)n * P.a.pg.pages_per_seq) : nullptr, (short)0,
      PAGED ? P.a.pg.pages_per_seq * 4 : 0, 0x00020000);
  auto table_of = [&](int raw) -> int {
    if constexpr (PAGED) {
      const int lp = ((page_of(raw) * BLOCK) >> log2p) + lane;
      return __builtin_amdgcn_raw_buffer_load_b32(trs, lp * 4, 0, 0);
    }
    return 0;
  };
  auto copy_block = [&](auto is_k, auto nwc, int raw, int tbl, char* dst, int wv)
      __attribute__((always_inline)) {
    constexpr bool IS_K = decltype(is_k)::value;
    constexpr int NW = decltype(nwc)::value;
    if constexpr (PAGED) {
      // K or V cache of KV head g; one physical page of one head is page * d elements, pages of
      // consecutive page numbers are Hkv of those apart.
      const uint64_t head_page_bytes = (uint64_t)kHeadDim * 2 << log2p;
      const uint64_t cache = (uint64_t)(IS_K ? P.a.k : P.a.v) + (uint64_t)g * head_page_bytes;
      copy_page_paged<BLOCK, NW, IS_K, PG == kPgWhole>(
          tbl, cache, head_page_bytes * (uint64_t)P.Hkv, n_pages, page_of(raw) * BLOCK, log2p, dst,
          wv, lane);
    } else {
      copy_page<BLOCK, NW, IS_K>(IS_K ? krs : vrs, dst, page_of(raw) * PAGE, wv, lane);
    }
  };

  // Prologue: K and V of page 0.
  auto first_entry = [&](int kk) -> int {
    if constexpr (OSK) return kk < cnt ? ld_uniform(lst + kk) : 0;
    else if constexpr (MASKED) return next_masked();
    else return raw_entry(kk);
  };
  const int raw0 = __builtin_amdgcn_readfirstlane(first_entry(0));
  const int raw1 = __builtin_amdgcn_readfirstlane(first_entry(1));
  const int raw2 = __builtin_amdgcn_readfirstlane(first_entry(2));
  int tbl_nxt = 0;
  if constexpr (PAGED) {
    // The first block's table entries come through scalar loads (lane k of tbl0 gets entry k), so
    // that its copies start without waiting for the Q fragments' vector loads issued above; the
    // next block's entries load as in the page loop.
    const int nseg = max(BLOCK >> log2p, 1);
    const int32_t* trow = P.a.pg.table + (size_t)n * P.a.pg.pages_per_seq +
                          ((page_of(raw0) * BLOCK) >> log2p);
    int tbl0 = 0;
#pragma unroll
    for (int kseg = 0; kseg < BLOCK / 16; ++kseg) {  // unconditional loads (clamped), issued together
      const int e = ld_uniform(trow + min(kseg, nseg - 1));
      tbl0 = lane == kseg ? e : tbl0;
    }
    tbl_nxt = table_of(raw1);
    if (cnt > 0) {
      copy_block(std::true_type{}, std::integral_constant<int, Cfg::kWaves>{}, raw0, tbl0, k_lds0, w);
      copy_block(std::false_type{}, std::integral_constant<int, Cfg::kWaves>{}, raw0, tbl0, v_lds0,
                 w);
    }
  } else {
    if (cnt > 0) {
      copy_block(std::true_type{}, std::integral_constant<int, Cfg::kWaves>{}, raw0, 0, k_lds0, w);
      copy_block(std::false_type{}, std::integral_constant<int, Cfg::kWaves>{}, raw0, 0, v_lds0, w);
    }
  }

  // O^T accumulators: tile dt holds d = 32 dt + 8 (r / 4) + 4 half + r % 4 of row qrow.
  f32x16_t o[4];
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[dt][r] = 0.f;
  float m = -INFINITY;  // running row max (raw logits), identical in both lane halves
  float lsum = 0.f;     // this lane half's partial row sum

  // LDS read offsets. K: key 32 t + l32, d slot 2 c + half (t is an immediate). V: transposing
  // reads of rows 32 t + 16 c2 + 8 a + 4 half + (i / 4) and d = 32 dt + 16 g16 + 4 (i % 4), with
  // i = lane % 16 and g16 = (lane / 16) % 2 (t, c2, a are immediates; one offset per dt).
  int k_rd[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) k_rd[c] = l32 * 256 + (((2 * c + half) ^ (l32 & 15)) << 4);
  int v_rd[4];
  {
    const int li = lane & 15, g16 = (lane >> 4) & 1;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt) {
      const int slot = 4 * dt + 2 * g16 + ((li & 3) >> 1);
      v_rd[dt] = (4 * half + (li >> 2)) * 256 + ((slot ^ ((li >> 2) << 2)) << 4) + 8 * (li & 1);
    }
  }
  const size_t log_off = ((size_t)(n * P.Hq + h) * P.nb + i) * P.nb;
  int ncomp = 0;
  // List entries of pages m (cur), m+1 (nxt) and m+2 (nxt2), scalar; pre holds entry m+3 in flight
  // and, for paged caches, tbl_nxt2 the physical pages of entry m+2.
  int cur = raw0, nxt = raw1, nxt2 = raw2;
  int pre = 0, tbl_nxt2 = 0;

  __builtin_amdgcn_s_waitcnt(0);  // prologue pages, list entries and Q fragments
  __syncthreads();

  // State handed from QK(m) to PV(m) of the same wave.
  f32x16_t s[KT];
  float mnew = -INFINITY;
  bool v_pend = false;  // page m is a valid entry

  // QK(m) on K buffer BUF.
  auto qk_half = [&](auto bufc) __attribute__((always_inline)) {
    constexpr int BUF = decltype(bufc)::value;
    const char* Kb = BUF ? k_lds1 : k_lds0;
    const int j = page_of(cur);
    v_pend = OSK ? listed(cur) : true;
    // S^T tile t: keys 32 t + 8 (r / 4) + 4 half + r % 4 (register r) of query row qrow. The d chunk
    // is the outer loop: the KT tiles are independent accumulation chains. The KT fragments of
    // chunk c + 1 are read from LDS right after the first MFMA of chunk c, so their latency hides
    // behind that chunk's MFMAs (it is exposed when the partner wave has no P V work to fill in).
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[t][r] = 0.f;
    bf16x8_t kf[2][KT];
#pragma unroll
    for (int t = 0; t < KT; ++t)
      kf[0][t] = as_bf16x8(*reinterpret_cast<const u32x4_t*>(Kb + k_rd[0] + t * 32 * 256));
    __builtin_amdgcn_sched_group_barrier(0x100, KT, 0);
#pragma unroll
    for (int c = 0; c < 8; ++c) {
      if (c + 1 < 8) {
#pragma unroll
        for (int t = 0; t < KT; ++t)
          kf[(c + 1) & 1][t] =
              as_bf16x8(*reinterpret_cast<const u32x4_t*>(Kb + k_rd[c + 1] + t * 32 * 256));
      }
#pragma unroll
      for (int t = 0; t < KT; ++t) s[t] = mfma32x32x16(kf[c & 1][t], qf[c], s[t]);
      if (c + 1 < 8) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);       // first MFMA of chunk c,
        __builtin_amdgcn_sched_group_barrier(0x100, KT, 0);      // the reads of chunk c + 1,
        __builtin_amdgcn_sched_group_barrier(0x008, KT - 1, 0);  // the rest of chunk c
      } else {
        __builtin_amdgcn_sched_group_barrier(0x008, KT, 0);
      }
    }
    if (j == i) {  // diagonal block: causal mask inside the tile
      // key 32 t + 8 (r / 4) + 4 half + r % 4 > query wl*32 + l32, with the lane part moved to the
      // right-hand side so that every compare is against an immediate
      // (the sign of qh - key selects -inf bit by bit, so no compare masks are kept in registers)
      int qh = wl * 32 + l32 - 4 * half;
      asm volatile("" : "+v"(qh));
#pragma unroll
      for (int t = 0; t < KT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          int d = qh - (32 * t + 8 * (r >> 2) + (r & 3));
          asm volatile("" : "+v"(d));
          const uint32_t masked = (uint32_t)(d >> 31);  // all ones where key > query
          const float sv = s[t][r];  // bit_cast of a vector element itself reads element 0
          const uint32_t bits = __builtin_bit_cast(uint32_t, sv);
          s[t][r] = __builtin_bit_cast(float, (bits & ~masked) | (0xFF800000u & masked));
        }
    }
    float mloc = -INFINITY;
#pragma unroll
    for (int t = 0; t < KT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) mloc = fmaxf(mloc, s[t][r]);
    mloc = half_max(mloc);
    mnew = v_pend ? fmaxf(m, mloc) : m;
    if constexpr (OSK) {
      // Eq. (skip): each head's b-row tile votes with its largest (m_loc - m), in nats. Unless
      // that margin is logged, only its comparison with tau matters: the tile is skipped exactly
      // when every row's margin is below tau, so a ballot replaces the cross-lane maximum and the
      // wave votes 0 (some row reaches tau; tau <= 0) or -inf (none does).
      const float d = (mloc - mnew) * P.scale;
      float marg;
      if (P.a.margin_log)
        marg = wave_max(d);
      else
        marg = __ballot(d >= tau) ? 0.f : -INFINITY;
      if (lane == 0) vote[BUF][w] = marg;
    }
  };

  // PV(kk) on V buffer BUF: the votes of this head's waves were posted in the previous phase.
  auto pv_half = [&](int kk, auto bufc) __attribute__((always_inline)) {
    constexpr int BUF = decltype(bufc)::value;
    const char* Vb = BUF ? v_lds1 : v_lds0;
    bool skip = !v_pend;
    if constexpr (OSK) {
      if (v_pend) {
        float dk = vote[BUF][hw * WPH];
#pragma unroll
        for (int ww = 1; ww < WPH; ++ww) dk = fmaxf(dk, vote[BUF][hw * WPH + ww]);
        skip = P.a.skip_on && (dk < tau);
        if (wl == 0 && lane == 0) {
          if (P.a.visit_log) P.a.visit_log[log_off + kk] = skip ? 2 : 1;
          if (P.a.margin_log) P.a.margin_log[log_off + kk] = dk;
        }
      }
    }
    // A skip implies m_loc < m in every row, so the running max is unchanged either way.
    if (!skip) {
      // A computing P V half is the critical path of its phase (softmax VALU, then its MFMAs,
      // beside the partner's Q K^T): its wave issues first, the partner fills the gaps.
      __builtin_amdgcn_s_setprio(1);
      const float alpha = __builtin_amdgcn_exp2f((m - mnew) * P.scale_log2);
      m = mnew;
      const float mb = mnew * P.scale_log2;
      if (__any(alpha != 1.f)) {  // the running max moved in some row of this wave
#pragma unroll
        for (int dt = 0; dt < 4; ++dt)
#pragma unroll
          for (int r = 0; r < 16; ++r) o[dt][r] *= alpha;
      }
      // O^T += V^T P^T over 16-key chunks kc = 2 t + c2: P^T element e of the chunk is register
      // 8 c2 + e of tile t (key 32 t + 16 c2 + 8 (e / 4) + 4 half + e % 4); the V^T operand is the
      // matching pair of transposing reads (e / 4 = a). The transposing reads are issued directly
      // so that the chunk and half-row offsets go into the instruction's offset field (the
      // compiler adds them to the address in a VALU op per read otherwise); the explicit wait
      // names the fragments, which hands them to the MFMAs and keeps their registers reserved
      // until the data has landed (the compiler does not see the reads as loads).
      // List and mask walks are software-pipelined: the V^T reads of chunk kc + 1 and the softmax
      // of chunk kc + 2 are issued behind the MFMAs of chunk kc (OSK 2.5 % faster). The dense
      // walk takes the softmax of the whole tile first, which measured 0.6 % faster there. Either
      // way the row sum takes the chunks, and their elements, in order.
      constexpr int KC = BLOCK / 16;
      constexpr bool kPipe = WALK != kWalkDense;
      float rs = 0.f;
      auto softmax_chunk = [&](int kc, bf16x8_t& pf) __attribute__((always_inline)) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float pv = __builtin_amdgcn_exp2f(
              fmaf(s[kc >> 1][8 * (kc & 1) + e], P.scale_log2, -mb));
          rs += pv;
          pf[e] = (__bf16)pv;
        }
      };
      int va[4];
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) va[dt] = (int)(size_t)COSA_LDS(Vb) + v_rd[dt];
      s16x4_t lo[2][4], hi[2][4];
      bf16x8_t pf[KC];
      if constexpr (kPipe) {
        softmax_chunk(0, pf[0]);
        softmax_chunk(1, pf[1]);
      } else {
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) softmax_chunk(kc, pf[kc]);
      }
#pragma unroll
      for (int dt = 0; dt < 4; ++dt) {
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(lo[0][dt]) : "v"(va[dt]), "i"(0));
        asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2"
                     : "=v"(hi[0][dt]) : "v"(va[dt]), "i"(8 * 256));
      }
#pragma unroll
      for (int kc = 0; kc < KC; ++kc) {
        const int cb = kc & 1, nx = cb ^ 1;
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(lo[cb][0]), "+v"(lo[cb][1]), "+v"(lo[cb][2]), "+v"(lo[cb][3]),
                       "+v"(hi[cb][0]), "+v"(hi[cb][1]), "+v"(hi[cb][2]), "+v"(hi[cb][3]));
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
          const bf16x8_t vf = __builtin_bit_cast(
              bf16x8_t, __builtin_shufflevector(lo[cb][dt], hi[cb][dt], 0, 1, 2, 3, 4, 5, 6, 7));
          o[dt] = mfma32x32x16(vf, pf[kc], o[dt]);
        }
        if (kc + 1 < KC) {
#pragma unroll
          for (int dt = 0; dt < 4; ++dt) {
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2"
                         : "=v"(lo[nx][dt]) : "v"(va[dt]), "i"((kc + 1) * 16 * 256));
            asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2"
                         : "=v"(hi[nx][dt]) : "v"(va[dt]), "i"((kc + 1) * 16 * 256 + 8 * 256));
          }
          if constexpr (kPipe) {
            if (kc + 2 < KC) softmax_chunk(kc + 2, pf[kc + 2]);
          }
        }
        if constexpr (!kPipe) {
          __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);  // the chunk's MFMAs ...
          __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);  // ... then the next chunk's reads
        }
      }
      lsum = fmaf(lsum, alpha, rs);
      ++ncomp;
      __builtin_amdgcn_s_setprio(0);
    }
  };

  // End of a phase: LDS writes done (and, with full, this wave's page copies landed), then the
  // workgroup barrier. The compiler barriers keep LDS accesses on their side of it.
  auto end_phase = [&](bool full) __attribute__((always_inline)) {
    if (full)
      __builtin_amdgcn_s_waitcnt(kVmcntLgkm0);
    else
      __builtin_amdgcn_s_waitcnt(kLgkm0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // Page kk, its buffers BUF: QK, fetch page kk+1 into the other buffers, barrier, PV, barrier.
  auto page = [&](int kk, auto bufc) __attribute__((always_inline)) {
    constexpr int BUF = decltype(bufc)::value;
    if constexpr (PERSIST) {
      if (kk == cnt - 1 && threadIdx.x == 0 && qtried < kNumXcd) {
        k_next = atomicAdd(&P.a.queue[qx * kOskQueueStep], 1u);
        have_next = true;
      }
    }
    if constexpr (!MASKED) pre = raw_entry(kk + 3);
    if constexpr (PAGED) tbl_nxt2 = table_of(nxt2);
    qk_half(bufc);
    const bool fetch = kk + 1 < cnt;
    constexpr auto NWH = std::integral_constant<int, WPH>{};
    if constexpr (Cfg::kStages == 1) {
      end_phase(true);  // this page's V has landed; every wave is done with its K
      if (fetch) copy_block(std::true_type{}, NWH, nxt, tbl_nxt, k_lds0, wl);
      pv_half(kk, bufc);
      end_phase(true);  // the next page's K has landed; every wave is done with this page's V
      if (fetch) copy_block(std::false_type{}, NWH, nxt, tbl_nxt, v_lds0, wl);
    } else {
      if (fetch) {
        if (hw == 0)
          copy_block(std::true_type{}, NWH, nxt, tbl_nxt, BUF ? k_lds0 : k_lds1, wl);
        else
          copy_block(std::false_type{}, NWH, nxt, tbl_nxt, BUF ? v_lds0 : v_lds1, wl);
      }
      end_phase(false);
      pv_half(kk, bufc);
      end_phase(true);
    }
    cur = nxt;
    nxt = nxt2;
    nxt2 = MASKED ? next_masked() : __builtin_amdgcn_readfirstlane(pre);
    tbl_nxt = tbl_nxt2;
  };

  // Head slot 1 runs one phase behind (launch_t says where).
  if (STAGGER && hw == 1) end_phase(false);
  if constexpr (Cfg::kStages == 1) {
    for (int kk = 0; kk < cnt; ++kk) page(kk, std::integral_constant<int, 0>{});
  } else {
    for (int kk = 0; kk < cnt; kk += 2) {
      page(kk, std::integral_constant<int, 0>{});
      if (kk + 1 < cnt) page(kk + 1, std::integral_constant<int, 1>{});
    }
  }
  if (STAGGER && hw == 0) end_phase(false);  // same barrier count for both head slots

  lsum = half_sum(lsum);
  const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
  uint16_t* op = P.a.o + qo_off + (size_t)qrow * kHeadDim;
#pragma unroll
  for (int dt = 0; dt < 4; ++dt)
#pragma unroll
    for (int rg = 0; rg < 4; ++rg) {
      const int d0 = 32 * dt + 8 * rg + 4 * half;
      uint32_t wv[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const __bf16 lo = (__bf16)(o[dt][4 * rg + 2 * e] * inv);
        const __bf16 hi = (__bf16)(o[dt][4 * rg + 2 * e + 1] * inv);
        wv[e] = (uint32_t)__builtin_bit_cast(uint16_t, lo) |
                ((uint32_t)__builtin_bit_cast(uint16_t, hi) << 16);
      }
      *reinterpret_cast<u32x2_t*>(op + d0) = u32x2_t{wv[0], wv[1]};
    }
  if constexpr (OSK) {
    if (wl == 0 && lane == 0 && P.a.n_computed)
      P.a.n_computed[(size_t)(n * P.Hq + h) * P.nb + i] = ncomp;
  }
  if constexpr (!PERSIST) break;
  }  // tiles of a persistent workgroup
}

int cu_count() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess ||
      hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
    return 256;
  return cus;
}

// Which heads' query blocks are walked together (unit_tile). Eight, one per XCD, so that each XCD's L2
// serves one head's pages at a time: with more, or with whole heads one after the other over all
// XCDs, long contexts lose that (16 / 16 heads, 64K tokens: 3.49 ms one at a time, 2.95 by eights, 3.21
// all at once). 1, 2 and 4 heads divide the XCDs in the same way; groups of 3, 5, 6 or 7 heads send every
// XCD through all of them and measure as one head at a time does at long contexts (dense, 4 query heads
// per KV head, 64K tokens: 3 heads 11.08 / 11.14 ms, 5 18.56 / 18.54, 6 22.2 / 21.9, 7 25.98 / 26.09) and
// better at short ones (8K: 247 / 208, 382 / 330, 440 / 385, 504 / 441 us).
// More where few tiles would leave CUs idle at the end (dense, 16 / 16 heads, 4K tokens 52 us by eights, 48
// all together). List walks: only the end of the grid has an idle end, so the last group takes the heads
// that are left once it holds two tiles per resident workgroup, and the groups in front of it stay at
// eight. When every group grew to four tiles per workgroup, batches of short sequences lost their L2 to it
// (prefill, 32 / 8 heads, 16 sequences of 16 blocks of 128 345 -> 335 us, 40 of 10 446 -> 440; 20 / 20 heads,
// 97 blocks 265 -> 250). Dense and masked walks keep growing every group, in whole eights: a tile's weight
// there is its position alone, and the heaviest first over all heads counts more (dense, 8 / 8 heads, 30
// sequences of 12 blocks: front groups of eight 196 us, all grown 186).
// Four where head pairs walk contexts of which eight heads' K and V exceed the 256 MiB last-level
// cache (by eights / by fours: 32 / 8 heads, prefill 768 blocks of 128 5.99 / 5.95 ms, 1024 10.27 / 10.22,
// masked 8.45 / 8.21; 16 / 8 heads, 1024 blocks, prefill 5.53 / 5.46, masked 7.78 / 7.33; dense the same
// within 0.2 %). Single heads, whose pages are read once per head, gain from eights there: 8 / 8 heads,
// 1024 blocks 3.37 and 3.44 ms.
void group_heads_of(AttnParams& P, const Shape& sh, int heads_per_wg, bool list, int resident) {
  const int heads = sh.B * sh.Hkv;
  const long long tiles = (long long)sh.nb * (sh.G / heads_per_wg);  // of one head
  const bool over_cache = 8LL * sh.L * kHeadDim * 4 > (256LL << 20);
  long long g = heads_per_wg == 2 && over_cache ? 4 : 8;
  while (!list && g < heads && g * tiles < 4LL * resident) g += 8;
  const long long last = list ? std::max(1LL, (2LL * resident + tiles - 1) / tiles) : 1;
  P.group_heads = (int)std::min<long long>(g, heads);
  P.n_front = heads > last ? (int)((heads - last) / P.group_heads) : 0;
  P.last_heads = heads - P.n_front * P.group_heads;
}

// The walking order of a pack, tiles_per_block tiles to a block of it. One sequence after the other keeps
// a sequence's pages in the L2 while its blocks are walked; only the end of the grid gains from heavy blocks
// first, so just the shortest sequences are ranked together, as many as hold two tiles per resident
// workgroup. All ranked together / this: 32 / 8 heads, 40 sequences of 10 blocks of 128 474 / 442 us, 100 of
// 5 522 / 487; all one after the other / this: 4 / 1 heads, 250, 100 and 17 blocks 391 / 364, 8 / 2 heads, 40,
// 39, 41 and five of 1 or 2 blocks 83 / 75.
PackOrder order_of(const SeqPack& sp, long long tiles_per_block, int resident) {
  PackOrder po;
  po.n = po.tail = sp.n;
  if (sp.n == 0) return po;
  auto len = [&](int q) { return sp.cu[q + 1] - sp.cu[q]; };
  int by_len[kMaxPackedSeqs];
  for (int q = 0; q < sp.n; ++q) by_len[q] = q;
  std::sort(by_len, by_len + sp.n,
            [&](int x, int y) { return len(x) != len(y) ? len(x) > len(y) : x < y; });
  for (long long tiles = 0; po.tail > 0 && tiles < 2LL * resident;)
    tiles += len(by_len[--po.tail]) * tiles_per_block;
  for (int k = 0, at = 0; k < kMaxPackedSeqs; ++k) {
    po.seq[k] = PackSeq{INT_MAX, 0, 0, 0.f};
    if (k >= sp.n) continue;
    const int q = by_len[k];
    po.seq[k] = PackSeq{at, sp.cu[q], len(q), sp.tau[q]};
    const int next = k >= po.tail && k + 1 < sp.n ? len(by_len[k + 1]) : 0;
    at += (k < po.tail ? 1 : k - po.tail + 1) * (len(q) - next);
  }
  return po;
}

template <int BLOCK, int HPW, int WALK, int PG>
void launch_t(const Shape& sh, AttnParams& P, const SeqPack& pack, int cus, hipStream_t stream) {
  using Cfg = TileCfg<BLOCK, HPW>;
  const int slots = (P.n_units + kNumXcd - 1) / kNumXcd * kNumXcd * (sh.G / HPW);
  const int resident = cus * Cfg::kWgPerCu;
  group_heads_of(P, sh, HPW, WALK == kWalkList, resident);
  P.pack = order_of(pack, (long long)P.last_heads * (sh.G / HPW), resident);
  // A grid that is resident as a whole, two or more workgroups to a CU: the CUs get their first
  // workgroups heaviest first, and their second ones lightest first, so that no CU holds the heavy tiles
  // of both rounds. All rounds heaviest first / folded, us: b = 64, 4 / 1 heads, 250 blocks, every block
  // kept 398 / 376, dense 331 / 309; b = 128, dense, 32 / 8 heads, 16 blocks 48.6 / 46.2, 8 / 2 heads, 64
  // blocks 167.5 / 156.8, prefill 91.8 / 87.2.
  P.fold = slots <= resident && slots > cus ? cus / kNumXcd : 0;
  // Head pairs. With b = 128 the two heads' waves share SIMDs, and the second head runs one phase behind
  // the first. With b = 64 they sit on different SIMDs, and it is another workgroup's wave that fills a
  // SIMD's gaps: there both heads run the same phase, so that a Q K^T half does not wait for the partner's
  // P V (packed 25K tokens, 16 / 4 heads 209.5 -> 203.6 us; 32 / 8 heads, 16K tokens 544 -> 520 us). Unless
  // nothing is skipped (every phase then has a P V half) and there is seldom another workgroup on the CU:
  // a resident grid, or a dense one of long walks that is not much larger. Same phase / one behind, us,
  // 4 / 1 heads: 250 blocks, every block kept 376 / 353, masked 183 / 174, dense 309 / 303; dense, 400
  // blocks (800 tiles) 661 / 644, 430 (860) 735 / 728, 440 (880) 767 / 778; 16 / 4 heads, 100 (800)
  // 169 / 173. With blocks skipped the same phase stays ahead, 198 / 212, and in short walks, where the
  // one phase more counts: 32 / 8 heads, 24 blocks, 30 % kept 27.9 / 28.4.
  const bool long_dense = WALK == kWalkDense && sh.nb >= 128;
  const bool behind =
      !P.a.skip_on && sh.nb >= 32 && 3LL * slots <= (long_dense ? 5LL : 3LL) * resident;
  if constexpr (WALK == kWalkList) {
    // A queue is of no use to a grid that is resident as a whole.
    if (P.a.queue != nullptr && slots > resident) {
      // As many workgroups as the LDS footprint admits, fed by the work queues: one per CU for head
      // pairs of b = 128, two for pairs of b = 64 (packed 25K tokens, 16 / 4 heads: 288 -> 230 us
      // against one).
      if (!P.a.queue_ready)
        hipLaunchKernelGGL(queue_reset, dim3(1), dim3(64), 0, stream, P.a.queue);
      hipLaunchKernelGGL((attention_kernel<BLOCK, HPW, WALK, PG, true, HPW == 2 && BLOCK == 128>),
                         dim3(resident), dim3(Cfg::kThreads), 0, stream, P);
      return;
    }
  }
  if (HPW == 2 && (BLOCK == 128 || behind))
    hipLaunchKernelGGL((attention_kernel<BLOCK, HPW, WALK, PG, false, HPW == 2>), dim3(slots),
                       dim3(Cfg::kThreads), 0, stream, P);
  else if constexpr (HPW == 1 || BLOCK == 64)
    hipLaunchKernelGGL((attention_kernel<BLOCK, HPW, WALK, PG, false, false>), dim3(slots),
                       dim3(Cfg::kThreads), 0, stream, P);
}

// Two heads per workgroup where the group size is even, unless there are few tiles, at most three
// head pairs for every two CUs: single heads then spread over the CUs more evenly, and a head's walk
// does not wait for its partner's. Pairs / single heads, us, query / KV heads, blocks of 128 (pairs):
//                  16/2, 24 (192)  64/8, 8 (256)  4/1, 120 (240)  8/4, 92 (368)  16/2, 56 (448)  8/4, 110 (440)
//   dense            70.1 / 59.5    32.8 / 27.1     319 / 275       291 / 276       190 / 194       363 / 363
//   masked, 40 %     48.3 / 42.2    30.5 / 26.6     196 / 171       154 / 147       109 / 107       182 / 178
//   prefill, 40 %    46.9 / 42.8    32.5 / 28.8     134 / 121       128 / 125       102 / 104       155 / 166
//   pages of 16      48.5 / 44.2    34.2 / 31.0     141 / 124       131 / 129       103 / 106       159 / 167
// 64-token blocks: list walks of up to one pair per CU only (prefill, 40 %, 32 / 8 heads, 16 blocks 23.1 /
// 22.5, 4 / 1 heads, 120 blocks 75.8 / 73.6). Elsewhere their pages are short, and fetching them once for
// both heads counts more (4 / 1 heads, 64 blocks: dense 72.7 / 75.3, masked 42.7 / 45.2).
template <int WALK, int PG>
void launch_shape(const Shape& sh, AttnParams& P, const SeqPack& pack, hipStream_t stream) {
  const int cus = cu_count();
  const long long pairs = (long long)P.n_units * (sh.G / 2);
  const bool few = sh.b == 128 ? 2 * pairs <= 3 * cus : WALK == kWalkList && pairs <= cus;
  const bool pair = (sh.G % 2) == 0 && !few;
  if (sh.b == 128) {
    if (pair) launch_t<128, 2, WALK, PG>(sh, P, pack, cus, stream);
    else launch_t<128, 1, WALK, PG>(sh, P, pack, cus, stream);
  } else {
    if (pair) launch_t<64, 2, WALK, PG>(sh, P, pack, cus, stream);
    else launch_t<64, 1, WALK, PG>(sh, P, pack, cus, stream);
  }
}

template <int WALK>
hipError_t launch(const Shape& sh, const AttnArgs& a, const SeqPack& pack, hipStream_t stream) {
  AttnParams P;
  P.a = a;
  P.Hq = sh.Hq;
  P.Hkv = sh.Hkv;
  P.L = sh.L;
  P.nb = sh.nb;
  P.G = sh.G;
  P.n_units = sh.B * sh.Hkv * sh.nb;
  P.scale = sh.scale;
  P.scale_log2 = sh.scale * 1.4426950408889634f;
  if constexpr (WALK == kWalkList) {
    if (a.pg.table == nullptr) launch_shape<kWalkList, kPgNone>(sh, P, pack, stream);
    else if ((1 << a.pg.log2_page) >= sh.b) launch_shape<kWalkList, kPgWhole>(sh, P, pack, stream);
    else launch_shape<kWalkList, kPgSplit>(sh, P, pack, stream);
  } else {
    launch_shape<WALK, kPgNone>(sh, P, pack, stream);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_osk_attention(const Shape& sh, const AttnArgs& a, const SeqPack& pack,
                                 hipStream_t stream) {
  return launch<kWalkList>(sh, a, pack, stream);
}

hipError_t launch_dense_attention(const Shape& sh, const AttnArgs& a, const SeqPack& pack,
                                 hipStream_t stream) {
  return launch<kWalkDense>(sh, a, pack, stream);
}

hipError_t launch_masked_attention(const Shape& sh, const AttnArgs& a, hipStream_t stream) {
  return launch<kWalkMask>(sh, a, SeqPack{}, stream);
}

}  // namespace cosa
