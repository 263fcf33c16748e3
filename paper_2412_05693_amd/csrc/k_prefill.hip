// K1: fused block-prefill attention with per-key score column sums, gfx950.
//
// One workgroup = one unit (sample, KV head) x one tile of 128/G block
// positions x all G query heads of the unit; wave w owns query head w % G and
// 32 consecutive positions.  For every query row the kernel computes the
// causal softmax attention over the unit's live cache entries plus the block's
// keys up to the row's own position (Sec. 3.1 block-wise prefill), writes the
// output, and adds the row's probabilities to a per-key partial sum (the
// sum_weights update of Sec. 3.2).  Per-workgroup partial sums land in the
// workspace; score_reduce_kernel folds them into the scores in a fixed order,
// so the result does not depend on scheduling.
//
// Exact column sums need every row's final softmax normaliser before any of
// its probabilities can be added to a key's sum.  The kernel therefore makes
// two sweeps over the key tiles:
//   sweep 1 (S^T = K Q^T orientation: one query per lane) -- online softmax,
//            O^T += V^T P^T on MFMA, final row max m and sum l;
//   sweep 2 (S = Q K^T orientation: one key per lane) -- recompute the logits,
//            P = exp2(z - m - log2 l) exactly, and sum over the rows held in
//            the lane's registers, so each lane ends with one key's column sum.
//
// Key tiles hold 64 rows from one source: the unit's cache rows [0, len0) first,
// then the block's input rows.  Tiles are copied global -> LDS by buffer loads
// that write LDS directly (no staging registers), tile t + 1's while tile t is
// worked on; rows past a source's range come back as zeros.  The 16-byte chunks of an LDS row are stored in an order
// that depends on the row (the copies read their source chunks in that order),
// so the MFMA operand reads are free of bank conflicts without padding.
// K rows of a 32-key sub-tile sit in LDS row order kappa (bits 2 and 3 of the
// row swapped), which makes the register layout of the S^T accumulator equal
// to the PV MFMA's B operand; V reaches the PV MFMA through gfx950's
// transposing LDS load (ds_read_b64_tr_b16).
#include <type_traits>

#include "bm_internal.h"

// a lambda of the kernel, always part of it: as a call (which the compiler would
// make of the larger float32 ones) it would move the registers it uses to memory
#define BM_LAMBDA __device__ __attribute__((always_inline))

namespace bm {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __bf16 __attribute__((vector_size(8))) bf16v4;   // operand type of the LDS transpose read
typedef __attribute__((address_space(3))) bf16v4 lds_bf16v4;
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
// the LDS object at byte `off` (an address kept as a number, so that it takes
// one register and an immediate offset)
template <typename T>
__device__ __forceinline__ T* lds_at(uint32_t off) { return (T*)(uintptr_t)off; }

constexpr float kNegInf = -__builtin_huge_valf();
constexpr float kPosInf = __builtin_huge_valf();
constexpr int kRsrcWord3 = 0x00020000;
constexpr float kRescaleLog2 = 8.0f;

// ---- prefill timeline (measurement builds: BM_PREFILL_TIMELINE) ----
// Thread 0 of each workgroup keeps the fields of include/bm_probe.h in
// registers and stores them at its end; in the ordinary build every use sits
// in an `if constexpr (kTimeline)` branch and nothing is emitted.
#ifdef BM_PREFILL_TIMELINE
constexpr bool kTimeline = true;
__device__ uint64_t g_timeline[(size_t)BM_TIMELINE_MAX_RECORDS * BM_TIMELINE_FIELDS];
__device__ __forceinline__ void timeline_store(int id, const uint64_t* tl) {
  if (threadIdx.x == 0 && id < BM_TIMELINE_MAX_RECORDS) {
#pragma unroll
    for (int i = 0; i < BM_TIMELINE_FIELDS; ++i) g_timeline[(size_t)id * BM_TIMELINE_FIELDS + i] = tl[i];
  }
}
#else
constexpr bool kTimeline = false;
__device__ __forceinline__ void timeline_store(int, const uint64_t*) {}
#endif
// the constant-rate real-time counter (read only in timeline builds)
__device__ __forceinline__ uint64_t tl_now() {
  if constexpr (kTimeline) return __builtin_amdgcn_s_memrealtime();
  return 0;
}

__device__ __forceinline__ int kappa(int m) {
  return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1);
}

// x of lane i combined with x of lane i ^ 32 through gfx950's cross-half swap
// (no LDS round trip); the swap returns the two values in the same order on
// both lanes, so both get bit-identical results
__device__ __forceinline__ float xhalf_max(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xhalf_sum(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  bf16x2 r = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, r);
}

// key index inside the 64-key tile held by accumulator register (i, j) of lane
// half h in S^T orientation, sub-tile st
__device__ __forceinline__ int st_key(int st, int i, int j, int h) {
  return 32 * st + 16 * (i >> 1) + 8 * h + 4 * (i & 1) + j;
}

template <bool BF16, int D>
struct Cfg {
  using E = typename std::conditional<BF16, uint16_t, float>::type;
  using qfrag_t = typename std::conditional<BF16, bf16x8, float>::type;
  using kfrag_t = typename std::conditional<BF16, bf16x8, f32x4>::type;   // one 16-byte read
  static constexpr int RB = D * (int)sizeof(E);          // bytes per K/V row
  static constexpr int CPR = RB / 16;                     // 16-byte chunks per row
  static constexpr int TILE_BYTES = kKeyTile * RB;        // one K or V tile in LDS
  static constexpr int RPS = 1024 / RB;                   // rows per 1 KB copy
  static constexpr int NCOPY = TILE_BYTES / 1024 / kWaves;   // copies per wave and tile
  static constexpr int QSTEPS = BF16 ? D / 16 : D / 2;   // MFMA K-steps over d
  static constexpr int MT = D / 32;                       // 32-row M-tiles of O^T
};


template <bool BF16, int D>
__device__ __forceinline__ f32x16 mfma_step(typename Cfg<BF16, D>::qfrag_t a,
                                            typename Cfg<BF16, D>::qfrag_t b, f32x16 c) {
  if constexpr (BF16) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
  }
}

// LDS rows are stored without padding; chunk c of row r sits at position
// c ^ swz(r) of its row, which spreads the chunks that one read instruction
// touches over the banks (a 256-byte line of them holds 256 / RB rows):
// K and output rows: 16 rows, the same chunk of each; V: rows 4 i .. 4 i + 3,
// the same 64 bytes of each.
template <bool BF16, int D>
__device__ __forceinline__ constexpr int swz_k(int r) {
  using C = Cfg<BF16, D>;
  return C::RB >= 256 ? r & 15 : (r >> 1) & 7;
}
template <bool BF16, int D>
__device__ __forceinline__ constexpr int swz_v(int r) {
  using C = Cfg<BF16, D>;
  return !BF16 ? 0 : C::RB >= 256 ? (r & 3) << 2 : ((r >> 1) & 1) << 2;
}

// Address in a K tile of the fragment of row n (and, 32 rows on, of row n + 32)
// for K-step kk, lane half h, from frag0 = k_frag0(n, h).  bf16: K-step kk
// contracts the 16-byte chunks 2 kk (lane half 0) and 2 kk + 1 (lane half 1) of
// d, so the two halves of a query row's load fall in one cache line
template <bool BF16, int D>
__device__ __forceinline__ int k_frag0(int n, int h) {
  using C = Cfg<BF16, D>;
  const int c = BF16 ? h : h * (C::CPR / 2);
  return n * C::RB + (c ^ swz_k<BF16, D>(n)) * 16;
}
// fp32: the same address rule for the chunk that holds K-steps 4 kk .. 4 kk + 3
template <bool BF16, int D>
__device__ __forceinline__ typename Cfg<BF16, D>::kfrag_t k_frag(const char* ks, int frag0, int kk) {
  return __builtin_bit_cast(typename Cfg<BF16, D>::kfrag_t,
                            *reinterpret_cast<const u32x4*>(ks + (frag0 ^ ((BF16 ? 32 : 16) * kk))));
}

struct Geo {
  int u, bi, hk, pt, w, lane, n, h, g, sub;
  int split;       // which of the launch's nsplit workgroups of this tile
  int pbase;       // first block position (relative to t0) of the workgroup
  int wrow0;       // first query row (relative to t0) of this wave
  int row;         // this lane's query row (relative to t0) in S^T orientation
  int wlast;       // last real query row of this wave
  bool qvalid;
  bool wave_active;
  bool works;      // some query row of this wave is real and no pad token
  int in_rows;     // block rows the workgroup reads: min(n_tok, pbase + PT)
  int ncf, nbt;    // whole cache tiles, block tiles
  int part;        // 1 if a partial cache tile follows the whole ones
  int nt;          // all tiles
  int nbu;         // block tiles that need no mask in this wave
  int pad;         // left pad tokens of the sample (positions < pad are pads)
  bool qpad;       // this lane's query row is a pad token
};

template <int G, bool PAD, bool SPLIT>
__device__ __forceinline__ Geo make_geo(const PrefillArgs& a) {
  Geo s;
  // Workgroups are dispatched round-robin over the 8 XCDs (each with its own
  // L2).  Renumber them so that consecutive logical ids -- the workgroups of
  // one unit -- land on the same XCD and share that unit's K/V in its L2.
  const int nwg = gridDim.x, L = blockIdx.x;
  const int q8 = nwg >> 3, r8 = nwg & 7, xcd = L & 7;
  int lin = xcd * q8 + min(xcd, r8) + (L >> 3);
  s.split = 0;
  if constexpr (SPLIT) {
    s.split = lin % a.nsplit;
    lin /= a.nsplit;
  }
  s.u = lin / a.npt_used;
  s.pt = lin - s.u * a.npt_used;
  s.bi = s.u / a.n_kv_heads;
  s.hk = s.u - s.bi * a.n_kv_heads;
  // the wave's number in a scalar register: what follows from it (rows, heads,
  // which tiles are masked) is then scalar work and scalar branches
  s.w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  s.lane = threadIdx.x & 63;
  s.n = s.lane & 31;
  s.h = s.lane >> 5;
  s.g = s.w % G;
  s.sub = s.w / G;
  constexpr int PT = kWaves * kRowsPerWave / G;
  s.pbase = s.pt * PT;
  s.wrow0 = s.pbase + s.sub * kRowsPerWave;
  s.row = s.wrow0 + s.n;
  s.qvalid = s.row < a.n_tok;
  s.wave_active = s.wrow0 < a.n_tok;
  s.wlast = min(a.n_tok - 1, s.wrow0 + kRowsPerWave - 1);
  s.in_rows = min(a.n_tok, s.pbase + PT);
  s.ncf = a.len0 / kKeyTile;
  s.nbt = (s.in_rows + kKeyTile - 1) / kKeyTile;
  s.part = a.len0 % kKeyTile != 0;
  s.nt = s.ncf + s.part + s.nbt;
  s.nbu = (s.wrow0 + 1) / kKeyTile;
  s.pad = PAD ? max(0, a.pad[s.bi]) : 0;
  s.works = s.wave_active && a.t0 + s.wlast >= s.pad;
  s.qpad = a.t0 + s.row < s.pad;
  return s;
}

// Where a tile comes from and which of its rows exist.
struct TileInfo {
  bool cache;      // rows from the unit's cache (else the block's input rows)
  int base;        // first source row of the tile
  int slot0;       // cache slot of the tile's row 0 (for the score sums)
  int valid;       // rows of the tile that exist
};

// tile t of sweep 1: the cache's rows in order, then the block's
__device__ __forceinline__ TileInfo tile_info(const PrefillArgs& a, const Geo& s, int t) {
  TileInfo ti;
  const int ntc = s.ncf + s.part;
  ti.cache = t < ntc;
  ti.base = (ti.cache ? t : t - ntc) * kKeyTile;
  ti.slot0 = ti.cache ? ti.base : a.len0 + ti.base;
  ti.valid = min(kKeyTile, (ti.cache ? a.len0 : s.in_rows) - ti.base);
  return ti;
}
// tile t of sweep 2, whose sums do not depend on the order: a partial cache tile
// comes last, so that the tiles without a mask are in one run
__device__ __forceinline__ TileInfo tile_info2(const PrefillArgs& a, const Geo& s, int t) {
  return tile_info(a, s, t < s.ncf ? t : t == s.nt - 1 && s.part ? s.ncf : t + s.part);
}

// does the wave see any key of the tile
__device__ __forceinline__ bool tile_active(const Geo& s, const TileInfo& ti) {
  return s.works && (ti.cache || ti.base <= s.wlast);
}

// Tiles of K (rows in kappa order) and V are copied into LDS with buffer loads
// that write LDS directly: wave w fills the NCOPY consecutive 1 KB pieces (RPS
// rows each) from NCOPY w on, lane i the 16-byte chunk i of each.  An
// instruction's immediate offset moves its LDS address and its source address
// alike, so up to four copies share one LDS base (the M0 register, whose change
// would have to wait for the copy before it) and a lane's source offset of copy j
// has the immediate taken off; kBias keeps it from going below zero.  The buffer
// resource starts kBias bytes before the tile's first source row and ends at the
// last row that exists (rows past it arrive as zeros); both come from scalar
// registers.
constexpr int kBias = 3072;

template <bool BF16, int D, bool K>
__device__ __forceinline__ int copy_offset(const Geo& s, int j) {
  using C = Cfg<BF16, D>;
  const int r = (s.w * C::NCOPY + j) * C::RPS + s.lane / C::CPR, p = s.lane % C::CPR;
  const int src = K ? (r & ~31) + kappa(r & 31) : r;
  return src * C::RB + (p ^ (K ? swz_k<BF16, D>(r) : swz_v<BF16, D>(r))) * 16 + kBias - 1024 * (j & 3);
}

// The wave's copies of one tile into the LDS tile at `dst`.  Written as assembly
// so that the compiler does not order the tile reads behind the copies in flight
// (it cannot tell the buffers apart once their choice is a run-time value):
// tile_fence() waits for a wave's copies, and the barrier behind it for everyone's.
// A load may read its resource five wait states after a vector instruction wrote one
// of those scalar registers (a reload of a spilled one is such an instruction), and the
// compiler does not count the states inside a block: s_mov and s_nop 3 are all five.
// M0 is a reserved register, so the compiler warns that it does not save it for a
// block that names it; no other code of these kernels uses M0 (checked on the built
// library by a test), and the warning is off for the three blocks alone.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int NCOPY>
__device__ __forceinline__ void copy_tile(uint32_t dst, u32x4 rsrc, const int (&off)[NCOPY], int w) {
  static_assert(NCOPY % 4 == 0 || NCOPY == 2, "copies per wave and tile");
  const uint32_t lds = __builtin_amdgcn_readfirstlane(dst + w * (NCOPY * 1024));
  if constexpr (NCOPY == 2) {
    asm volatile(
        "s_mov_b32 m0, %3\n\ts_nop 3\n\tbuffer_load_dwordx4 %0, %2, 0 offen lds\n\t"
        "buffer_load_dwordx4 %1, %2, 0 offen offset:1024 lds"
        ::"v"(off[0]), "v"(off[1]), "s"(rsrc), "s"(lds) : "m0");
  } else {
#pragma unroll
    for (int j = 0; j < NCOPY; j += 4)
      asm volatile(
          "s_mov_b32 m0, %5\n\ts_nop 3\n\tbuffer_load_dwordx4 %0, %4, 0 offen lds\n\t"
          "buffer_load_dwordx4 %1, %4, 0 offen offset:1024 lds\n\t"
          "buffer_load_dwordx4 %2, %4, 0 offen offset:2048 lds\n\t"
          "buffer_load_dwordx4 %3, %4, 0 offen offset:3072 lds"
          ::"v"(off[j]), "v"(off[j + 1]), "v"(off[j + 2]), "v"(off[j + 3]), "s"(rsrc),
          "s"(__builtin_amdgcn_readfirstlane(lds + 1024 * j)) : "m0");
  }
}

// 64 words, one from byte offset `off` of each lane, to LDS at `dst`
__device__ __forceinline__ void copy_words(uint32_t dst, u32x4 rsrc, int off) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 3\n\tbuffer_load_dword %0, %1, 0 offen lds"
               ::"v"(off), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane(dst)) : "m0");
}
#pragma clang diagnostic pop

// wait for the wave's copies; LDS may hold new tiles from here on
__device__ __forceinline__ void tile_fence() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <bool BF16, int D, int G, bool PAD, bool SPLIT>
__global__ void __launch_bounds__(kThreads, (BF16 || D == 64) ? 2 : 1) prefill_attn_kernel(PrefillArgs a) {
  // PAD: the launch has left padding (a separate instantiation, so the common
  // case carries none of its registers).  SPLIT: each position tile has a.nsplit
  // workgroups that all run sweep 1 and share what follows (see split_of)
  using C = Cfg<BF16, D>;
  using E = typename C::E;
  constexpr int RB = C::RB;
  // tiles that need no mask go through the interleaved loops, with left padding from
  // the block on for which the unit has no pad left
  constexpr bool FAST = BF16;
  // two K and two V tile buffers; parity t & 1 of tile t in sweep 1, (nt + t) & 1
  // in sweep 2
  __shared__ __attribute__((aligned(2 * C::TILE_BYTES))) char kv[4 * C::TILE_BYTES];
  char* const kbuf = kv;
  char* const vbuf = kv + 2 * C::TILE_BYTES;
  __shared__ float cs[3][kWaves][kKeyTile];
  // positions of the cached keys of tile t in pk_ring[t % 3] (left padding
  // only): a wave may still read tile t's when tile t + 1's are being fetched
  __shared__ int32_t pk_ring[3][kKeyTile];
  // the block's last query's weights per wave (TOVA's key)
  __shared__ float lws[3][kWaves][kKeyTile];
  uint64_t tl[BM_TIMELINE_FIELDS] = {};
  if constexpr (kTimeline) tl[BM_TL_ENTRY] = tl_now();
  Geo s = make_geo<G, PAD, SPLIT>(a);
  const int tid = threadIdx.x;
  auto stamp = [&](int field) BM_LAMBDA {
    if constexpr (kTimeline) tl[field] = tl_now();
  };
  auto timeline_end = [&]() BM_LAMBDA {
    if constexpr (kTimeline) {
      tl[BM_TL_END] = tl_now();
      // HW_ID (all 32 bits) and, above it, XCC_ID (hardware registers 4 and 20)
      tl[BM_TL_HW_ID] = (uint64_t)__builtin_amdgcn_s_getreg(0xF804) |
                        ((uint64_t)__builtin_amdgcn_s_getreg(0xF814) << 32);
      tl[BM_TL_ITEM] = ((uint64_t)s.u << 32) | (uint32_t)s.pt;
      tl[BM_TL_TILES] = (uint64_t)s.nt;
      timeline_store(blockIdx.x, tl);
    }
  };
  // end of a tile: wait for this wave's copies, then for every wave
  auto wait_and_sync = [&](int f_wait, int f_barrier) BM_LAMBDA {
    if constexpr (kTimeline) {
      const uint64_t a0 = tl_now();
      tile_fence();
      const uint64_t a1 = tl_now();
      __syncthreads();
      tl[f_wait] += a1 - a0;
      tl[f_barrier] += tl_now() - a1;
    } else {
      tile_fence();
      __syncthreads();
    }
  };

  constexpr int PT = kWaves * kRowsPerWave / G;   // block positions per workgroup

  // Left padding: past the pads, the smallest cached position tells whether the cache
  // still holds one (a score-ranked cut removes pads first: their scores are 0)
  // and, if not, the unmasked loops run.  With the skipped pad tiles and pad rows:
  // b=8, 40 heads, s=3584, up to 1024 pads (one prompt without), per prompt and in
  // turn with one former kernel: 1.044x -> 1.068x of its speed (1950 us)
  int pos_min = -1;
  if constexpr (PAD) {
    if (s.pad > 0 && a.t0 >= s.pad) {
      const int32_t* pc = a.pos + (int64_t)s.u * a.cap;
      pos_min = s.pad;
#pragma unroll 4
      for (int j = tid; j < a.len0; j += kThreads) pos_min = min(pos_min, pc[j]);
    }
  }

  // ---- append the workgroup's block rows to the cache tail (Sec. 3.2: new
  //      entries start with score 0; the score is written by score_reduce).
  //      The loads are issued here, with the query loads and the first tile
  //      copies behind them, and the stores follow the wait those need anyway,
  //      so the workgroup waits for memory once before its first tile. ----
  const int64_t plane = ((int64_t)s.bi * a.n_kv_heads + s.hk) * a.seq_ld;
  constexpr int NA = (PT * C::CPR + kThreads - 1) / kThreads;   // chunks per thread
  const int app_chunks = s.split == 0 ? (s.in_rows - s.pbase) * C::CPR : 0;
  u32x4 app_k[NA], app_v[NA];
  {
    const E* kin = static_cast<const E*>(a.kin);
    const E* vin = static_cast<const E*>(a.vin);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int c = tid + i * kThreads;
      if (c < app_chunks) {
        const int r = s.pbase + c / C::CPR, cc = c % C::CPR;
        const int64_t src = (plane + r) * D + cc * (16 / sizeof(E));
        app_k[i] = *reinterpret_cast<const u32x4*>(kin + src);
        app_v[i] = *reinterpret_cast<const u32x4*>(vin + src);
      }
    }
  }
  auto append_store = [&]() BM_LAMBDA {
    E* kc = static_cast<E*>(a.kc);
    E* vc = static_cast<E*>(a.vc);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
      const int c = tid + i * kThreads;
      if (c < app_chunks) {
        const int r = s.pbase + c / C::CPR, cc = c % C::CPR;
        const int64_t dst = ((int64_t)s.u * a.cap + a.len0 + r) * D + cc * (16 / sizeof(E));
        *reinterpret_cast<u32x4*>(kc + dst) = app_k[i];
        *reinterpret_cast<u32x4*>(vc + dst) = app_v[i];
      }
    }
    if (s.split != 0) return;
    for (int r = s.pbase + tid; r < s.in_rows; r += kThreads)
      a.pos[(int64_t)s.u * a.cap + a.len0 + r] = a.t0 + r;
  };

  // ---- row sources of the tiles (out-of-range rows read as zero) ----
  const uint64_t kc_base = (uint64_t)(static_cast<const E*>(a.kc) + (int64_t)s.u * a.cap * D);
  const uint64_t vc_base = (uint64_t)(static_cast<const E*>(a.vc) + (int64_t)s.u * a.cap * D);
  const uint64_t ki_base = (uint64_t)(static_cast<const E*>(a.kin) + plane * D);
  const uint64_t vi_base = (uint64_t)(static_cast<const E*>(a.vin) + plane * D);
  auto rsrc_of = [&](uint64_t p, int bytes) BM_LAMBDA {
    return u32x4{(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)p),
                 (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(p >> 32)) & 0xFFFFu,
                 (uint32_t)__builtin_amdgcn_readfirstlane(bytes), (uint32_t)kRsrcWord3};
  };
  auto tile_src = [&](const TileInfo& ti, bool kside) BM_LAMBDA {
    const uint64_t p = ti.cache ? (kside ? kc_base : vc_base) : (kside ? ki_base : vi_base);
    return rsrc_of(p + (uint64_t)(ti.base * RB) - kBias,
                   ((ti.cache ? a.len0 : s.in_rows) - ti.base) * RB + kBias);
  };
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_void*)kv;
  int koff[C::NCOPY], voff[C::NCOPY];
#pragma unroll
  for (int j = 0; j < C::NCOPY; ++j) {
    koff[j] = copy_offset<BF16, D, true>(s, j);
    voff[j] = copy_offset<BF16, D, false>(s, j);
  }
  const uint64_t pos_base = (uint64_t)(a.pos + (int64_t)s.u * a.cap);
  auto dma_k = [&](int par, const TileInfo& ti, int t) BM_LAMBDA {
    copy_tile(lds0 + par * C::TILE_BYTES, tile_src(ti, true), koff, s.w);
    if (PAD && s.pad > 0 && ti.cache && s.w == 0) {
      // the tile's key positions, in key order, next to the K rows
      const u32x4 r = rsrc_of(pos_base, a.len0 * 4);
      copy_words((uint32_t)(uintptr_t)(lds_void*)pk_ring[t % 3], r, (ti.base + s.lane) * 4);
    }
  };
  // bit k set: key k of tile ti is a pad token (cache keys through the LDS copy
  // of their positions); uniform across the workgroup
  auto pad_bits = [&](const TileInfo& ti, const int32_t* pk) BM_LAMBDA -> uint64_t {
    if (!PAD || s.pad == 0) return 0;
    if (ti.cache) return __ballot(pk[s.lane] < s.pad);
    const int n = min(max(s.pad - a.t0 - ti.base, 0), kKeyTile);
    return n >= 64 ? ~0ull : ((1ull << n) - 1);
  };
  auto dma_v = [&](int par, const TileInfo& ti) BM_LAMBDA {
    copy_tile(lds0 + (2 + par) * C::TILE_BYTES, tile_src(ti, false), voff, s.w);
  };

  // ---- query fragments: lane (n, h) holds row n; bf16: the d-chunks 2 kk + h
  //      (the order k_frag reads K in), fp32: d-range [h*D/2, (h+1)*D/2) ----
  typename C::qfrag_t qf[C::QSTEPS];
  {
    const int qh = s.hk * G + s.g;
    const E* q = static_cast<const E*>(a.q) +
                 (((int64_t)s.bi * a.n_heads + qh) * a.seq_ld + s.row) * D;
#pragma unroll
    for (int kk = 0; kk < C::QSTEPS; ++kk) {
      if constexpr (BF16) {
        const u32x4 w = s.qvalid ? *reinterpret_cast<const u32x4*>(q + 8 * (2 * kk + s.h))
                                 : u32x4{0, 0, 0, 0};
        qf[kk] = __builtin_bit_cast(bf16x8, w);
      } else {
        qf[kk] = s.qvalid ? q[s.h * (D / 2) + kk] : 0.0f;
      }
    }
  }

  stamp(BM_TL_QUERY_ISSUED);
  const int nt = s.nt;
  // sweep 2's tiles of this workgroup: n2 from lo2 on.  Of three or more workgroups
  // the first stores the outputs and the others make the sums; two share the tiles
  int lo2 = 0, n2 = nt;
  if constexpr (SPLIT) {
    const int first = a.nsplit > 2, parts = a.nsplit - first, k = s.split - first;
    lo2 = k < 0 ? 0 : nt * k / parts;
    n2 = k < 0 ? 0 : nt * (k + 1) / parts - lo2;
  }
  const float c2 = a.scale_log2;
  // the row this lane's causal mask uses (padding rows reuse the last real row)
  const int qrow = s.qvalid ? s.row : a.n_tok - 1;

  // logits of one tile: S^T (one query per lane) or S (one key per lane); the
  // K fragments of step kk + 1 are read while the MFMAs of step kk run
  const int frag0 = k_frag0<BF16, D>(s.n, s.h);
  auto qk_tile = [&](auto st_tag, const char* ks, f32x16* acc) BM_LAMBDA {
    constexpr bool ST = decltype(st_tag)::value;
    int f0 = frag0;
    asm volatile("" : "+v"(f0));   // the swizzled addresses are formed here, not kept
    acc[0] = f32x16{};
    acc[1] = f32x16{};
    constexpr int SPR = BF16 ? 1 : 4;   // K-steps per read
    typename C::kfrag_t kf[2][2];
    kf[0][0] = k_frag<BF16, D>(ks, f0, 0);
    kf[0][1] = k_frag<BF16, D>(ks + 32 * RB, f0, 0);
#pragma unroll
    for (int kr = 0; kr < C::QSTEPS / SPR; ++kr) {
      if (kr + 1 < C::QSTEPS / SPR) {
        kf[(kr + 1) & 1][0] = k_frag<BF16, D>(ks, f0, kr + 1);
        kf[(kr + 1) & 1][1] = k_frag<BF16, D>(ks + 32 * RB, f0, kr + 1);
      }
#pragma unroll
      for (int e = 0; e < SPR; ++e)
#pragma unroll
        for (int st = 0; st < 2; ++st) {
          typename C::qfrag_t kv;
          if constexpr (BF16) kv = kf[kr & 1][st];
          else kv = kf[kr & 1][st][e];
          acc[st] = ST ? mfma_step<BF16, D>(kv, qf[kr * SPR + e], acc[st])
                       : mfma_step<BF16, D>(qf[kr * SPR + e], kv, acc[st]);
        }
    }
    if constexpr (BF16) {
      // pin the order: the reads of step kk + 1 go out before the MFMAs of
      // step kk (left alone, the scheduler sinks each read to its MFMA)
      __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);   // DS reads
#pragma unroll
      for (int kk = 0; kk + 2 < C::QSTEPS; ++kk) {
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0); // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
    }
  };
  auto qk_st = [&](const char* ks, f32x16* acc) BM_LAMBDA { qk_tile(std::true_type{}, ks, acc); };
  auto qk_s = [&](const char* ks, f32x16* acc) BM_LAMBDA { qk_tile(std::false_type{}, ks, acc); };

  // ======================= sweep 1: online softmax + PV =======================
  f32x16 oacc[C::MT];
#pragma unroll
  for (int mt = 0; mt < C::MT; ++mt) oacc[mt] = f32x16{};
  float m_run = kNegInf, l_run = 0.0f;

  // left padding: a real query row sees no pad key (a pad row keeps its causal
  // keys; its output and score contributions are dropped later).  The lane's
  // keys all have bit 3 equal to h, so the pad bits are shifted once.
  auto hide_pads = [&](f32x16* sacc, uint64_t padk) BM_LAMBDA {
    const uint64_t hide = s.qpad ? 0 : (padk >> (8 * s.h));
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if ((hide >> st_key(st, r >> 2, r & 3, 0)) & 1) sacc[st][r] = kNegInf;
  };

  // logits and P of the tile in work.  bf16: P packed, half by half, as the PV
  // MFMA's B operand; fp32: P replaces the logits in sl
  f32x16 sl[2];
  u32x4 pp[2][2];
  auto pack_p = [&](int half) BM_LAMBDA {
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        pp[half][q][i] = pack_bf16x2(sl[half][8 * q + 2 * i], sl[half][8 * q + 2 * i + 1]);
  };
  // The reference m_run moves only when some row of the wave sees a logit more
  // than kRescaleLog2 above it: the probabilities stay below 2^kRescaleLog2
  // (exact in fp32, fine in bf16) and the O rescale is rare.
  auto raise_max = [&](float tmax) BM_LAMBDA {
    if (__ballot(tmax * c2 > m_run + kRescaleLog2) != 0) {
      const float m_new = fmaxf(m_run, tmax * c2);
      // (a padded row that has seen no key yet keeps m = -inf: nothing to scale)
      const float alpha = PAD && m_new == kNegInf ? 1.0f : __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
      m_run = m_new;
#pragma unroll
      for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[mt][r] *= alpha;
    }
  };
  // What the logits are taken against.  With left padding a row's first tiles can be
  // all pad keys: m_run is still -inf there and every logit is -inf, so subtract 0 to
  // get p = 0, not NaN.  A launch with padding keeps to that after its pads are gone
  // (logits that overflow to -inf weigh nothing there); without padding every row
  // sees a key in its first tile.
  auto reference = [&]() BM_LAMBDA { return PAD && m_run == kNegInf ? 0.0f : m_run; };
  auto exp_tile = [&](float m_sub) BM_LAMBDA {
    float psum = 0.0f;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(fmaf(sl[st][r], c2, -m_sub));
        sl[st][r] = p;
        psum += p;
      }
    l_run += psum;
    if constexpr (BF16) {
      pack_p(0);
      pack_p(1);
    }
  };
  auto softmax_tile = [&](auto mask_tag, const TileInfo& ti) BM_LAMBDA {
    constexpr bool MASK = decltype(mask_tag)::value;
    f32x16* sacc = sl;
    if constexpr (MASK) {
      // key k of the tile is visible iff k <= lim_k
      // (the lane half's 8 h comes off the limit, so each key compares against
      // a constant and no register holds its index)
      const int lim_k = (ti.cache ? ti.valid - 1 : qrow - ti.base) - 8 * s.h;
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          sacc[st][r] = st_key(st, r >> 2, r & 3, 0) <= lim_k ? sacc[st][r] : kNegInf;
    }
    // tile max on the raw logits (the scale is positive), then one fma per exp2
    float tmax = kNegInf;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sacc[st][r]);
    raise_max(xhalf_max(tmax));
    exp_tile(reference());
  };

  // A operand (V^T) of the PV MFMA: lane (n, h) needs V[key][32 mt + n] for the
  // 8 keys 16 ks4 + 8 h + e of P's k-slots.  The LDS transpose load gives lane i
  // of a 16-lane group column i of the 4 x 16 block formed by the group's lanes
  // 4r..4r+3 (row r), so lane 4r + c points at V[key0 + r][d0 + 4c] and receives
  // V[key0 + 0..3][d0 + i].  (The swizzle of a row depends on row % 4 alone;
  // rows of 16 ks4 and 4 further on have the same.)
  const int j16 = s.lane & 15, dhalf = (s.lane >> 4) & 1;
  const int vrow = 8 * s.h + (j16 >> 2);
  const int vbase = vrow * RB + 16 * swz_v<BF16, D>(vrow) + (16 * dhalf + 4 * (j16 & 3)) * 2;
  auto v_frag = [&](const char* vs, int vb, int ks4, int mt) BM_LAMBDA {
    const char* p = vs + (vb ^ (64 * mt)) + 16 * ks4 * RB;
    const bf16v4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16v4*)p);
    const bf16v4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16v4*)(p + 4 * RB));
    const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
    return u32x4{l2.x, l2.y, h2.x, h2.y};
  };
  typedef __attribute__((ext_vector_type(C::MT))) float vrow_t;
  // O^T += V^T P^T of one tile
  auto pv_tile = [&](const char* vs) BM_LAMBDA {
    if constexpr (BF16) {
      int vb = vbase;
      asm volatile("" : "+v"(vb));
      // the reads of K-step ks4 + 1 are issued before the MFMAs of step ks4
      u32x4 vf[2][C::MT];
#pragma unroll
      for (int mt = 0; mt < C::MT; ++mt) vf[0][mt] = v_frag(vs, vb, 0, mt);
#pragma unroll
      for (int ks4 = 0; ks4 < 4; ++ks4) {
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt)
          if (ks4 + 1 < 4) vf[(ks4 + 1) & 1][mt] = v_frag(vs, vb, ks4 + 1, mt);
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt)
          oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8, vf[ks4 & 1][mt]),
              __builtin_bit_cast(bf16x8, pp[ks4 >> 1][ks4 & 1]), oacc[mt], 0, 0, 0);
      }
    } else {
#pragma unroll
      for (int st = 0; st < 2; ++st)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          // M-tile mt, row n stands for d = MT n + mt, so that a lane's values of
          // all M-tiles are neighbours: one read per key
          const int key = st_key(st, r >> 2, r & 3, s.h);
          const vrow_t vv = *reinterpret_cast<const vrow_t*>(vs + key * RB + s.n * (4 * C::MT));
#pragma unroll
          for (int mt = 0; mt < C::MT; ++mt)
            oacc[mt] = __builtin_amdgcn_mfma_f32_32x32x2f32(vv[mt], sl[st][r], oacc[mt], 0, 0, 0);
        }
    }
  };

  // One step of the interleaved loop: QK^T of tile t (into zn), the softmax of
  // tile t - 1 (zo, whose running maximum is settled) and its PV product.
  // What bounds it: per tile and wave 1024 cycles of MFMA (32 of 32 cycles) beside the
  // softmax's VALU work and the operands' LDS reads; two waves per SIMD cover each
  // other's phases only in part (b=64 s=4096, bound 512: counters put the matrix pipe
  // at 40% of a launch's cycles, 30% with the phases one after the other, and the clock
  // at 2.0 of 2.4 GHz; a tile of this sweep takes 1.92 us with two workgroups on a
  // compute unit, 2.16 before).  So the order is pinned, MFMA by MFMA: the QK MFMAs
  // with 24 of a lane's 32 logits between them, then the PV MFMAs with the last 8
  // and the maximum of zn.  VALU work is staged over three places (x = logit -
  // reference, e = exp2, sum and pack), so that no instruction waits for the one
  // before it; operand reads go out kAhead MFMAs early.  Sums keep the order of
  // exp_tile.  Per prompt, with the copies' shared LDS base: full cache b=4 s=8192
  // 2702 -> 2582 us, b=1 s=4096 556 -> 528 us, b=256 s=2048 2% faster.
  auto interleaved_step = [&](f32x16 (&zn)[2], const f32x16 (&zo)[2], uint32_t (&ka)[C::QSTEPS],
                              uint32_t (&va)[C::MT]) BM_LAMBDA {
    if constexpr (FAST) {
      constexpr int NI = C::QSTEPS, NQ = 2 * NI, NP = 4 * C::MT, kAhead = 3, NB = kAhead + 1;
      bf16x8 kf[NB];
      u32x4 vf[NB];
      auto k_fetch = [&](int j) BM_LAMBDA {
        kf[j % NB] = __builtin_bit_cast(bf16x8, *lds_at<lds_u32x4>(ka[j % NI] + (j / NI) * 32 * RB));
      };
      auto v_fetch = [&](int j) BM_LAMBDA {
        const int ks4 = j / C::MT, mt = j % C::MT;
        const bf16v4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(lds_at<lds_bf16v4>(va[mt] + 16 * ks4 * RB));
        const bf16v4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(lds_at<lds_bf16v4>(va[mt] + (16 * ks4 + 4) * RB));
        const u32x2 l2 = __builtin_bit_cast(u32x2, lo), h2 = __builtin_bit_cast(u32x2, hi);
        vf[j % NB] = u32x4{l2.x, l2.y, h2.x, h2.y};
      };
      float x[2][2], e[2][2], psum = 0.0f;
      const float m_sub = reference();
      auto args = [&](int p) BM_LAMBDA {   // pair p: logits 2 p, 2 p + 1 of the lane
#pragma unroll
        for (int l = 0; l < 2; ++l) x[p & 1][l] = fmaf(zo[p / 8][2 * (p % 8) + l], c2, -m_sub);
      };
      auto exps = [&](int p) BM_LAMBDA {
#pragma unroll
        for (int l = 0; l < 2; ++l) e[p & 1][l] = __builtin_amdgcn_exp2f(x[p & 1][l]);
      };
      auto sums = [&](int p) BM_LAMBDA {
        psum += e[p & 1][0];
        psum += e[p & 1][1];
        pp[p / 8][(p / 4) & 1][p & 3] = pack_bf16x2(e[p & 1][0], e[p & 1][1]);
      };
      auto pair = [&](int p) BM_LAMBDA {
        exps(p);
        if (p > 0) sums(p - 1);
        if (p + 1 < 16) args(p + 1);
      };
#pragma unroll
      for (int j = 0; j < kAhead; ++j) k_fetch(j);
      args(0);
#pragma unroll
      for (int j = 0; j < NQ; ++j) {
        __builtin_amdgcn_sched_barrier(0);
        zn[j / NI] = mfma_step<BF16, D>(kf[j % NB], qf[j % NI], j % NI == 0 ? f32x16{} : zn[j / NI]);
        __builtin_amdgcn_sched_barrier(0);
        if (j + kAhead < NQ)
          k_fetch(j + kAhead);
        else
          v_fetch(j + kAhead - NQ);
#pragma unroll
        for (int p = 0; p < 12; ++p)
          if (p * NQ / 12 == j) pair(p);
      }
      float tmax = kNegInf;
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        __builtin_amdgcn_sched_barrier(0);
        oacc[j % C::MT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            __builtin_bit_cast(bf16x8, vf[j % NB]),
            __builtin_bit_cast(bf16x8, pp[j / (2 * C::MT)][(j / C::MT) & 1]), oacc[j % C::MT], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (j + kAhead < NP) v_fetch(j + kAhead);
#pragma unroll
        for (int p = 12; p < 16; ++p)
          if ((p - 12) * NP / 8 == j) pair(p);
        if (NP / 2 == j) sums(15);
#pragma unroll
        for (int r = 0; r < 32 / NP; ++r)
          tmax = fmaxf(tmax, zn[j / (NP / 2)][(j % (NP / 2)) * (32 / NP) + r]);
      }
      __builtin_amdgcn_sched_barrier(0);
      l_run += psum;
      raise_max(xhalf_max(tmax));
    }
  };

  // prologue: K(0) lands in LDS
  dma_k(0, tile_info(a, s, 0), 0);
  stamp(BM_TL_COPIES_ISSUED);
  tile_fence();
  append_store();
  if constexpr (PAD) {
    // no pad among the unit's keys and the block's rows: from here on as without padding
    const int pads_left = __syncthreads_or(pos_min < s.pad);
    s.pad = __builtin_amdgcn_readfirstlane(pads_left ? s.pad : 0);
  } else {
    __syncthreads();
  }
  stamp(BM_TL_FIRST_TILE);
  // Step t: K(t) and V(t-1) are in LDS; K(t+1) and V(t) are fetched meanwhile
  // (last step: sweep 2's first K tile; its position ring slot is free, nobody
  // reads tile nt - 3's any more).
  auto fetch1 = [&](int t) BM_LAMBDA {
    const uint64_t issue0 = tl_now();
    const int par = t & 1;
    if (t + 1 < nt)
      dma_k(par ^ 1, tile_info(a, s, t + 1), t + 1);
    else if (SPLIT ? n2 > 0 : a.accumulate != 0)
      dma_k(par ^ 1, tile_info2(a, s, lo2), nt);
    dma_v(par, tile_info(a, s, t));
    if constexpr (kTimeline) tl[BM_TL_S1_COPY_ISSUE] += tl_now() - issue0;
  };
  bool p_live = false;   // P of the tile before waits for its PV product
  // one step with running maxima: PV of tile t - 1, then tile t's logits and P
  auto sweep1_step = [&](auto mask_tag, int t) BM_LAMBDA {
    const int par = t & 1;
    const TileInfo ti = tile_info(a, s, t);
    fetch1(t);
    if (p_live) pv_tile(vbuf + (par ^ 1) * C::TILE_BYTES);
    p_live = !decltype(mask_tag)::value || tile_active(s, ti);
    // a tile of pad keys alone adds nothing to a real row, and pad rows are dropped
    const uint64_t padk = PAD ? pad_bits(ti, pk_ring[t % 3]) : 0;
    if (PAD && padk == ~0ull) p_live = false;
    if (p_live) {
      qk_st(kbuf + par * C::TILE_BYTES, sl);
      if constexpr (PAD) {
        if (padk) hide_pads(sl, padk);
      }
      softmax_tile(mask_tag, ti);
    }
    wait_and_sync(BM_TL_S1_WAIT, BM_TL_S1_BARRIER);
  };
  // Runs of tiles without a mask and the masked ones after each: the whole cache
  // tiles and a partial one, then the block's tiles up to the diagonal (one run
  // in all when no partial tile lies between).
  int t1 = 0;
#pragma nounroll
  for (int run = 0; t1 < nt; ++run) {
    const bool split = s.part && run == 0;
    const int run_end = !s.works ? t1 : split ? s.ncf : s.ncf + s.part + s.nbu;
    if constexpr (FAST) {
      if (t1 < run_end && (!PAD || s.pad == 0)) {
        fetch1(t1);
        if (p_live) pv_tile(vbuf + ((t1 & 1) ^ 1) * C::TILE_BYTES);
        qk_st(kbuf + (t1 & 1) * C::TILE_BYTES, sl);
        float tmax = kNegInf;
#pragma unroll
        for (int st = 0; st < 2; ++st)
#pragma unroll
          for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, sl[st][r]);
        raise_max(xhalf_max(tmax));
        wait_and_sync(BM_TL_S1_WAIT, BM_TL_S1_BARRIER);
        // operand addresses: K of parity t & 1, V of the other one (the buffers
        // of the two parities differ in one address bit)
        uint32_t ka[C::QSTEPS], va[C::MT];
#pragma unroll
        for (int i = 0; i < C::QSTEPS; ++i)
          ka[i] = lds0 + (t1 & 1) * C::TILE_BYTES + (uint32_t)(frag0 ^ (32 * i));
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt)
          va[mt] = lds0 + (2 + ((t1 & 1) ^ 1)) * C::TILE_BYTES + (uint32_t)(vbase ^ (64 * mt));
        auto step = [&](f32x16 (&zn)[2], const f32x16 (&zo)[2], int t) BM_LAMBDA {
          fetch1(t);
#pragma unroll
          for (int i = 0; i < C::QSTEPS; ++i) ka[i] ^= C::TILE_BYTES;
#pragma unroll
          for (int mt = 0; mt < C::MT; ++mt) va[mt] ^= C::TILE_BYTES;
          interleaved_step(zn, zo, ka, va);
          wait_and_sync(BM_TL_S1_WAIT, BM_TL_S1_BARRIER);
        };
        f32x16 sm[2];   // logits alternate between sl and sm
        for (++t1; t1 + 1 < run_end; t1 += 2) {
          step(sm, sl, t1);
          step(sl, sm, t1 + 1);
        }
        if (t1 < run_end) {
          step(sm, sl, t1);
          sl[0] = sm[0];
          sl[1] = sm[1];
          ++t1;
        }
        // the run's last tile: P (its PV product belongs to the next step)
        exp_tile(reference());
        p_live = true;
      }
    }
    if constexpr (!FAST || PAD)
      for (; t1 < run_end; ++t1) sweep1_step(std::false_type{}, t1);
    const int masked_end = split ? s.ncf + 1 : nt;
    for (; t1 < masked_end; ++t1) sweep1_step(std::true_type{}, t1);
  }
  if (p_live) pv_tile(vbuf + ((nt - 1) & 1) * C::TILE_BYTES);
  if constexpr (BF16) __syncthreads();   // the V buffers are free for the output rows
  stamp(BM_TL_SWEEP1_END);

  // ---- finish rows: normalise, store O, row log-sum-exp (log2 units) ----
  const float l_tot = xhalf_sum(l_run);
  float lse2 = kPosInf;
  if (s.wave_active) {
    const float inv = 1.0f / l_tot;
    lse2 = s.qvalid && !s.qpad ? m_run + __builtin_amdgcn_logf(l_tot) : kPosInf;
    // a pad row has no output (zeros)
    const float sc = s.qpad ? 0.0f : inv;
    if constexpr (BF16) {
      // The wave's 32 output rows are contiguous in memory (one head, 32
      // consecutive positions).  They go through LDS -- the V buffers are
      // idle once sweep 1 is over; each wave uses its own 32-row region (rows
      // swizzled like K's) -- so the stores are whole 1 KB runs instead of 16
      // bytes per row per instruction.
      static_assert(kWaves * kRowsPerWave * RB == 2 * C::TILE_BYTES, "the waves' rows fill the V buffers");
      char* ost = vbuf + s.w * (kRowsPerWave * RB);
#pragma unroll
      for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d0 = 32 * mt + 8 * i + 4 * s.h;
          const u32x2 w = {pack_bf16x2(oacc[mt][4 * i + 0] * sc, oacc[mt][4 * i + 1] * sc),
                           pack_bf16x2(oacc[mt][4 * i + 2] * sc, oacc[mt][4 * i + 3] * sc)};
          *reinterpret_cast<u32x2*>(ost + s.n * RB + ((d0 * 2) ^ (16 * swz_k<BF16, D>(s.n)))) = w;
        }
      // the output row's address is computed here rather than kept from the
      // query load (which would hold two registers through both sweeps)
      int orow0 = s.wrow0, ohead = s.bi * a.n_heads + s.hk * G + s.g;
      asm volatile("" : "+v"(orow0), "+v"(ohead));
      char* o = reinterpret_cast<char*>(static_cast<E*>(a.o) + ((int64_t)ohead * a.seq_ld + orow0) * D);
      constexpr int RUNS = kRowsPerWave * RB / 1024;   // 1 KB runs per wave
      constexpr int RPR = 1024 / RB;                   // rows per run
#pragma unroll
      for (int j = 0; j < RUNS; ++j) {
        const int r = RPR * j + s.lane / (RB / 16), c = s.lane % (RB / 16);
        const u32x4 v =
            *reinterpret_cast<const u32x4*>(ost + r * RB + 16 * (c ^ swz_k<BF16, D>(r)));
        if (s.wrow0 + r < a.n_tok && s.split == 0)
          *reinterpret_cast<u32x4*>(o + (int64_t)r * RB + c * 16) = v;
      }
    } else if (s.qvalid && s.split == 0) {
      int orow = s.row, ohead = s.bi * a.n_heads + s.hk * G + s.g;
      asm volatile("" : "+v"(orow), "+v"(ohead));
      E* o = static_cast<E*>(a.o) + ((int64_t)ohead * a.seq_ld + orow) * D;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r >> 2) + 4 * s.h + (r & 3);
        vrow_t x;
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) x[mt] = oacc[mt][r] * sc;
        *reinterpret_cast<vrow_t*>(o + C::MT * row) = x;
      }
    }
  }

  // ======================= sweep 2: exact column sums ========================
  // (skipped when the caller asked for outputs only)
  stamp(BM_TL_OUTPUT_STORED);
  if (SPLIT ? n2 == 0 : !a.accumulate) {
    timeline_end();
    return;
  }
  // S orientation: lane (n, h) holds key n of a 32-key sub-tile and rows
  // 8i + 4h + j of the wave's 32 rows in accumulator register 4i + j.
  float lse_r[16];
#pragma unroll
  for (int r = 0; r < 16; ++r) lse_r[r] = __shfl(lse2, 8 * (r >> 2) + 4 * s.h + (r & 3));
  float* partial = a.partial + ((int64_t)s.u * a.npt_stride + s.pt) * a.cap;
  // TOVA: the workgroup holding the block's last row also keeps that row's
  // weights (summed over the heads) for every key; its waves for that row find
  // it in accumulator register ri of lane half hr
  const int last_row = a.n_tok - 1;
  const bool wg_last = a.lastw && s.pbase <= last_row && last_row < s.pbase + PT;
  const bool wave_last = wg_last && s.wrow0 <= last_row && last_row < s.wrow0 + kRowsPerWave;
  const int rl = last_row - s.wrow0;
  const int ri = 4 * (rl >> 3) + (rl & 3), hr = (rl >> 2) & 1;
  float lse_last = lse_r[0];
#pragma unroll
  for (int r = 1; r < 16; ++r) lse_last = r == ri ? lse_r[r] : lse_last;

  auto sweep2_tile = [&](auto mask_tag, f32x16* acc, const TileInfo& ti, float (*cs)[kKeyTile]) BM_LAMBDA {
    constexpr bool MASK = decltype(mask_tag)::value;
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const int key = 32 * st + kappa(s.n);
      float csum = 0.0f;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float x = fmaf(acc[st][r], c2, -lse_r[r]);
        if constexpr (MASK) {
          const int qr = s.wrow0 + 8 * (r >> 2) + 4 * s.h + (r & 3);
          const int lim_k = ti.cache ? ti.valid - 1 : qr - ti.base;
          x = key <= lim_k ? x : kNegInf;
        }
        csum += __builtin_amdgcn_exp2f(x);
      }
      csum = xhalf_sum(csum);
      if (s.h == 0) cs[s.w][key] = csum;
    }
  };

  stamp(BM_TL_SWEEP2_START);
  // Step t: K(t) is in LDS (sweep 1's last step fetched K(0)); K(t+1) is fetched
  // meanwhile.  After the step's barrier tile t - 1's sums of all waves are in cs.
  auto fetch2 = [&](int t) BM_LAMBDA {
    if (t + 1 < n2) dma_k((nt + t + 1) & 1, tile_info2(a, s, lo2 + t + 1), nt + t + 1);
  };
  // add the waves' sums of tile t (the waves take turns)
  auto store_sums = [&](int t) BM_LAMBDA {
    const TileInfo ti = tile_info2(a, s, lo2 + t);
    if (s.w == (t & (kWaves - 1)) && s.lane < ti.valid) {
      float acc = 0.0f;
#pragma unroll
      for (int w = 0; w < kWaves; ++w) acc += cs[t % 3][w][s.lane];
      partial[ti.slot0 + s.lane] = acc;
      if (wg_last) {
        float lw = 0.0f;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) lw += lws[t % 3][w][s.lane];
        a.lastw[(int64_t)s.u * a.cap + ti.slot0 + s.lane] = lw;
      }
    }
  };
  auto sweep2_step = [&](auto mask_tag, int t) BM_LAMBDA {
    const TileInfo ti = tile_info2(a, s, lo2 + t);
    float (*ct)[kKeyTile] = cs[t % 3];
    f32x16* cur = sl;
    fetch2(t);
    const uint64_t padk = PAD ? pad_bits(ti, pk_ring[(nt + t) % 3]) : 0;
    if ((!decltype(mask_tag)::value || tile_active(s, ti)) && !(PAD && padk == ~0ull)) {
      qk_s(kbuf + ((nt + t) & 1) * C::TILE_BYTES, cur);
      sweep2_tile(mask_tag, cur, ti, ct);
      if constexpr (PAD) {
        // a pad key is visible to no real row (pad rows add nothing: lse = +inf)
        if (padk && s.h == 0) {
#pragma unroll
          for (int st = 0; st < 2; ++st) {
            const int key = 32 * st + kappa(s.n);
            if ((padk >> key) & 1) ct[s.w][key] = 0.0f;
          }
        }
      }
    } else if (s.lane < 32) {
      ct[s.w][s.lane] = 0.0f;
      ct[s.w][32 + s.lane] = 0.0f;
    }
    if (wg_last) {
      // the last row sees every key of the tile (pads aside)
#pragma unroll
      for (int st = 0; st < 2; ++st) {
        const int key = 32 * st + kappa(s.n);
        float v = 0.0f;
        if (wave_last && tile_active(s, ti)) {
          float z = cur[st][0];
#pragma unroll
          for (int r = 1; r < 16; ++r) z = r == ri ? cur[st][r] : z;
          v = s.h == hr ? __builtin_amdgcn_exp2f(fmaf(z, c2, -lse_last)) : 0.0f;
          v = xhalf_sum(v);
          if (PAD && ((padk >> key) & 1)) v = 0.0f;
        }
        if (s.h == 0) lws[t % 3][s.w][key] = v;
      }
    }
    wait_and_sync(BM_TL_S2_WAIT, BM_TL_S2_BARRIER);
    if (t > 0) store_sums(t - 1);
  };
  // the sums of one key half of tile t by themselves (z: its logits): the first half
  // before the interleaved loop and the last one behind it
  auto sums_half = [&](const f32x16& z, int half, int t) BM_LAMBDA {
    float csum = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) csum += __builtin_amdgcn_exp2f(fmaf(z[r], c2, -lse_r[r]));
    csum = xhalf_sum(csum);
    if (s.h == 0) cs[t % 3][s.w][32 * half + kappa(s.n)] = csum;
  };
  // one tile of the interleaved loop: half by half, QK^T of tile t and the sums
  // of the half before it
  auto interleaved_tile2 = [&](uint32_t (&ka)[C::QSTEPS], int t) BM_LAMBDA {
    if constexpr (FAST) {
      constexpr int NI = C::QSTEPS, LPI = 16 / NI, kAhead = 3, NB = kAhead + 1;
      bf16x8 kf[NB];
      auto fetch = [&](int j) BM_LAMBDA {
        kf[j % NB] = __builtin_bit_cast(bf16x8, *lds_at<lds_u32x4>(ka[j % NI] + (j / NI) * 32 * RB));
      };
#pragma unroll
      for (int j = 0; j < kAhead; ++j) fetch(j);
      float csum[2] = {0.0f, 0.0f};
#pragma unroll
      for (int j = 0; j < 2 * NI; ++j) {
        const int u = j / NI, i = j % NI;
        __builtin_amdgcn_sched_barrier(0);
        if (j + kAhead < 2 * NI) fetch(j + kAhead);
#pragma unroll
        for (int l = 0; l < LPI; ++l)
          csum[u] += __builtin_amdgcn_exp2f(fmaf(sl[u ^ 1][i * LPI + l], c2, -lse_r[i * LPI + l]));
        __builtin_amdgcn_sched_barrier(0);
        sl[u] = mfma_step<BF16, D>(qf[i], kf[j % NB], i == 0 ? f32x16{} : sl[u]);
      }
      __builtin_amdgcn_sched_barrier(0);
      csum[0] = xhalf_sum(csum[0]);
      csum[1] = xhalf_sum(csum[1]);
      if (s.h == 0) {
        cs[(t - 1) % 3][s.w][32 + kappa(s.n)] = csum[0];
        cs[t % 3][s.w][kappa(s.n)] = csum[1];
      }
    }
  };
  // tiles without a mask: the whole cache tiles and the block's up to the diagonal
  const int nun2 = s.works ? min(max(s.ncf + s.nbu - lo2, 0), n2) : 0;
  int t2 = 0;
  if (FAST && (!PAD || s.pad == 0) && !wg_last && nun2 > 0) {
    fetch2(0);
    qk_s(kbuf + (nt & 1) * C::TILE_BYTES, sl);
    sums_half(sl[0], 0, 0);
    wait_and_sync(BM_TL_S2_WAIT, BM_TL_S2_BARRIER);
    uint32_t ka[C::QSTEPS];
#pragma unroll
    for (int i = 0; i < C::QSTEPS; ++i)
      ka[i] = lds0 + (nt & 1) * C::TILE_BYTES + (uint32_t)(frag0 ^ (32 * i));
    for (t2 = 1; t2 < nun2; ++t2) {
      fetch2(t2);
#pragma unroll
      for (int i = 0; i < C::QSTEPS; ++i) ka[i] ^= C::TILE_BYTES;
      interleaved_tile2(ka, t2);
      wait_and_sync(BM_TL_S2_WAIT, BM_TL_S2_BARRIER);
      store_sums(t2 - 1);
    }
    sums_half(sl[1], 1, t2 - 1);
  }
  for (; t2 < nun2; ++t2) sweep2_step(std::false_type{}, t2);
  for (; t2 < n2; ++t2) sweep2_step(std::true_type{}, t2);
  __syncthreads();
  store_sums(n2 - 1);
  timeline_end();
}

// Fold the per-workgroup partial column sums into the scores, in workgroup
// order: score[j] = (j < len0 ? score[j] : 0) + sum over workgroups that saw j
// (without accumulation: new entries get 0, older scores stay).
// Grid: (units, slot chunks of 256); every thread owns one slot.  The partial
// rows are read eight at a time, all eight loads issued before any is used:
// row indices are clamped into the rows the slot has and the terms outside
// them are selected to zero, so the sum keeps its order bit for bit.
__global__ void __launch_bounds__(256) score_reduce_kernel(PrefillArgs a, int pt_positions) {
  const int u = blockIdx.x;
  const int n = a.len0 + a.n_tok;
  const int j = blockIdx.y * 256 + threadIdx.x;
  if (j < n) {
    const float* part = a.partial + (int64_t)u * a.npt_stride * a.cap + j;
    float* score = a.score + (int64_t)u * a.cap;
    const int pt0 = j < a.len0 ? 0 : (j - a.len0) / pt_positions;
    const int last = a.npt_used - 1;
    float acc = j < a.len0 ? score[j] : 0.0f;
    if (a.accumulate) {
      for (int c0 = pt0 & ~7; c0 <= last; c0 += 8) {
        float x[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) x[c] = part[(int64_t)min(max(c0 + c, pt0), last) * a.cap];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const int pt = c0 + c;
          acc += pt >= pt0 && pt <= last ? x[c] : 0.0f;
        }
      }
    }
    score[j] = acc;
  }
  if (blockIdx.y == 0 && threadIdx.x == 0) a.len[u] = n;
}

// Workgroups per position tile.  A launch of fewer workgroups than compute units
// takes as long as one of them, and sweep 2 is a third of that: idle units take
// over its tiles, each after a sweep 1 of its own (every one needs the rows'
// normalisers).  Sums and outputs stay the same bit for bit.  us a prompt, block by
// block, with one workgroup per tile -> with those of this rule:
//   workgroups (one per tile)       64 (4)     84-88 (3, 2)  104 (2)    128 (2)
//   bf16 d=128 G=4 s=4096           514 -> 444 524 -> 453    524 -> 460 531 -> 470
//   bf16 d=128 G=1 s=4096, B=512    449 -> 371 452 -> 386    454 -> 392 456 -> 398
//   bf16 d=64 G=2 s=1999, B=100     453 -> 385 458 -> 408    462 -> 410 465 -> 415
//   float32 d=64 G=1 s=512, B=64    244 -> 208 248 -> 224    249 -> 226 251 -> 228
//   float32 d=128 G=4 s=1024, B=128 695 -> 587 699 -> 605    703 -> 615 709 -> 626
// and 32 workgroups of the first 513 -> 435, 8 of the fourth 234 -> 195.  With a second
// workgroup on a compute unit the repeated sweep 1 would cost time again (a wave's
// tile takes half as long again beside another's), and past four the outputs'
// store is as long as the sums.
constexpr int kComputeUnits = 256;
constexpr int kMaxSplit = 4;
// Outputs that overlap the queries rule it out: the workgroups of a tile read the same
// query rows, and the first stores outputs while others may not have begun (one
// workgroup reads its rows before it stores them, so attention in place is right).
// Timeline builds never split: their records are one workgroup's, both sweeps whole.
int split_of(const PrefillArgs& a, int row_bytes) {
  if (kTimeline || !a.accumulate) return 1;
  const int64_t planes = (int64_t)a.units * (a.n_heads / a.n_kv_heads);
  const uintptr_t span = (uintptr_t)(((planes - 1) * a.seq_ld + a.n_tok) * row_bytes);
  const uintptr_t q = (uintptr_t)a.q, o = (uintptr_t)a.o;
  if (q < o + span && o < q + span) return 1;
  return max(1, min(kMaxSplit, kComputeUnits / (a.units * a.npt_used)));
}

template <bool BF16, int D, int G, bool SPLIT>
hipError_t launch_s(const PrefillArgs& a, hipStream_t stream) {
  dim3 grid((unsigned)(a.units * a.npt_used * a.nsplit));
  if (a.pad)
    hipLaunchKernelGGL((prefill_attn_kernel<BF16, D, G, true, SPLIT>), grid, dim3(kThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((prefill_attn_kernel<BF16, D, G, false, SPLIT>), grid, dim3(kThreads), 0, stream, a);
  return hipGetLastError();
}

template <bool BF16, int D, int G>
hipError_t launch_t(PrefillArgs a, hipStream_t stream) {
  a.nsplit = split_of(a, Cfg<BF16, D>::RB);
  return a.nsplit > 1 ? launch_s<BF16, D, G, true>(a, stream) : launch_s<BF16, D, G, false>(a, stream);
}

template <bool BF16, int D>
hipError_t launch_g(const PrefillArgs& a, int group, hipStream_t stream) {
  switch (group) {
    case 1: return launch_t<BF16, D, 1>(a, stream);
    case 2: return launch_t<BF16, D, 2>(a, stream);
    case 4: return launch_t<BF16, D, 4>(a, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_prefill(const PrefillArgs& a, int dtype, int head_dim, int group,
                          hipStream_t stream) {
  if (dtype == BM_BF16) {
    if (head_dim == 128) return launch_g<true, 128>(a, group, stream);
    if (head_dim == 64) return launch_g<true, 64>(a, group, stream);
  } else if (dtype == BM_F32) {
    if (head_dim == 128) return launch_g<false, 128>(a, group, stream);
    if (head_dim == 64) return launch_g<false, 64>(a, group, stream);
  }
  return hipErrorInvalidValue;
}

int prefill_split(const PrefillArgs& a, int row_bytes) { return split_of(a, row_bytes); }

bool timeline_enabled() { return kTimeline; }

hipError_t read_timeline(uint64_t* dst, int n_records) {
#ifdef BM_PREFILL_TIMELINE
  return hipMemcpyFromSymbol(dst, HIP_SYMBOL(g_timeline),
                             (size_t)n_records * BM_TIMELINE_FIELDS * sizeof(uint64_t), 0,
                             hipMemcpyDeviceToHost);
#else
  (void)dst;
  (void)n_records;
  return hipErrorNotSupported;
#endif
}

hipError_t launch_score_reduce(const PrefillArgs& a, hipStream_t stream) {
  const int group = a.n_heads / a.n_kv_heads;
  const unsigned chunks = (unsigned)((a.len0 + a.n_tok + 255) / 256);
  hipLaunchKernelGGL(score_reduce_kernel, dim3((unsigned)a.units, chunks), dim3(256), 0, stream,
                     a, positions_per_wg(group));
  return hipGetLastError();
}

}  // namespace bm
