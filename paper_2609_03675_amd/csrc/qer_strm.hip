// qer_strm_kernel: m_j = scale * max_i sum over the contraction of q_i k_j for
// bf16 rows (LOGIT mode, Eq. 6-7), on gfx950.
//
// HBM-bound: about n_q flop per byte of keys.  What the kernel has to do is
// keep the key stream deep and undisturbed, so keys go from HBM to LDS by DMA
// (no registers held in flight) and nothing but MFMAs happens to them:
//  * one workgroup of 8 waves per CU; a wave owns 32 keys and all (at most
//    16 QB) query rows of a chunk, over the whole contraction or, for inputs
//    of few tiles, one of NS slices of it;
//  * the contraction runs in segments of 64 elements (128 bytes of a row, the
//    shape that streams at full rate: 8 rows x 128 bytes per instruction).  A
//    wave has SL slots of one segment of its keys in LDS: it copies a slot
//    to registers (4 fragments), refills it at once with the segment SL
//    ahead, and multiplies from registers;
//  * the queries' segments are shared by the workgroup, in SL buffers; each
//    wave brings its share SL - 1 segments ahead, so one barrier per segment
//    publishes the next and retires the last;
//  * both sides sit in LDS as rows of 128 bytes whose 16-byte chunk c is at
//    slot c ^ (row / 2 % 8): the DMA writes its lanes' 16 bytes consecutively,
//    so the permutation is made by the lanes' global addresses, and 16 rows'
//    reads of one chunk fall on all 64 banks.
// S = Q K^T (32x32x16 MFMA, queries as the A operand): a lane holds one key
// and 16 query rows of a block in registers, so the max over the rows is in
// registers but for one exchange between the half waves.
// The pipeline runs over all rounds of a workgroup's share (NS = 1).
// Measured against keys loaded to registers in operand shape by a lane select
// and a DPP rotation, queries restaged through registers (28 heads of 128):
// 32 rows x 32768 keys 41.6 -> 37.5 us (6.3 TB/s), 64 x 46080 75 -> 57 (5.8),
// 128 x 50176 151 -> 74 (one pass over K; it took two), 32 streams of 128 rows
// (2.5 GB) 569 with the operand-order copy of the queries -> 480 (5.2).  Twice
// the keys per wave with two slots (a quarter of the query traffic) took 497.
#include "qer_strm.h"

#include <algorithm>
#include <climits>
#include <cmath>

namespace cofie {
namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((__vector_size__(8 * sizeof(__bf16))));
typedef __attribute__((address_space(3))) void lds_void;

constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kSegBytes = 128;
constexpr int kKeyDma = 4;  // key DMA instructions per segment and wave

// LDS of a configuration: the query buffers [SL][NS][P 16 QB rows][128], then
// the waves' key slots [8][SL][32 rows][128].  (The last 32-row block of an
// odd QB reads 16 rows past its term's; those products are never used.)
__host__ __device__ constexpr int strm_q_bytes(int QB, int P, int NS) { return NS * P * QB * 16 * kSegBytes; }
constexpr int kKeyBytes = 32 * kSegBytes;
__host__ __device__ constexpr int strm_lds(int QB, int P, int NS, int SL) {
  return SL * (strm_q_bytes(QB, P, NS) + kWaves * kKeyBytes);
}

// DMA instruction i of 8 rows x 128 bytes: lane l brings row 8 i + l / 8's
// chunk (l % 8) ^ (row / 2 % 8) to slot l % 8.
__host__ __device__ __forceinline__ int strm_chunk(int i, int l) { return (l & 7) ^ ((4 * (i & 1) + (l >> 4)) & 7); }
// Fragment of MFMA step j (16 elements) of a 32-row block: lane l reads row
// l % 32's chunk 2 j + l / 32.
__host__ __device__ __forceinline__ int strm_frag(int j, int l) {
  const int r = l & 31;
  return r * kSegBytes + 16 * ((2 * j + (l >> 5)) ^ ((r >> 1) & 7));
}

// The part of a share [f_begin, f_end) that lies in one sequence, and its
// rounds: each of at most `cap` tiles, of equal size (to a tile).
struct Piece {
  int tb, te, rounds;  // tiles of the sequence
};
__host__ __device__ __forceinline__ Piece strm_piece(const QerStreamDesc& sd, int f_begin, int f_end, int cap) {
  Piece p;
  p.tb = (f_begin > sd.tile0 ? f_begin : sd.tile0) - sd.tile0;
  const int s_end = sd.tile0 + sd.ntiles;
  p.te = (s_end < f_end ? s_end : f_end) - sd.tile0;
  p.rounds = p.te > p.tb ? (p.te - p.tb + cap - 1) / cap : 0;
  return p;
}
// Keys [k0, k1) of wave group g of KG in round r of a piece (k1 - k0 <= 32).
__host__ __device__ __forceinline__ void strm_window(const Piece& p, int r, int g, int KG, int n_keys, int& k0, int& k1) {
  const int n = p.te - p.tb;
  const int t0 = p.tb + (int)((int64_t)n * r / p.rounds), t1 = p.tb + (int)((int64_t)n * (r + 1) / p.rounds);
  k0 = 16 * (t0 + (t1 - t0) * g / KG);
  k1 = 16 * (t0 + (t1 - t0) * (g + 1) / KG);
  k1 = k1 < n_keys ? k1 : n_keys;
}
// Row (relative to the window) that instruction i's lane l loads: past the
// window its last row again, an empty window the row it would begin at.
__host__ __device__ __forceinline__ int strm_row(int i, int l, int keys) {
  const int r = 8 * i + (l >> 3);
  return r < keys ? r : (keys > 0 ? keys - 1 : 0);
}

// Query DMA instruction i of a segment (slice i / (2 P QB), then term and 8
// rows): lane l's byte offset from row q0 of the first term.  Rows past the
// chunk repeat its last.
__host__ __device__ __forceinline__ int64_t strm_q_off(int i, int l, int P, int QB, int32_t nq_total, int32_t n_rows,
                                                       int64_t row_bytes, int64_t slice_bytes) {
  const int sl = i / (2 * P * QB), b = i % (2 * P * QB), p = b / (2 * QB);
  const int row = 8 * (b % (2 * QB)) + (l >> 3);
  const int64_t grow = (int64_t)p * nq_total + (row < n_rows ? row : n_rows - 1);
  return grow * row_bytes + sl * slice_bytes + 16 * strm_chunk(b, l);
}

// A wave-uniform value in scalar registers (the loop state that forms it looks
// divergent to the compiler).
__device__ __forceinline__ uint32_t uniform(uint32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ const uint8_t* uniform(const uint8_t* p) {
  const uint64_t v = (uint64_t)p;
  return (const uint8_t*)(((uint64_t)uniform((uint32_t)(v >> 32)) << 32) | uniform((uint32_t)v));
}

__device__ __forceinline__ uint32_t lds_addr(const char* p) { return (uint32_t)(size_t)(lds_void*)p; }

// 64 lanes x 16 bytes from base + off (bytes) to 1 KiB of LDS at `dst`.  Not
// seen by the compiler's wait insertion: the loops below wait for it.  Nor by
// its hazard recognizer: a scalar base that a VALU instruction wrote
// (v_readfirstlane) may be read by a vector-memory instruction only 5 wait
// states later, and M0 one wait state after its write, hence the s_nop 4.
__device__ __forceinline__ void dma(const uint8_t* base, uint32_t off, uint32_t dst) {
  asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "{m0}"(dst) : "memory");
}
__device__ __forceinline__ void dma_nt(const uint8_t* base, uint32_t off, uint32_t dst) {
  asm volatile("s_nop 4\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off), "s"(base), "{m0}"(dst) : "memory");
}
// All but this wave's last N vector-memory operations are done, its LDS reads
// too; then the workgroup's barrier.
template <int N>
__device__ __forceinline__ void wait_barrier() {
  static_assert(N < 64, "vmcnt field");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(N) : "memory");
}
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ float max_x32(float v) {
  const auto p = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}

// Wait before segment s with rem segments after it (SL - 1 or more: any): what
// may still be in flight is newer than the segment's keys and queries -- the
// keys of the next SL - 1 segments and the queries of the next SL - 2.
template <int SL, int QW>
__device__ __forceinline__ void wait_segment(int rem) {
  constexpr int KI = kKeyDma;
  constexpr int N = (SL - 1) * KI + (SL - 2) * QW;
  if (rem >= SL - 1) wait_barrier<N>();
  else if (rem == 0) wait_barrier<0>();
  else if (rem == 1) wait_barrier<KI + (SL > 2 ? QW : 0)>();
  else wait_barrier<2 * KI + (SL > 3 ? 2 : 1) * QW>();
}

template <int QB, int P, int NS, int SL>
__global__ __launch_bounds__(kThreads) void qer_strm_kernel(StrmArgs a) {
  constexpr int QT = (QB + 1) / 2;                    // 32-row query blocks
  constexpr int KG = kWaves / NS, CAP = 2 * KG;      // wave groups (key windows), tiles per round
  constexpr int QI = NS * P * QB * 2;                 // query DMA instructions per segment
  constexpr int QW = (QI + kWaves - 1) / kWaves;      // of each wave (past QI: an earlier one again)
  constexpr int KI = kKeyDma;
  static_assert(SL >= 2 && SL <= 4, "wait_segment");
  extern __shared__ __align__(16) char lds[];
  const int tid = threadIdx.x, l = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int slice = wave % NS, grp = wave / NS;
  char* const qlds = lds;
  char* const klds = lds + SL * strm_q_bytes(QB, P, NS) + wave * SL * kKeyBytes;
  const uint32_t q_dst = lds_addr(qlds), k_dst = lds_addr(klds);
  const int64_t slice_bytes = (int64_t)a.nseg * kSegBytes;
  if (blockIdx.x == 0 && a.clear)
    for (int i = tid; i < a.nclear; i += kThreads) a.clear[i] = 0;

  const int wg = a.xcd_order ? (int)((blockIdx.x & 7) * (a.nwg >> 3) + (blockIdx.x >> 3)) : (int)blockIdx.x;
  const int f_begin = (int)((int64_t)a.tiles * wg / a.nwg);
  const int f_end = (int)((int64_t)a.tiles * (wg + 1) / a.nwg);

  // the rounds of the share, in order
  struct Rnd {
    int s, r;  // sequence, round of its piece; s = n_seq: none
    QerStreamDesc sd;
    Piece pc;
  };
  auto seek = [&](Rnd& x, int s) __attribute__((always_inline)) {  // the first round of sequence s or later
    for (x.s = s, x.r = 0; x.s < a.n_seq; ++x.s) {
      x.sd = a.seq ? a.seq[x.s] : a.one;
      if (x.sd.tile0 >= f_end) {
        x.s = a.n_seq;
        break;
      }
      x.pc = strm_piece(x.sd, f_begin, f_end, CAP);
      if (x.pc.rounds > 0) break;
    }
  };
  auto next_of = [&](Rnd& x) __attribute__((always_inline)) {
    if (++x.r >= x.pc.rounds) seek(x, x.s + 1);
  };

  // DMA sources of a round: uniform bases and this lane's byte offsets
  struct Src {
    const uint8_t* kbase;
    const uint8_t* qbase;
    uint32_t koff[KI];
    uint32_t qoff[QW];
  };
  auto source = [&](const Rnd& x, Src& o) __attribute__((always_inline)) {
    int k0, k1;
    strm_window(x.pc, x.r, grp, KG, x.sd.n_keys, k0, k1);
    o.kbase = a.K + (x.sd.key0 + (k1 > k0 ? k0 : 0)) * a.row_bytes + slice * slice_bytes;
#pragma unroll
    for (int i = 0; i < KI; ++i)
      o.koff[i] = (uint32_t)(strm_row(i, l, k1 - k0) * a.row_bytes) + 16u * strm_chunk(i, l);
    o.qbase = a.Q + (int64_t)x.sd.q0 * a.row_bytes;
#pragma unroll
    for (int j = 0; j < QW; ++j)
      o.qoff[j] = (uint32_t)strm_q_off((wave + kWaves * j) % QI, l, P, QB, a.nq_total, x.sd.n_rows, a.row_bytes, slice_bytes);
  };
  auto q_dma = [&](const Src& o, int seg, int buf) __attribute__((always_inline)) {
    const uint8_t* base = uniform(o.qbase + (int64_t)seg * kSegBytes);
    const uint32_t dst = uniform(q_dst + buf * strm_q_bytes(QB, P, NS));
#pragma unroll
    for (int j = 0; j < QW; ++j) dma(base, o.qoff[j], dst + 1024 * ((wave + kWaves * j) % QI));
  };
  auto k_dma = [&](const Src& o, int seg, int slot) __attribute__((always_inline)) {
    const uint8_t* base = uniform(o.kbase + (int64_t)seg * kSegBytes);
    const uint32_t dst = uniform(k_dst + slot * kKeyBytes);
#pragma unroll
    for (int i = 0; i < KI; ++i) dma_nt(base, o.koff[i], dst + 1024 * i);
  };

  Rnd cur, nxt;
  seek(cur, 0);
  if (cur.s >= a.n_seq) return;
  Src sc, sn;
  source(cur, sc);
  int fo[4];  // this lane's fragment bytes of the four MFMA steps of a segment
#pragma unroll
  for (int j = 0; j < 4; ++j) fo[j] = strm_frag(j, l);

  f32x16 acc[QT];
  const int nseg = a.nseg;  // at least SL
  int slot = 0;             // of the current segment (query buffer and key slot)
  bool fresh = true;        // nothing in flight for the current round
  while (cur.s < a.n_seq) {
    nxt = cur;
    next_of(nxt);
    // with contraction slices the rounds' sums meet in LDS, so each round
    // starts its pipeline anew
    const bool more = NS == 1 && nxt.s < a.n_seq;
    if (more) source(nxt, sn);
    if (fresh) {
      slot = 0;
      k_dma(sc, 0, 0);
#pragma unroll
      for (int i = 0; i + 1 < SL; ++i) {
        q_dma(sc, i, i);
        k_dma(sc, i + 1, i + 1);
      }
      fresh = false;
    }
#pragma unroll
    for (int qt = 0; qt < QT; ++qt)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[qt][e] = 0.f;
    for (int seg = 0; seg < nseg; ++seg) {
      wait_segment<SL, QW>(more ? SL : nseg - 1 - seg);
      const char* qb = qlds + slot * strm_q_bytes(QB, P, NS) + slice * (P * QB * 16 * kSegBytes);
      const char* kb = klds + slot * kKeyBytes;
      const int before = slot == 0 ? SL - 1 : slot - 1;  // the buffer of the segment before: free now
      if (seg + SL - 1 < nseg) q_dma(sc, seg + SL - 1, before);
      else if (more) q_dma(sn, seg + SL - 1 - nseg, before);
      uint4 kf[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) kf[j] = *reinterpret_cast<const uint4*>(kb + fo[j]);
      wait_lds();  // the slot is in registers: refill it
      if (seg + SL < nseg) k_dma(sc, seg + SL, slot);
      else if (more) k_dma(sn, seg + SL - nseg, slot);
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int p = 0; p < P; ++p)
#pragma unroll
          for (int qt = 0; qt < QT; ++qt) {
            const uint4 qf = *reinterpret_cast<const uint4*>(qb + (p * QB * 16 + qt * 32) * kSegBytes + fo[j]);
            acc[qt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, qf),
                                                              __builtin_bit_cast(bf16x8, kf[j]), acc[qt], 0, 0, 0);
          }
      slot = slot + 1 == SL ? 0 : slot + 1;
    }

    int k0, k1;
    strm_window(cur.pc, cur.r, grp, KG, cur.sd.n_keys, k0, k1);
    if constexpr (NS > 1) {
      // the slices' sums: slices 1 .. NS-1 publish their accumulators over
      // the (now idle) buffers, slice 0 adds them in slice order
      float* red = reinterpret_cast<float*>(lds);
      constexpr int W = QT * 16 * 64;  // floats per wave
      __syncthreads();
      if (slice > 0) {
#pragma unroll
        for (int qt = 0; qt < QT; ++qt)
#pragma unroll
          for (int e = 0; e < 16; ++e)
            red[(grp * (NS - 1) + slice - 1) * W + (qt * 16 + e) * 64 + l] = acc[qt][e];
      }
      __syncthreads();
      if (slice == 0) {
#pragma unroll
        for (int sl = 1; sl < NS; ++sl)
#pragma unroll
          for (int qt = 0; qt < QT; ++qt)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[qt][e] += red[(grp * (NS - 1) + sl - 1) * W + (qt * 16 + e) * 64 + l];
      }
      __syncthreads();  // before the next round's DMA overwrites them
      fresh = true;
    }
    if (slice == 0) {
      // register e of a block holds query row 8 (e / 4) + 4 (l / 32) + e % 4
      // (registers 0-7: its first 16 rows), column l % 32 the key
      const int key = k0 + (l & 31);
      auto store = [&](int g, float v) __attribute__((always_inline)) {
        if (l >= 32 || key >= k1) return;
        float* dst = a.m + g * a.m_stride + key;
        const float x = v * a.scale;
        // a query that began in an earlier launch continues its max
        const bool cont = a.group_rows ? (int64_t)g * a.group_rows < cur.sd.q0 : a.accumulate != 0;
        *dst = cont ? fmaxf(*dst, x) : x;
      };
      float vg = -INFINITY;
      int gcur = -1;
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        if (16 * b >= cur.sd.n_rows) break;
        float v = -INFINITY;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int ee = 8 * (b & 1) + e;
          const int row = 32 * (b >> 1) + 8 * (ee >> 2) + 4 * (l >> 5) + (ee & 3);
          v = fmaxf(v, row < cur.sd.n_rows ? acc[b >> 1][ee] : -INFINITY);
        }
        v = max_x32(v);
        const int g = a.group_rows ? (cur.sd.q0 + 16 * b) / a.group_rows : 0;
        if (g != gcur) {
          if (gcur >= 0) store(gcur, vg);
          gcur = g;
          vg = v;
        } else {
          vg = fmaxf(vg, v);
        }
      }
      if (gcur >= 0) store(gcur, vg);
    }
    cur = nxt;
    sc = sn;
    if (NS > 1 && cur.s < a.n_seq) source(cur, sc);
  }
}

// ---- host side --------------------------------------------------------------------------

constexpr int kLdsMax = 160 * 1024;

// Key slots of a configuration: as many segments in flight as LDS holds.
constexpr int strm_slots(int QB, int P, int NS) {
  for (int sl = 4; sl > 2; --sl)
    if (strm_lds(QB, P, NS, sl) <= kLdsMax) return sl;
  return 2;
}

// Address model of qer_strm_kernel (dry run): the rounds of every workgroup
// as the kernel walks them, its key and query DMA at both ends of each
// round's segments, the LDS it fills and reads, its stores of m.
void model_strm(const StrmArgs& a, int QB, int P, int NS, int SL, size_t lds) {
  const int KG = kWaves / NS, CAP = 2 * KG, QI = NS * P * QB * 2, KI = kKeyDma, QT = (QB + 1) / 2;
  const int64_t slice_bytes = (int64_t)a.nseg * kSegBytes;
  dry_range((int64_t)lds, 0, kLdsMax + 1, "score: LDS beyond a CU's 160 KiB");
  dry_range(a.nseg, SL, INT32_MAX, "score: fewer segments than slots");
  dry_range(a.row_bytes - NS * slice_bytes, 0, 1, "score: the slices' segments are not the row");
  if (a.xcd_order) dry_range(a.nwg % 8, 0, 1, "score: XCD order needs whole groups of 8 workgroups");
  if (a.clear && a.nclear > 0) dry_access(a.clear, 0, 4 * (int64_t)a.nclear, "score: arrival counters");
  const int64_t ring = SL * (int64_t)(strm_q_bytes(QB, P, NS) + kWaves * kKeyBytes);
  dry_lds(0, ring, (int64_t)lds, "score: buffers");
  if (NS > 1) dry_lds(0, (int64_t)KG * (NS - 1) * QT * 16 * 256, (int64_t)lds, "score: slice sums");
  int frag = 0;  // the last byte a fragment read reaches in its 32 rows
  for (int j = 0; j < 4; ++j)
    for (int l = 0; l < 64; ++l) frag = std::max(frag, strm_frag(j, l) + 16);
  dry_range(frag, 0, 32 * kSegBytes + 1, "score: fragment past its 32 rows");
  dry_lds((SL - 1) * (int64_t)strm_q_bytes(QB, P, NS) + (NS - 1) * P * QB * 16 * kSegBytes +
              ((P - 1) * QB * 16 + (QT - 1) * 32) * kSegBytes, frag, (int64_t)lds, "score: query fragment");
  const QerStreamDesc* seq = nullptr;
  if (a.seq) {
    seq = static_cast<const QerStreamDesc*>(dry_shadow(a.seq));
    if (!seq) {
      dry_range(0, 0, 0, "score: sequence table without a host copy");
      return;
    }
    dry_access(a.seq, 0, a.n_seq * (int64_t)sizeof(QerStreamDesc), "score: sequence table");
  }
  for (int wg = 0; wg < a.nwg; ++wg) {
    const int f_begin = (int)((int64_t)a.tiles * wg / a.nwg), f_end = (int)((int64_t)a.tiles * (wg + 1) / a.nwg);
    for (int s = 0; s < a.n_seq; ++s) {
      const QerStreamDesc sd = seq ? seq[s] : a.one;
      if (sd.tile0 >= f_end) break;
      const Piece pc = strm_piece(sd, f_begin, f_end, CAP);
      if (pc.rounds <= 0) continue;
      dry_range(pc.tb, 0, pc.te, "score: piece");
      dry_range(pc.te, 1, (int64_t)sd.ntiles + 1, "score: piece past its sequence");
      dry_range(sd.n_rows, 1, 16 * (int64_t)QB + 1, "score: query rows of a chunk");
      for (int i = 0; i < QI; ++i)
        for (int l = 0; l < 64; ++l) {
          const int64_t off = strm_q_off(i, l, P, QB, a.nq_total, sd.n_rows, a.row_bytes, slice_bytes);
          dry_range(off, 0, int64_t(1) << 32, "score: query offset past 32 bits");
          for (int64_t seg : {int64_t(0), (int64_t)a.nseg - 1})
            dry_access(a.Q, sd.q0 * a.row_bytes + off + seg * kSegBytes, 16, "score: query load");
        }
      int next = 16 * pc.tb;  // the windows follow one another
      for (int r = 0; r < pc.rounds; ++r)
        for (int g = 0; g < KG; ++g) {
          int k0, k1;
          strm_window(pc, r, g, KG, sd.n_keys, k0, k1);
          dry_range(k0 - next, 0, 1, "score: a window begins where the one before ends");
          dry_range(k1 - k0, 0, 33, "score: window wider than the wave's keys");
          next = k1 > k0 && k1 % 16 == 0 ? k1 : (k1 > k0 ? (k1 + 15) / 16 * 16 : next);
          const int64_t base = (sd.key0 + (k1 > k0 ? k0 : 0)) * a.row_bytes;
          for (int i = 0; i < KI; ++i)
            for (int l = 0; l < 64; ++l) {
              const int64_t off = strm_row(i, l, k1 - k0) * a.row_bytes + 16 * strm_chunk(i, l);
              dry_range(off, 0, int64_t(1) << 32, "score: key offset past 32 bits");
              dry_access(a.K, base + off, 16, "score: key load");
              dry_access(a.K, base + off + a.row_bytes - kSegBytes, 16, "score: key load");
            }
          if (k1 <= k0) continue;
          dry_range(k1 - 1, 0, a.m_stride, "score: key past the row of m");
          for (int b = 0; b < QB && 16 * b < sd.n_rows; ++b) {
            const int64_t q = a.group_rows ? (sd.q0 + 16 * b) / a.group_rows : 0;
            dry_access(a.m, (q * a.m_stride + k0) * 4, 4 * (int64_t)(k1 - k0), "score: m");
          }
        }
      dry_range(next - 16 * pc.te, 0, 1, "score: the windows cover the piece");
    }
  }
}

template <int QB, int P, int NS, int SL>
int launch_t(const StrmArgs& a, hipStream_t s) {
  constexpr int QT = (QB + 1) / 2;
  constexpr size_t lds = std::max(strm_lds(QB, P, NS, SL), (kWaves / NS) * (NS - 1) * QT * 16 * 256);
  static_assert(lds <= (size_t)kLdsMax, "LDS of a CU");
  const auto k = qer_strm_kernel<QB, P, NS, SL>;
  int rc = allow_lds(k, lds);
  if (rc) return rc;
  if (dry_run()) {
    model_strm(a, QB, P, NS, SL, lds);
    return COFIE_OK;
  }
  return launch("qer_score", k, dim3((unsigned)a.nwg), dim3(kThreads), lds, s, a);
}

template <int QB, int P, int NS>
int launch_qb(const StrmArgs& a, hipStream_t s) {
  constexpr int SL = strm_slots(QB, P, NS);
  if constexpr (SL > 2)
    if (a.nseg >= SL) return launch_t<QB, P, NS, SL>(a, s);
  return launch_t<QB, P, NS, 2>(a, s);
}

}  // namespace

// The slices: the least time is one round with every wave at work, so tiles
// that would not give each of a CU's 8 waves 32 keys split the contraction
// (16 / NS tiles per CU and round).  A slice needs two segments for the
// pipeline.  Three query terms take at most two slices: their query buffers
// fill the LDS.  Score kernel, 28 heads of 128: 16 x 144 keys 9.3 us (8
// slices), 50 x 144 13.9 (8), 128 x 256 37.5 (2); the register-fed kernel with
// its 4, 4 and 1 slices 16.5, 19.6 and 41.6.
StrmPlan plan_strm(int64_t tiles, int64_t Lc, int P, int rows, int cus) {
  StrmPlan p{0, 0, 0};
  if (tiles <= 0 || Lc % 64 != 0 || Lc / 64 < 2) return p;
  const int64_t nseg = Lc / 64, per_cu = (tiles + cus - 1) / cus;
  auto max_rows = [&](int ns) { return P == 3 ? 64 : (ns == 8 ? 32 : (ns == 4 ? 64 : 128)); };
  p.NS = 1;
  for (int ns = P == 1 ? 8 : 2; ns > 1; ns /= 2)
    if (per_cu <= 16 / ns && nseg % ns == 0 && nseg / ns >= 2 && rows <= max_rows(ns)) {
      p.NS = ns;
      break;
    }
  p.max_rows = max_rows(p.NS);
  if (rows > p.max_rows) p.NS = 0;
  p.nwg = (int)std::min<int64_t>(cus, tiles);
  return p;
}

int launch_strm(const StrmArgs& a, const StrmPlan& p, int P, int rows, hipStream_t s) {
  const int qb = (rows + 15) / 16;
  if (rows < 1 || rows > p.max_rows || (P != 1 && P != 3))
    return set_error(COFIE_EHIP, "streaming score kernel: %d rows, %d terms", rows, P);
  if (P == 3) {
    if (p.NS == 2) {
      if (qb == 1) return launch_qb<1, 3, 2>(a, s);
      if (qb == 2) return launch_qb<2, 3, 2>(a, s);
      return qb == 3 ? launch_qb<3, 3, 2>(a, s) : launch_qb<4, 3, 2>(a, s);
    }
    if (qb == 1) return launch_qb<1, 3, 1>(a, s);
    if (qb == 2) return launch_qb<2, 3, 1>(a, s);
    return qb == 3 ? launch_qb<3, 3, 1>(a, s) : launch_qb<4, 3, 1>(a, s);
  }
  switch (p.NS) {
    case 8: return qb == 1 ? launch_qb<1, 1, 8>(a, s) : launch_qb<2, 1, 8>(a, s);
    case 4:
      if (qb == 1) return launch_qb<1, 1, 4>(a, s);
      if (qb == 2) return launch_qb<2, 1, 4>(a, s);
      return qb == 3 ? launch_qb<3, 1, 4>(a, s) : launch_qb<4, 1, 4>(a, s);
    case 2:
      if (qb == 1) return launch_qb<1, 1, 2>(a, s);
      if (qb == 2) return launch_qb<2, 1, 2>(a, s);
      if (qb == 3) return launch_qb<3, 1, 2>(a, s);
      return qb == 4 ? launch_qb<4, 1, 2>(a, s) : launch_qb<8, 1, 2>(a, s);
    default:
      if (qb == 1) return launch_qb<1, 1, 1>(a, s);
      if (qb == 2) return launch_qb<2, 1, 1>(a, s);
      if (qb == 3) return launch_qb<3, 1, 1>(a, s);
      return qb == 4 ? launch_qb<4, 1, 1>(a, s) : launch_qb<8, 1, 1>(a, s);
  }
}

}  // namespace cofie
