// FP16 GEMM update C = alpha * op(A) op(B) + beta * R for gfx950.
//
// Sec. 4.1 of the paper describes the GEMM primitive (output tile loaded as
// the accumulation buffer) that serves the QKV / output / FFN projections in
// forward, data-gradient and weight-gradient form.  The MT-3000 dataflow
// (DDR -> GSM -> SM / AM staging, VLIW micro-kernel) is replaced here by the
// CDNA4 form of the same idea:
//   * a workgroup owns a BM x BN output tile held in MFMA accumulators
//     (16x16x32 FP16 MFMA, FP32 accumulate).  256x256, 256x128, 128x256,
//     128x128 and 64x64 tiles use 4 waves, one per SIMD, in a 2x2 grid with
//     their accumulators in AGPRs; their main loop is a fixed sequence of asm
//     statements (fragment reads a whole k-step ahead, MFMAs, direct loads,
//     counter waits), so that one wave keeps its matrix unit fed without a
//     second wave to cover its waits.  Every layout, the fused epilogues and
//     the split-K partial tiles use it; only the ragged-K form of layouts with
//     a K-contiguous operand uses compiler-scheduled loops (8 waves, two per
//     SIMD, at 256x256: the other wave covers LDS and barrier waits);
//   * K is walked in 64-wide slices, in two LDS stages at 256x256 and up to
//     eight at smaller tiles.  Operands move HBM -> LDS with direct buffer
//     loads (16 B per lane, no register staging), issued one or more slices
//     ahead so that they overlap the current slice's MFMA work -- the
//     overlap of operand preparation with MACs that the paper's micro-kernel
//     pipeline provides.  In 8-wave tiles only one wave per SIMD issues them
//     ("loader waves"), with uniform (scalar) addressing;
//   * each operand keeps its HBM orientation in LDS.  A K-contiguous operand
//     (forward A and B, dgrad A) is stored row-major; an M/N-contiguous one
//     (dgrad B, wgrad A and B) is stored k-major and read with the gfx950
//     LDS transpose read (ds_read_b64_tr_b16), so every (transA, transB)
//     runs the same MFMA loop at the same speed;
//   * LDS positions are XOR-swizzled so that both the direct loads and the
//     MFMA operand reads are free of bank conflicts (16 lanes x 16 B per LDS
//     cycle);
//   * tiles are ordered so that each XCD gets a contiguous range of tiles,
//     grouped eight tile-rows at a time for L2 reuse of A and B.
//   Buffer loads return zeros out of range, which provides the M, N and K
//   tails without branches.
//   * results leave through LDS, 16 rows of a wave at a time, so that memory
//     sees whole lines (see the epilogue).
//   gemm_plan chooses the launch: one tile size, or whole rounds of 256x256
//   tiles and a tail of smaller ones, or, when the caller provides an FP32
//   workspace, a tail (or the whole product) of 256x256 tiles whose K is split
//   over several workgroups (epilogue 3 stores their partial sums;
//   splitk_reduce_kernel adds them in a fixed order and applies alpha,
//   beta * R and the bias).
#include <type_traits>
#include <utility>

#include "common.hpp"
#include "kernels.hpp"

namespace lt {
namespace {

// One operand tile: R rows (M for A, N for B) x BK.
//   KC  (K-contiguous in HBM): LDS row-major, CPR = BK/8 16-byte chunks per
//       row; chunk c of row r sits at position c ^ swz(r), which places the
//       16 consecutive rows read by one LDS cycle (16 lanes x 16 B) in 16
//       different bank groups.
//   !KC (row index contiguous in HBM): LDS k-major, 2R bytes per k-row;
//       16-byte chunk c (rows 8c..8c+7) of k-row k sits at position
//       kpos(c, k) = ((c >> 2) ^ (k & 3)) * 4 + ((c & 3) ^ 2 * ((k >> 3) & 1)):
//       the transpose reads of one MFMA operand (4 k-rows x 32 bytes per
//       16-lane group, groups 8 k-rows apart) then hit every bank once.
//       With R = 64 a k-row is half the banks wide: k's parity picks the
//       half, and chunk pair c >> 1 sits at (c >> 1) ^ (k bit 1, k bit 3).
// Both are filled by direct global -> LDS loads issued as opaque
// instructions, so the caller orders them with explicit vmcnt waits.
template <int R, int BK, bool KC, int NT, bool PAIRED = false, int PB = 32>
struct Operand {
  static constexpr int BYTES = R * BK * 2;
  static constexpr int NINST = BYTES / 1024;        // 1 KiB direct loads per slice
  static constexpr int PERW = NINST / (NT / 64);     // ... per wave
  static_assert(NINST % (NT / 64) == 0, "slice must split across waves");
  static constexpr int CPR = BK / 8;                 // KC: 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;               // KC: rows per direct load
  static constexpr int KR_PER = 1024 / (2 * R);      // !KC: k-rows per direct load
  static constexpr int LPR = 64 / KR_PER;            // !KC: lanes per k-row
  static_assert(CPR >= 4 && CPR <= 16, "KC layout needs 32 <= BK <= 128");

  __device__ static __forceinline__ int swz(int r) { return (r / (16 / CPR)) & (CPR - 1); }
  // !KC chunk position; an involution in c for fixed k
  __device__ static __forceinline__ int kpos(int c, int k) {
    if constexpr (R == 64) return c ^ ((((k >> 1) & 1) | (((k >> 3) & 1) << 1)) << 1);
    return (((c >> 2) ^ (k & 3)) << 2) | ((c & 3) ^ (((k >> 3) & 1) << 1));
  }

  uint32_t voff[PERW];
  const lt_half* base;
  int64_t ld, row0;
  uint32_t nrec;

  // PAIRED (K-contiguous only): tile row r = 32*blk + w reads matrix row
  // row0 + 32*(blk/2) + w, plus pair_off for odd blk: alternating 32-row
  // blocks of two row ranges (gate and up rows of a fused projection);
  // `rows` bounds the index inside each range.
  __device__ __forceinline__ void init(const lt_half* b, int64_t ld_, int64_t row0_, int64_t rows,
                                       int wave, int lane, int64_t pair_off = 0) {
    base = b;
    ld = ld_;
    row0 = row0_;
    if constexpr (PAIRED) {
      static_assert(KC, "paired rows are K-contiguous");
      nrec = 0x7fffffff;
#pragma unroll
      for (int t = 0; t < PERW; ++t) {
        const int r = (wave * PERW + t) * RPI + lane / CPR;
        const int64_t idx = row0 + PB * (r / (2 * PB)) + (r % PB);
        const int64_t abs_row = idx + ((r / PB) & 1 ? pair_off : 0);
        const int c = (lane % CPR) ^ swz(r);
        voff[t] = idx < rows ? (uint32_t)((abs_row * ld + c * 8) * 2) : kOOB;
      }
    } else if constexpr (KC) {
      // rows past the matrix fall outside the buffer and read as zero
      // (32-bit sums: the scalar unit has no 64-bit compare, and a range
      // held in a vector register would reach the descriptor through a
      // v_readfirstlane, whose result the asm loads may not use at once)
      const int left = (int)rows - (int)row0;
      nrec = __builtin_amdgcn_readfirstlane((uint32_t)(left < R ? left : R) * (uint32_t)ld * 2);
#pragma unroll
      for (int t = 0; t < PERW; ++t) {
        const int r = (wave * PERW + t) * RPI + lane / CPR;
        const int c = (lane % CPR) ^ swz(r);
        voff[t] = (uint32_t)((r * ld + c * 8) * 2);
      }
    } else {
      nrec = 0x7fffffff;
#pragma unroll
      for (int t = 0; t < PERW; ++t) {
        const int k = (wave * PERW + t) * KR_PER + lane / LPR;
        const int c = kpos(lane % LPR, k);             // chunk that lands at position lane % LPR
        voff[t] = row0 + c * 8 < rows ? (uint32_t)((k * ld + c * 8) * 2) : kOOB;
      }
    }
  }

  // Direct loads of the slice starting at k0 into the LDS tile at `lds`;
  // kvalid < BK only for the last slice of a ragged K.
  __device__ __forceinline__ void load(char* lds, int64_t k0, int kvalid, int wave, int lane) const {
    if constexpr (KC) {
      // descriptor based at column k0 of row row0: the range shrinks by the
      // same 2*k0 bytes, so rows past the matrix still read as zero (paired
      // rows carry absolute offsets and explicit out-of-range offsets)
      const lt_half* b = PAIRED ? base + k0 : base + row0 * ld + k0;
      const uint32_t n = PAIRED ? nrec : nrec - (uint32_t)(k0 * 2);
      if (kvalid >= BK) {
#pragma unroll
        for (int t = 0; t < PERW; ++t) {
          const int i = wave * PERW + t;
          lds_dma16_opaque(b, n, lds + i * 1024, voff[t]);
        }
      } else {
#pragma unroll
        for (int t = 0; t < PERW; ++t) {
          const int i = wave * PERW + t;
          const int r = i * RPI + lane / CPR;
          const uint32_t off = ((lane % CPR) ^ swz(r)) * 8 >= kvalid ? kOOB : voff[t];
          lds_dma16_opaque(b, n, lds + i * 1024, off);
        }
      }
    } else {
      const lt_half* b = base + k0 * ld + row0;
      if (kvalid >= BK) {
#pragma unroll
        for (int t = 0; t < PERW; ++t) {
          const int i = wave * PERW + t;
          lds_dma16_opaque(b, nrec, lds + i * 1024, voff[t]);
        }
      } else {
#pragma unroll
        for (int t = 0; t < PERW; ++t) {
          const int i = wave * PERW + t;
          const uint32_t off = i * KR_PER + lane / LPR >= kvalid ? kOOB : voff[t];
          lds_dma16_opaque(b, nrec, lds + i * 1024, off);
        }
      }
    }
  }

  // buffer descriptor of the full K-contiguous slice at k0 (uniform)
  __device__ __forceinline__ u32x4 desc(int64_t k0) const {
    const uint64_t b = (uint64_t)(!KC ? base + k0 * ld + row0 : PAIRED ? base + k0 : base + row0 * ld + k0);
    u32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((uint32_t)b);
    r[1] = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32) & 0xffffu);
    r[2] = __builtin_amdgcn_readfirstlane(!KC || PAIRED ? nrec : nrec - (uint32_t)(k0 * 2));
    r[3] = 0x00020000u;
    return r;
  }

  // one direct load (index t of this wave's PERW) of the K-contiguous slice
  // at k0 with kv = clamp(K - k0, 0, BK) valid columns; kv = 0 fills the
  // tile with zeros and touches no memory (every offset out of range)
  __device__ __forceinline__ void load1(char* lds, int64_t k0, int kv, int t, int wave,
                                        int lane) const {
    const int i = wave * PERW + t;
    const int64_t kb = kv > 0 ? k0 : 0;
    if constexpr (KC) {
      const lt_half* b = PAIRED ? base + kb : base + row0 * ld + kb;
      const uint32_t n = PAIRED ? nrec : nrec - (uint32_t)(kb * 2);
      const int r = i * RPI + lane / CPR;
      const uint32_t off = ((lane % CPR) ^ swz(r)) * 8 >= kv ? kOOB : voff[t];
      lds_dma16_opaque(b, n, lds + i * 1024, off);
    } else {
      const lt_half* b = base + kb * ld + row0;
      const uint32_t off = i * KR_PER + lane / LPR >= kv ? kOOB : voff[t];
      lds_dma16_opaque(b, nrec, lds + i * 1024, off);
    }
  }

  // K % 8 != 0 (K-contiguous tiles only; the k-major layout loads whole
  // k-rows, so its rows past K are already zero): the chunk of each row that
  // straddles K was loaded whole and holds the row's next elements in memory
  // (padding up to the leading dimension) past K.  Threads t < R of the
  // workgroup zero elements kvalid % 8 .. 7 of row t's chunk kvalid / 8 in
  // the LDS tile.  Called between the barrier after which the slice is
  // resident and a barrier before its first fragment read.
  __device__ __forceinline__ void zero_k_tail(char* lds, int kvalid, int t) const {
    static_assert(KC, "k-major tiles need no fix-up");
    if (t < 0 || t >= R) return;
    const int e0 = kvalid & 7;
    char* q = lds + t * (CPR * 16) + (((kvalid >> 3) ^ swz(t)) << 4);
    u32x4 v = *reinterpret_cast<const u32x4*>(q);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      // 16-bit elements 2w and 2w + 1 of the chunk
      const uint32_t keep = (2 * w < e0 ? 0x0000ffffu : 0u) | (2 * w + 1 < e0 ? 0xffff0000u : 0u);
      v[w] &= keep;
    }
    *reinterpret_cast<u32x4*>(q) = v;
  }

  // MFMA operand (16x16x32): rows rb..rb+15 (lane row = lane % 16),
  // reduction indices kk*32 + 8*(lane/16) + 0..7.
  __device__ __forceinline__ half8 frag(const char* lds, int rb, int kk, int lane) const {
    if constexpr (KC) {
      const int r = rb + (lane & 15);
      const int c = kk * 4 + (lane >> 4);
      return as_half8(*reinterpret_cast<const u32x4*>(lds + r * (CPR * 16) + ((c ^ swz(r)) << 4)));
    } else {
      // Two transpose reads (h = 0, 1).  Within 16-lane group G = L/16, lane
      // s = L%16 reads the 4 rows at m = rb + 4*(s%4) of k-row
      // kk*32 + 8G + 4h + s/4, and receives row rb + s of k-rows
      // kk*32 + 8G + 4h + 0..3.
      const int m = rb + 4 * (lane & 3);
      const int c = m >> 3;
      const int inoff = (m & 7) * 2;
      v4s part[2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int k = kk * 32 + 8 * (lane >> 4) + 4 * h + ((lane & 15) >> 2);
        part[h] = lds_read_tr16(lds + k * (2 * R) + kpos(c, k) * 16 + inoff);
      }
      return as_half8(pack_v4s_pair(part[0], part[1]));
    }
  }
};

// s_waitcnt vmcnt(n * PER), n clamped to [0, MAXN]: wait until at most n
// slices of direct loads (PER instructions each) are still in flight.
template <int PER, int MAXN>
__device__ __forceinline__ void wait_slices(int n) {
  if constexpr (MAXN > 0) {
    if (n >= MAXN) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(MAXN * PER) : "memory");
      return;
    }
    wait_slices<PER, MAXN - 1>(n);
  } else {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  }
}

// ---- building blocks of the 4-wave main loop ----
// The loop is written as asm statements that the compiler keeps in program
// order (volatile asm).  Two rules make that safe with the compiler still
// allocating the registers:
//   * a fragment read issued by asm is, to the compiler, complete at once; its
//     registers must not be read, copied or reused before the explicit
//     lgkmcnt wait.  Every fragment is consumed only by MFMA asm after that
//     wait (xfence re-defines the two halves of a transposed fragment after
//     the wait, so that joining them happens there), and the fragments read
//     for a step that never runs are kept allocated until the final wait
//     (xkeep);
//   * MFMAs issued by asm are not seen by the compiler's hazard checks: the
//     wait states before any other instruction reads an accumulator are in
//     one statement that takes every accumulator as an operand.
template <int... I, class F>
__device__ __forceinline__ void sfor_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void sfor(F&& f) {
  sfor_impl(std::make_integer_sequence<int, N>{}, f);
}
// direct 16-byte-per-lane load into LDS at m0 = mbase + OFF (uniform); the
// addition sets SCC, which may otherwise hold a loop condition or a carry; the
// s_nop is the wait state between a write of M0 and a load into LDS
template <int OFF>
__device__ __forceinline__ void dma16_at(uint32_t mbase, uint32_t voff, u32x4 desc) {
  asm volatile("s_add_u32 m0, %0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(mbase), "v"(voff), "s"(desc), "n"(OFF)
               : "memory", "scc");
}
// LDS transpose read of one half of a k-major fragment
template <int OFF>
__device__ __forceinline__ void xrd_tr(u32x2& d, uint32_t a) {
  asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(d) : "v"(a), "n"(OFF));
}
// the two halves are (re)defined here: nothing that joins them moves above
__device__ __forceinline__ void xfence(u32x2& a, u32x2& b) {
  asm volatile("" : "+v"(a), "+v"(b));
}
// keep a value's registers allocated up to this point
__device__ __forceinline__ void xkeep(const half8& a) { asm volatile("" ::"v"(a)); }
__device__ __forceinline__ void xkeep(const u32x2& a, const u32x2& b) { asm volatile("" ::"v"(a), "v"(b)); }
// read q of a 4-wave step: fragments in the order B0, A0, B1.., A1..,
// ra (rb) reads per A (B) fragment; op 0 = A, 1 = B
struct X4Rd {
  int op, f, h;
};
constexpr X4Rd x4_read(int q, int tm, int tn, int ra, int rb) {
  for (int e = 0; e < tm + tn; ++e) {
    const int op = e == 0 ? 1 : e == 1 ? 0 : e <= tn ? 1 : 0;
    const int f = e <= 1 ? 0 : e <= tn ? e - 1 : e - tn;
    const int n = op ? rb : ra;
    if (q < n) return X4Rd{op, f, q};
    q -= n;
  }
  return X4Rd{-1, 0, 0};
}
// Schedule of a 4-wave step of nm MFMAs: the slice barrier (second step)
// comes after MFMA x4_bar; the reads of the next step are spread over x4_win
// MFMAs from x4_beg on (second step: behind the barrier).  64 MFMAs per step
// leave room for a wide window; a shorter step needs its reads out early.
constexpr int x4_bar(int nm) { return nm >= 64 ? 1 : nm >= 32 ? 3 : nm >= 16 ? 1 : 1; }
constexpr int x4_beg(int nm, int s) { return s == 1 || nm >= 64 ? x4_bar(nm) + 1 : nm >= 16 ? 1 : 0; }
constexpr int x4_win(int nm) { return nm >= 64 ? 48 : nm >= 32 ? 20 : nm >= 16 ? 4 : 2; }
// reads issued before MFMA idx of a step on set s
constexpr int x4_q0(int idx, int nrd, int nm, int s) {
  const int b = x4_beg(nm, s), w = x4_win(nm);
  const int q = idx < b ? 0 : ((idx - b) * nrd + w - 1) / w;
  return q < nrd ? q : nrd;
}
// direct loads issued before the slot after MFMA idx: n, spread over the
// MFMAs from the barrier on
constexpr int x4_l0(int idx, int n, int nm) {
  const int b = x4_bar(nm), wide = nm / n, tight = (nm - b) / n;
  const int step = b + (n - 1) * wide < nm ? wide : tight > 0 ? tight : 1;
  const int q = idx <= b ? 0 : (idx - b + step - 1) / step;
  return idx >= nm ? n : q < n ? q : n;
}
// LDS read of a K-contiguous fragment
template <int OFF>
__device__ __forceinline__ void xrd(half8& d, uint32_t a) {
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(d) : "v"(a), "n"(OFF));
}
// c becomes a value (and AGPRs) of its own
__device__ __forceinline__ void xown(f32x4& c) { asm volatile("" : "+a"(c)); }
// c += a b (16x16x32), c in AGPRs
__device__ __forceinline__ void xmma(f32x4& c, const half8& a, const half8& b) {
  asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

__device__ __forceinline__ float sigmoid_f(float x) { return 1.f / (1.f + __expf(-x)); }

template <int BM, int BN, int WGM, int WGN, int BK, int NS, bool TA, bool TB, int EPI,
          bool RK = false>
__global__ void __launch_bounds__(WGM * WGN * kWave)
gemm_f16_kernel(int64_t M, int64_t N, int64_t K, float alpha,
                const lt_half* __restrict__ A, int64_t lda,
                const lt_half* __restrict__ B, int64_t ldb, float beta,
                const lt_half* R, int64_t ldr, lt_half* C, int64_t ldc, int tiles_m,
                int tiles_n, int group_m, lt_half* X1, int64_t ldx1, int64_t Fb, int64_t P,
                const lt_half* bias) {
  constexpr int NT = WGM * WGN * kWave;
  constexpr int WTM = BM / WGM, WTN = BN / WGN;   // wave tile
  constexpr int TM = WTM / 16, TN = WTN / 16;     // 16x16 MFMA blocks per wave
  static_assert(EPI != 1 || TB, "paired gate/up tiles: K-contiguous weights");
  // Loader waves: in an 8-wave tile only waves 0-3 (one per SIMD) issue the
  // direct loads, twice as many each; the other four waves only compute.
  // Fewer waves feeding the shared load queues measured 4-13% faster in
  // every layout.
  constexpr int NWAVE = NT / kWave;
  constexpr int LOADERS = NWAVE >= 8 ? 4 : NWAVE;
  constexpr bool SPLIT_ISSUE = LOADERS < NWAVE;
  using OA = Operand<BM, BK, !TA, LOADERS * kWave>;
  // EPI 1: a wave's columns are WTN/2 gate rows and the same WTN/2 up rows
  using OB = Operand<BN, BK, TB, LOADERS * kWave, EPI == 1, WTN / 2>;
  constexpr int STAGE = OA::BYTES + OB::BYTES;
  constexpr int PER_SLICE = OA::PERW + OB::PERW;  // direct loads per wave per slice
  static_assert(NS >= 2 && (NS - 1) * PER_SLICE <= 63, "vmcnt range");
  __shared__ __attribute__((aligned(1024))) char smem[NS * STAGE];

  if constexpr (EPI == 3) {
    // split-K unit blockIdx.y of gridDim.y: slices [y*kc, (y+1)*kc) of the
    // reduction, as a product of its own over the offset operands
    const int64_t kc = ((K + BK - 1) / BK + gridDim.y - 1) / gridDim.y;
    const int64_t k0 = (int64_t)blockIdx.y * kc * BK;
    A += TA ? k0 * lda : k0;
    B += TB ? k0 : k0 * ldb;
    K = K - k0 < kc * BK ? K - k0 : kc * BK;
  }
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar addressing
  const int wm = wave / WGN;
  const int wn = wave % WGN;

  // ---- tile ordering: contiguous range per XCD (consecutive workgroups go
  // to the 8 XCDs in turn), then column-major within groups of group_m
  // tile rows, so that the tiles resident on one XCD share A and B panels ----
  int pid = blockIdx.x;
  const int nwg = gridDim.x;
  if ((nwg & 7) == 0) {
    const int per = nwg >> 3;
    pid = (pid & 7) * per + (pid >> 3);
  }
  const int group_size = group_m * tiles_n;
  const int first_m = (pid / group_size) * group_m;
  const int gm = min(tiles_m - first_m, group_m);
  const int in_group = pid % group_size;
  const int64_t m0 = (int64_t)(first_m + in_group % gm) * BM;
  // EPI 1: a tile covers BN/2 gate columns and the same BN/2 up columns
  const int64_t n0 = (int64_t)(in_group / gm) * (EPI == 1 ? BN / 2 : BN);

  OA oa;
  OB ob;
  // (waves that load nothing set their operands up too: behind a branch the
  // buffer ranges would not stay in scalar registers)
  const bool loader = !SPLIT_ISSUE || wave < LOADERS;
  oa.init(A, lda, m0, M, wave, lane);
  if constexpr (EPI == 1) ob.init(B, ldb, n0, Fb, wave, lane, P);
  else ob.init(B, ldb, n0, N, wave, lane);

  f32x4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

  const int nk = (int)((K + BK - 1) / BK);
  // (K is at most 2^30: 32-bit sums stay in scalar registers, as in init)
  auto kvalid = [&](int kt) {
    const int rem = (int)K - kt * BK;
    return rem >= BK ? BK : rem;
  };
  auto stage_of = [&](int kt) { return smem + (kt % NS) * STAGE; };
  auto issue = [&](int kt) {
    if (!loader) return;
    char* st = stage_of(kt);
    oa.load(st, (int64_t)kt * BK, kvalid(kt), wave, lane);
    ob.load(st + OA::BYTES, (int64_t)kt * BK, kvalid(kt), wave, lane);
  };
  // RK (ragged K, not a multiple of 8; plain epilogue only): the last
  // slice's K-contiguous tiles are cleared past K, between two barriers.  A
  // separate instantiation, so that no branch sits at the slice barrier of
  // the other kernels (their first MFMAs after it are scheduled across it).
  static_assert(!RK || EPI == 0, "ragged K: plain epilogue");
  constexpr bool KFIX = RK && (!TA || TB);
  static_assert(!KFIX || (TA ? 0 : BM) + (TB ? BN : 0) <= NT, "one thread per tile row");
  auto fix_k_tail = [&](int kt) {
    if constexpr (KFIX) {
      char* st = stage_of(kt);
      const int kv = kvalid(kt);
      if constexpr (!TA) oa.zero_k_tail(st, kv, tid);
      if constexpr (TB) ob.zero_k_tail(st + OA::BYTES, kv, TA ? tid : tid - BM);
      __syncthreads();
    }
  };
  constexpr bool ragged_k = KFIX;

  constexpr bool X4 = NT == 256 && BK == 64 && !RK && EPI <= 3;
  if constexpr (X4) {
    // One wave per SIMD, 2x2 wave grid, accumulators in AGPRs.  Every
    // fragment read, MFMA and counter wait of the loop is an ordered asm
    // statement: a step's MFMAs run on one register set while the reads of
    // the next step fill the other; after the slice barrier the direct loads
    // of slice kt+NS are spread over the step's MFMAs.
    //   256x256 tiles: two 64 KiB LDS stages; 16 loads, 128 MFMAs a slice, so
    //     one slice of lead covers the load latency.  Slices run in pairs, so
    //     that both stage offsets are compile-time constants.
    //   smaller tiles: a slice is 1/2 to 1/16 of that work, so the LDS holds
    //     3 to 8 stages instead and loads run NS - 1 slices ahead; the stage is a
    //     uniform offset, added to the fragment addresses once per step.
    constexpr bool AK = !TA, BKC = TB;           // K-contiguous operands (row reads)
    constexpr bool DYN = NS > 2;
    static_assert(DYN || (BM == 256 && BN == 256), "two stages: 256x256 tiles");
    static_assert(NS * STAGE <= 160 * 1024 && NS * PER_SLICE <= 63, "stages");
    constexpr int XRA = AK ? 1 : 2, XRB = BKC ? 1 : 2;
    constexpr int NRD = TM * XRA + TN * XRB;    // LDS reads per step
    constexpr int NM = TM * TN;                 // MFMAs per step
    constexpr int BAR = x4_bar(NM);
    half8 xa[2][TM], xb[2][TN];                // fragments of K-contiguous operands
    u32x2 ta[2][TM][2], tb[2][TN][2];          // ... of k-major ones (two transpose reads)
    const uint32_t sbase = (uint32_t)(uintptr_t)smem;
    // K-contiguous: fragment f of k-step kk at r[stage][kk] + 2048 f
    auto lterm = [&](int kk) {
      const int r = lane & 15;
      const int c = kk * 4 + (lane >> 4);
      return (uint32_t)(r * 128 + ((c ^ (r >> 1)) << 4));
    };
    // k-major: read h of fragment f, k-step kk at z[stage][f] + 64 R kk + 8 R h
    // for R rows (the fragment's XOR-swizzled position differs per lane only
    // in address bits 5..7, which no other term touches); rb = first row
    auto zaddr = [&](auto R_, int rb) {
      constexpr int R = decltype(R_)::value;
      const uint32_t kl = (lane >> 2) & 3, g1 = (lane >> 4) & 1;
      const uint32_t k = 8 * (lane >> 4) + kl;
      const uint32_t x = 16 * ((lane & 3) >> 1) + 8 * (lane & 1);
      if constexpr (R == 64)
        return k * 128 + (((uint32_t)(rb >> 4) ^ ((kl >> 1) | (g1 << 1))) << 5) + x;
      else
        return k * (2 * R) + 256 * (uint32_t)(rb >> 7) +
               ((((uint32_t)((rb >> 5) & 3) ^ kl) << 6) | (((uint32_t)((rb >> 4) & 1) ^ g1) << 5)) + x;
    };
    constexpr int NP = DYN ? 1 : 2;             // stages with addresses of their own
    uint32_t ra[NP][2], rb[NP][2], za[NP][TM], zb[NP][TN];
#pragma unroll
    for (int p = 0; p < NP; ++p) {
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        ra[p][kk] = sbase + p * STAGE + wm * (WTM * 128) + lterm(kk);
        rb[p][kk] = sbase + p * STAGE + OA::BYTES + wn * (WTN * 128) + lterm(kk);
      }
#pragma unroll
      for (int f = 0; f < TM; ++f)
        za[p][f] = sbase + p * STAGE + zaddr(std::integral_constant<int, BM>{}, wm * WTM + 16 * f);
#pragma unroll
      for (int f = 0; f < TN; ++f)
        zb[p][f] = sbase + p * STAGE + OA::BYTES + zaddr(std::integral_constant<int, BN>{}, wn * WTN + 16 * f);
    }
    // read q of the step into set D, from stage P (DYN: from the stage at
    // offset so), k-step KK
    auto xread = [&](auto Q_, auto D_, auto P_, auto KK_, uint32_t so) __attribute__((always_inline)) {
      constexpr X4Rd r = x4_read(decltype(Q_)::value, TM, TN, XRA, XRB);
      constexpr int D = decltype(D_)::value, P = DYN ? 0 : decltype(P_)::value, KK = decltype(KK_)::value;
      if constexpr (r.op == 0) {
        if constexpr (AK) xrd<r.f * 2048>(xa[D][r.f], DYN ? ra[P][KK] + so : ra[P][KK]);
        else xrd_tr<KK * 64 * BM + r.h * 8 * BM>(ta[D][r.f][r.h], DYN ? za[P][r.f] + so : za[P][r.f]);
      } else {
        if constexpr (BKC) xrd<r.f * 2048>(xb[D][r.f], DYN ? rb[P][KK] + so : rb[P][KK]);
        else xrd_tr<KK * 64 * BN + r.h * 8 * BN>(tb[D][r.f][r.h], DYN ? zb[P][r.f] + so : zb[P][r.f]);
      }
    };
    // before MFMA idx of a step on set S: the fragments it is the first to use
    // have landed; the k-major halves are joined only after the wait.
    //   256x256: one wait for the whole set at the step's start, normally
    //     already met (the reads had the last 16 MFMAs to land).
    //   smaller tiles: LDS reads land in order and are issued in the order of
    //     first use, so each first use waits until only the reads behind it
    //     may be outstanding: this set's later ones and the q0(idx) reads of
    //     the next set issued so far.  No scalar load may be in flight then (it
    //     shares the counter): none is in the loop, and the loop is entered
    //     with the counter at zero.
    auto xwait = [&](auto S_, auto IDX_) __attribute__((always_inline)) {
      constexpr int S = decltype(S_)::value, idx = decltype(IDX_)::value;
      if constexpr (DYN) {
        constexpr int i = idx / TN, j = idx % TN;
        if constexpr (i == 0 || j == 0) {
          // reads of this set up to the later of its first-used fragments
          constexpr int pos = i > 0 ? TN * XRB + (i + 1) * XRA : (j + 1) * XRB + XRA;
          constexpr int left = NRD - pos + x4_q0(idx, NRD, NM, S);
          asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(left < 15 ? left : 15) : "memory");
          if constexpr (!AK && j == 0) xfence(ta[S][i][0], ta[S][i][1]);
          if constexpr (!BKC && i == 0) xfence(tb[S][j][0], tb[S][j][1]);
        }
      } else if constexpr (idx == 0) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if constexpr (!AK) {
#pragma unroll
          for (int f = 0; f < TM; ++f) xfence(ta[S][f][0], ta[S][f][1]);
        }
        if constexpr (!BKC) {
#pragma unroll
          for (int f = 0; f < TN; ++f) xfence(tb[S][f][0], tb[S][f][1]);
        }
      }
    };
    auto fragA = [&](auto S_, int i) __attribute__((always_inline)) {
      constexpr int S = decltype(S_)::value;
      if constexpr (AK) return xa[S][i];
      else return __builtin_bit_cast(half8, __builtin_shufflevector(ta[S][i][0], ta[S][i][1], 0, 1, 2, 3));
    };
    auto fragB = [&](auto S_, int j) __attribute__((always_inline)) {
      constexpr int S = decltype(S_)::value;
      if constexpr (BKC) return xb[S][j];
      else return __builtin_bit_cast(half8, __builtin_shufflevector(tb[S][j][0], tb[S][j][1], 0, 1, 2, 3));
    };
    using Z0 = std::integral_constant<int, 0>;
    using Z1 = std::integral_constant<int, 1>;
    // Every accumulator starts as a value of its own.  As copies of one zero
    // the compiler may give an accumulator another register behind the first
    // loop than inside it, and the move at that loop's exit reads it before
    // its last MFMA has written it (asm MFMAs are outside the hazard checks).
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) xown(acc[i][j]);
    // prologue: slices 0 .. NS-1 in flight (those past K fill their stage
    // with zeros), slice 0 resident, its first k-step's fragments into set 0
    auto kv_of = [&](int kt) {
      const int rem = (int)K - kt * BK;
      return rem >= BK ? BK : rem > 0 ? rem : 0;
    };
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
#pragma unroll
      for (int t = 0; t < (OA::PERW > OB::PERW ? OA::PERW : OB::PERW); ++t) {
        if (t < OA::PERW)
          oa.load1(smem + sl * STAGE, (int64_t)sl * BK, kv_of(sl), t, wave, lane);
        if (t < OB::PERW)
          ob.load1(smem + sl * STAGE + OA::BYTES, (int64_t)sl * BK, kv_of(sl), t, wave, lane);
      }
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * PER_SLICE) : "memory");
    __syncthreads();
    sfor<NRD>([&](auto Q) __attribute__((always_inline)) { xread(Q, Z0{}, Z0{}, Z0{}, 0u); });
    if constexpr (DYN) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    const uint32_t mbase_a = __builtin_amdgcn_readfirstlane(sbase + wave * OA::PERW * 1024);
    const uint32_t mbase_b = __builtin_amdgcn_readfirstlane(sbase + OA::BYTES + wave * OB::PERW * 1024);
    // One 32-wide k-step on set S; the next step's fragments come from
    // stage P (DYN: the stage at offset so), k-step KK.  LD: 0 no loads, 1
    // loads of any slice at lk0 (lkv valid columns, masked), 2 loads of a full
    // slice through the descriptors dA, dB; into stage LP (DYN: at offset lo).
    auto xstep = [&](auto S_, auto P_, auto KK_, uint32_t so, auto LD_, int64_t lk0, int lkv, auto LP_,
                     uint32_t lo, u32x4 dA, u32x4 dB) __attribute__((always_inline)) {
      constexpr int S = decltype(S_)::value;
      constexpr int LD = decltype(LD_)::value;
      constexpr int LO = DYN ? 0 : decltype(LP_)::value * STAGE;
      sfor<NM>([&](auto IDX) __attribute__((always_inline)) {
        constexpr int idx = decltype(IDX)::value;
        constexpr int i = idx / TN, j = idx % TN;
        xwait(S_, IDX);
        xmma(acc[i][j], fragB(S_, j), fragA(S_, i));
        // the slice barrier after the second step's first MFMAs (they run on
        // registers and cover the barrier's skew): slice kt+1 resident for
        // every wave, and nobody reads slice kt's stage any more
        if constexpr (S == 1 && idx == BAR) {
          // (the stage's last reads, those of set 1, have landed here)
          if constexpr (DYN)
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NS - 2) * PER_SLICE) : "memory");
          else
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * PER_SLICE) : "memory");
          __syncthreads();
        }
        constexpr int q0 = x4_q0(idx, NRD, NM, S), q1 = idx == NM - 1 ? NRD : x4_q0(idx + 1, NRD, NM, S);
        sfor<q1 - q0>([&](auto R_) __attribute__((always_inline)) {
          xread(std::integral_constant<int, q0 + decltype(R_)::value>{}, std::integral_constant<int, S ^ 1>{}, P_,
                KK_, so);
        });
        constexpr int l0 = x4_l0(idx, PER_SLICE, NM), l1 = x4_l0(idx + 1, PER_SLICE, NM);
        if constexpr (LD != 0 && idx >= BAR)
          sfor<l1 - l0>([&](auto T_) __attribute__((always_inline)) {
            constexpr int t = l0 + decltype(T_)::value;
            if constexpr (LD == 1) {
              if constexpr (t < OA::PERW) oa.load1(smem + LO + lo, lk0, lkv, t, wave, lane);
              else ob.load1(smem + LO + lo + OA::BYTES, lk0, lkv, t - OA::PERW, wave, lane);
            } else {
              if constexpr (t < OA::PERW)
                dma16_at<LO + t * 1024>(DYN ? mbase_a + lo : mbase_a, oa.voff[t], dA);
              else
                dma16_at<LO + (t - OA::PERW) * 1024>(DYN ? mbase_b + lo : mbase_b, ob.voff[t - OA::PERW], dB);
            }
          });
      });
    };
    using NO = std::integral_constant<int, 0>;
    using YS = std::integral_constant<int, 1>;
    using FS = std::integral_constant<int, 2>;
    const u32x4 dz = {0, 0, 0, 0};
    // slice kt in stage P (DYN: at offset so; the next slice's at sn): its two
    // steps, and the loads of slice kt + NS into the stage it frees
    auto xslice = [&](int kt, auto P_, uint32_t so, uint32_t sn, auto FAST_) __attribute__((always_inline)) {
      constexpr int P = decltype(P_)::value;
      constexpr bool FAST = decltype(FAST_)::value;
      xstep(Z0{}, P_, Z1{}, so, NO{}, 0, 0, P_, 0u, dz, dz);
      const int64_t lk0 = (int64_t)(kt + NS) * BK;
      if constexpr (FAST)
        xstep(Z1{}, std::integral_constant<int, P ^ 1>{}, Z0{}, sn, FS{}, 0, 0, P_, so, oa.desc(lk0),
              ob.desc(lk0));
      else
        xstep(Z1{}, std::integral_constant<int, P ^ 1>{}, Z0{}, sn, YS{}, lk0, kv_of(kt + NS), P_, so, dz, dz);
    };
    // slices whose loads (slice kt + NS) are whole slices inside K take the
    // unmasked loads
    const int nkf = (int)(K / BK);
    int kt = 0;
    if constexpr (DYN) {
      uint32_t so = 0;
      auto next = [&](uint32_t s_) { return s_ + STAGE == NS * STAGE ? 0u : s_ + STAGE; };
      for (; kt + NS < nkf; ++kt) {
        const uint32_t sn = next(so);
        xslice(kt, Z0{}, so, sn, std::true_type{});
        so = sn;
      }
      for (; kt < nk; ++kt) {
        const uint32_t sn = next(so);
        xslice(kt, Z0{}, so, sn, std::false_type{});
        so = sn;
      }
    } else {
      // Pairs of slices (stage 0, stage 1).  For an odd slice count the last
      // pair's second slice lies past K: its stage was filled with zeros, so
      // its products add exact zeros (an accumulator that starts at +0 never
      // holds -0), and the loop body has no branch.
      for (; kt + 3 < nkf; kt += 2) {
        xslice(kt, Z0{}, 0u, 0u, std::true_type{});
        xslice(kt + 1, Z1{}, 0u, 0u, std::true_type{});
      }
      for (; kt < nk; kt += 2) {
        xslice(kt, Z0{}, 0u, 0u, std::false_type{});
        xslice(kt + 1, Z1{}, 0u, 0u, std::false_type{});
      }
    }
    // The last step read the fragments of a step that never runs: their
    // registers stay allocated until those reads have landed, so that no
    // epilogue value is placed where a late LDS result would overwrite it.
    // The MFMAs are opaque to the compiler's hazard checks: the wait states
    // before the accumulators may be read sit in one statement that takes
    // every accumulator, so no spill or copy of one can be placed between
    // the last MFMA and the wait.
#define X4_W2(i) "+a"(acc[i][0]), "+a"(acc[i][1])
#define X4_W4(i) X4_W2(i), "+a"(acc[i][2]), "+a"(acc[i][3])
#define X4_W8(i) X4_W4(i), "+a"(acc[i][4]), "+a"(acc[i][5]), "+a"(acc[i][6]), "+a"(acc[i][7])
#define X4_END(...)                                                                       \
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7\n\t"     \
               "s_nop 7\n\ts_nop 7\n\ts_nop 7\n\ts_nop 7"                                 \
               : __VA_ARGS__                                                              \
               :                                                                          \
               : "memory")
    if constexpr (TM == 8 && TN == 8)
      X4_END(X4_W8(0), X4_W8(1), X4_W8(2), X4_W8(3), X4_W8(4), X4_W8(5), X4_W8(6), X4_W8(7));
    else if constexpr (TM == 8 && TN == 4)
      X4_END(X4_W4(0), X4_W4(1), X4_W4(2), X4_W4(3), X4_W4(4), X4_W4(5), X4_W4(6), X4_W4(7));
    else if constexpr (TM == 4 && TN == 8)
      X4_END(X4_W8(0), X4_W8(1), X4_W8(2), X4_W8(3));
    else if constexpr (TM == 4 && TN == 4)
      X4_END(X4_W4(0), X4_W4(1), X4_W4(2), X4_W4(3));
    else {
      static_assert(TM == 2 && TN == 2, "wave tiles of the 4-wave loop");
      X4_END(X4_W2(0), X4_W2(1));
    }
#undef X4_W2
#undef X4_W4
#undef X4_W8
#undef X4_END
#pragma unroll
    for (int f = 0; f < TM; ++f) {
      if constexpr (AK) xkeep(xa[0][f]);
      else xkeep(ta[0][f][0], ta[0][f][1]);
    }
#pragma unroll
    for (int f = 0; f < TN; ++f) {
      if constexpr (BKC) xkeep(xb[0][f]);
      else xkeep(tb[0][f][0], tb[0][f][1]);
    }
  } else {
  // Fragments: A in place (each re-read right after its last use), B
  // double-buffered (used by every A row of a step).
  half8 fa[TM], fb[2][TN];

  // ---- prologue: slices 0 .. NS-1 in flight, wait for slice 0 ----
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < nk) issue(s);
  wait_slices<PER_SLICE, NS - 1>(min(NS - 1, nk - 1));
  __syncthreads();
  if (ragged_k && nk == 1) fix_k_tail(0);

  // One MFMA step on (fa, fb[S]).  With LD, the fragments of the next step
  // (32-wide k-step kk of stage st) are read meanwhile: after the MFMAs of A
  // row i come the reads of fa[i] and, for the first TN rows, of fb[S^1][i],
  // so every read overlaps the MFMAs that follow it.  S and LD are
  // compile-time constants so that the fragment arrays stay in registers.
  constexpr int KS = BK / 32;
  static_assert(KS % 2 == 0, "B fragments alternate buffers within a slice");
  constexpr int RA = TA ? 2 : 1;   // LDS reads per A fragment (transpose reads: 2)
  constexpr int RB = TB ? 1 : 2;   // ... per B fragment
  // B fragments read after A row i: fb[j] for j % TM == i (BPI of them while
  // i < NBI; one for each of the first TN rows when TN <= TM).
  static_assert(TN <= TM || TN % TM == 0, "B fragments must spread over the A rows");
  constexpr int BPI = TN <= TM ? 1 : TN / TM;
  constexpr int NBI = TN <= TM ? TN : TM;
  // First fragments, read in the order the steps read theirs (after A row i:
  // the B fragments of row i, then A fragment i).  The LDS counter waits at
  // the top of the slice loop then hold for the entry from here as well as
  // for the loop's back edge; with all B fragments read last, the waits the
  // compiler derived for the merged entry stalled each slice's first MFMAs
  // on the reads of the previous step's last rows.
  if (nk > 0) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (i < NBI) {
#pragma unroll
        for (int q = 0; q < BPI; ++q)
          fb[0][i + q * TM] = ob.frag(smem + OA::BYTES, wn * WTN + (i + q * TM) * 16, 0, lane);
      }
      fa[i] = oa.frag(smem, wm * WTM + i * 16, 0, lane);
    }
  }
  auto step = [&](auto S_, auto LD_, const char* st, int kk, auto&& after_first_row) {
    constexpr int S = decltype(S_)::value;
    constexpr bool LD = decltype(LD_)::value;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = mfma16(fb[S][j], fa[i], acc[i][j]);
      if (i == 0) after_first_row(std::integral_constant<int, 0>{});
      if (i == TM / 2) after_first_row(std::integral_constant<int, 1>{});
      if constexpr (LD) {
        if (i < NBI) {
#pragma unroll
          for (int q = 0; q < BPI; ++q) {
            const int j = i + q * TM;
            fb[S ^ 1][j] = ob.frag(st + OA::BYTES, wn * WTN + j * 16, kk, lane);
          }
        }
        fa[i] = oa.frag(st, wm * WTM + i * 16, kk, lane);
      }
    }
    if constexpr (LD) {
#pragma unroll
      for (int i = 0; i < NBI; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, TN, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, BPI * RB + RA, 0);
      }
#pragma unroll
      for (int i = NBI; i < TM; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, TN, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, RA, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  using C0 = std::integral_constant<int, 0>;
  using C1 = std::integral_constant<int, 1>;
  using YES = std::integral_constant<bool, true>;

  // Per slice kt: step 0, then the barrier after which slice kt+1 is
  // resident and nobody reads slice kt's stage any more.  Step 1 runs on
  // registers while reading slice kt+1's first fragments; after its first
  // MFMAs are queued, the loads of slice kt+NS go into the freed stage,
  // almost a full slice ahead of their wait.
  for (int kt = 0; kt < nk; ++kt) {
    static_assert(KS == 2, "one step before and one after the slice barrier");
    step(C0{}, YES{}, stage_of(kt), 1, [](auto) {});
    // slices after kt+1 that are already issued may stay in flight
    wait_slices<PER_SLICE, NS - 2>(min(kt + NS - 1, nk - 1) - (kt + 1));
    __syncthreads();
    if (ragged_k && kt + 2 == nk) fix_k_tail(kt + 1);
    // (after the last slice these reads of a stale stage are unused; reading
    // unconditionally keeps one copy of the fragments live across the loop)
    step(C1{}, YES{}, stage_of(kt + 1), 0, [&](auto part) {
      constexpr int PART = decltype(part)::value;
      if (!loader || kt + NS >= nk) return;
      if constexpr (!SPLIT_ISSUE) {
        if constexpr (PART == 0) issue(kt + NS);
      } else {
        // loader waves: A's loads after the first A row, B's after row TM/2
        char* st = stage_of(kt + NS);
        if constexpr (PART == 0)
          oa.load(st, (int64_t)(kt + NS) * BK, kvalid(kt + NS), wave, lane);
        else
          ob.load(st + OA::BYTES, (int64_t)(kt + NS) * BK, kvalid(kt + NS), wave, lane);
      }
    });
  }

  }  // !X4

  // ---- epilogue ----
  // lane holds column m = ... + lane % 16 and rows n = ... + 4*(lane/16) + 0..3
  if constexpr (EPI == 3) {
    // FP32 partial sums of this split, unscaled: W[split][m][n], ldc floats
    // per row (C is the workspace)
    float* W = reinterpret_cast<float*>(C) + (int64_t)blockIdx.y * M * ldc;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int64_t m = m0 + wm * WTM + i * 16 + (lane & 15);
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        const int64_t n = n0 + wn * WTN + j * 16 + 4 * (lane >> 4);
        if (m < M && n < N)
          *reinterpret_cast<float4*>(W + m * ldc + n) =
              make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
      }
    }
  } else {
    // Each wave passes its accumulators through LDS, 16 rows at a time (FP32,
    // wave-private, rows 16 bytes apart in the banks), so that a lane gets
    // 8 consecutive columns of one row: R, G, U and bias are then read and
    // results written 16 bytes per lane, whole 128-byte lines per row.  In
    // the accumulator layout a store instruction touched 16 rows with 32
    // bytes each.
    constexpr int NC = EPI == 1 ? WTN / 2 : WTN;       // output columns of the wave
    constexpr int CH = NC / 8;                         // 8-column chunks per row
    constexpr int RPP = 64 / CH < 16 ? 64 / CH : 16;   // rows per pass over the lanes
    constexpr int NPASS = 16 / RPP;
    constexpr int PITCH = WTN + 4;                     // floats per staged row
    constexpr int NL = EPI == 2 ? 2 : 1;               // 16-byte reads per chunk
    constexpr int PF = TM < 3 ? TM : 3;                // row groups of reads in flight
    static_assert(NWAVE * 16 * PITCH * 4 <= NS * STAGE, "staging fits in LDS");
    const bool reads = EPI == 2 || (EPI == 0 && beta != 0.f);   // uniform over the grid
    const bool has_bias = EPI == 0 && bias != nullptr;
    const int64_t ncols = EPI == 1 ? Fb : N;
    const int crow = lane / CH, ccol = 8 * (lane % CH);
    const bool lane_on = 64 / CH <= 16 || crow < 16;   // 16-column tiles: half the lanes
    const int64_t mb = m0 + wm * WTM + crow;
    const int64_t n = n0 + wn * NC + ccol;
    // loads still in flight (the slices past K) and other waves' last reads
    // of the stages come first
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    float* stg = reinterpret_cast<float*>(smem) + wave * (16 * PITCH);
    float* const wr = stg + (lane & 15) * PITCH + 4 * (lane >> 4);
    const float* const rd = stg + (lane_on ? crow : 0) * PITCH + ccol;
    half8 bv;
    if (has_bias) {
#pragma unroll
      for (int e = 0; e < 8; ++e) bv[e] = (_Float16)0;
      if (n + 8 <= N) {
        bv = as_half8(ld16(bias + n));
      } else {
        // bias holds exactly N entries
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (n + e < N) bv[e] = __builtin_bit_cast(_Float16, bias[n + e]);
      }
    }
    // FULL: the whole tile lies inside the matrix -- no branch between the
    // loads and stores, which keeps the completion-counter waits exact.
    // Otherwise loads come from addresses clamped into the matrix (values of
    // out-of-range chunks are never stored; a chunk that starts before N is
    // read whole: rows are readable up to N rounded up to 8, as leading
    // dimensions are multiples of 8).  R may be C itself: every row group is
    // read before any group from it on is stored.
    auto finish = [&](auto FULL_) __attribute__((always_inline)) {
      constexpr bool FULL = decltype(FULL_)::value;
      half8 in[PF][NPASS][NL];
      auto load_group = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
          const int64_t m = mb + i * 16 + p * RPP;
          const int64_t mc = FULL || m < M ? m : M - 1;
          const int64_t nc = FULL || n < N ? n : 0;
          if constexpr (EPI == 2) {
            in[i % PF][p][0] = as_half8(ld16(X1 + mc * ldx1 + nc));
            in[i % PF][p][NL - 1] = as_half8(ld16(X1 + mc * ldx1 + P + nc));
          } else {
            in[i % PF][p][0] = as_half8(ld16(R + mc * ldr + nc));
          }
        }
      };
      auto stage_group = [&](int i) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<f32x4*>(wr + 16 * j) = acc[i][j];
      };
      auto put = [&](lt_half* dst, const half8& v) __attribute__((always_inline)) {
        if (FULL || EPI != 0 || n + 8 <= N) {
          st16(dst, as_u32x4(v));
        } else {
          // the last 1-7 columns of a ragged N, taken from the packed bits
          // (the element-indexed form of such stores compiled to stores of
          // element 0 only)
          const u32x4 w = as_u32x4(v);
#pragma unroll
          for (int e = 0; e < 7; ++e)
            if (n + e < N) dst[e] = (lt_half)(w[e / 2] >> (16 * (e & 1)));
        }
      };
      if (reads) {
#pragma unroll
        for (int i = 0; i < PF; ++i) load_group(i);
      }
      stage_group(0);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        f32x4 raw[NPASS][EPI == 1 ? 4 : 2];
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
          const float* q = rd + p * RPP * PITCH;
          raw[p][0] = *reinterpret_cast<const f32x4*>(q);
          raw[p][1] = *reinterpret_cast<const f32x4*>(q + 4);
          if constexpr (EPI == 1) {
            raw[p][2] = *reinterpret_cast<const f32x4*>(q + NC);
            raw[p][3] = *reinterpret_cast<const f32x4*>(q + NC + 4);
          }
        }
        // (a wave's LDS accesses run in order: the next group may follow at once)
        if (i + 1 < TM) stage_group(i + 1);
        // one wait for the group's reads, before their first use
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        float v[NPASS][8], u[EPI == 1 ? NPASS : 1][8];
#pragma unroll
        for (int p = 0; p < NPASS; ++p)
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            v[p][e] = alpha * raw[p][e / 4][e % 4];
            if constexpr (EPI == 1) u[p][e] = alpha * raw[p][2 + e / 4][e % 4];
          }
#pragma unroll
        for (int p = 0; p < NPASS; ++p) {
          const int64_t m = mb + i * 16 + p * RPP;
          const bool on = (FULL || (m < M && n < ncols)) && lane_on;
          half8 o0, o1, o2;
          if constexpr (EPI == 1) {
            // GU[m][n] = G, GU[m][F + n] = U, A[m][n] = silu(G) U (from the
            // FP32 values, one rounding each)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float g = v[p][e];
              o0[e] = (_Float16)g;
              o1[e] = (_Float16)u[p][e];
              o2[e] = (_Float16)(g * sigmoid_f(g) * u[p][e]);
            }
          } else if constexpr (EPI == 2) {
            // v = dA; dG = dA U s (1 + G (1 - s)),  dU = dA silu(G),  s = sigmoid(G)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float gv = (float)in[i % PF][p][0][e], uv = (float)in[i % PF][p][NL - 1][e];
              const float sg = sigmoid_f(gv);
              o0[e] = (_Float16)(v[p][e] * uv * sg * (1.f + gv * (1.f - sg)));
              o1[e] = (_Float16)(v[p][e] * gv * sg);
            }
          } else {
            if (reads) {
#pragma unroll
              for (int e = 0; e < 8; ++e) v[p][e] += beta * (float)in[i % PF][p][0][e];
            }
            if (has_bias) {
#pragma unroll
              for (int e = 0; e < 8; ++e) v[p][e] += (float)bv[e];
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) o0[e] = (_Float16)v[p][e];
          }
          if ((FULL && 64 / CH <= 16) || on) {
            put(C + m * ldc + n, o0);
            if constexpr (EPI != 0) put(C + m * ldc + P + n, o1);
            if constexpr (EPI == 1) put(X1 + m * ldx1 + n, o2);
          }
        }
        if (reads && i + PF < TM) load_group(i + PF);
      }
    };
    if (m0 + BM <= M && n0 + (EPI == 1 ? BN / 2 : BN) <= ncols)
      finish(std::true_type{});
    else
      finish(std::false_type{});
  }
}

template <int BM, int BN, int WGM, int WGN, int BK, int NS, bool TA, bool TB, int EPI,
          bool RK = false>
hipError_t launch(const GemmArgs& g, hipStream_t s, int splits = 1) {
  const int tiles_m = (int)((g.M + BM - 1) / BM);
  const int tiles_n = EPI == 1 ? (int)((g.F + BN / 2 - 1) / (BN / 2)) : (int)((g.N + BN - 1) / BN);
  hipLaunchKernelGGL((gemm_f16_kernel<BM, BN, WGM, WGN, BK, NS, TA, TB, EPI, RK>),
                     dim3(tiles_m * tiles_n, splits), dim3(WGM * WGN * kWave), 0, s, g.M, g.N, g.K, g.alpha,
                     g.A, g.lda, g.B, g.ldb, g.beta, g.R, g.ldr, g.C, g.ldc, tiles_m, tiles_n, 8,
                     g.X1, g.ldx1, g.F, g.pair_off > 0 ? g.pair_off : g.F, g.bias);
  return hipGetLastError();
}

// The same product restricted to output columns [n0, ...) (in units of
// output columns; for the gate/up epilogue, of gate columns).
template <bool TA, bool TB, int EPI>
GemmArgs column_part(const GemmArgs& g, int64_t n0) {
  GemmArgs t = g;
  if (EPI == 1) {
    t.pair_off = g.pair_off > 0 ? g.pair_off : g.F;
    t.B = g.B + n0 * g.ldb;        // gate rows n0..; up rows stay pair_off further
    t.F = g.F - n0;
    t.N = 2 * t.F;
    t.C = g.C + n0;
    t.X1 = g.X1 + n0;
  } else {
    t.B = TB ? g.B + n0 * g.ldb : g.B + n0;
    t.N = g.N - n0;
    t.C = g.C + n0;
    t.R = g.R + n0;
    if (g.bias) t.bias = g.bias + n0;
    if (EPI == 2) {
      t.pair_off = g.pair_off > 0 ? g.pair_off : g.F;
      t.X1 = g.X1 + n0;
    }
  }
  return t;
}

// ... restricted to output rows [m0, ...).
template <bool TA, bool TB, int EPI>
GemmArgs row_part(const GemmArgs& g, int64_t m0) {
  GemmArgs t = g;
  t.A = TA ? g.A + m0 : g.A + m0 * g.lda;
  t.M = g.M - m0;
  t.C = g.C + m0 * g.ldc;
  t.R = g.R + m0 * g.ldr;
  if (EPI != 0) t.X1 = g.X1 + m0 * g.ldx1;
  return t;
}

// C = alpha * sum_s W[s] + beta * R + bias over an Mt x Nt region, the
// splits summed in ascending order; eight columns per thread (Nt % 8 == 0).
__global__ void __launch_bounds__(256)
splitk_reduce_kernel(const float* __restrict__ W, int S, int64_t Mt, int64_t Nt, float alpha,
                     float beta, const lt_half* R, int64_t ldr, const lt_half* __restrict__ bias,
                     lt_half* C, int64_t ldc) {
  const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t n8 = Nt / 8;
  if (idx >= Mt * n8) return;
  const int64_t m = idx / n8, n = (idx % n8) * 8;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = 0.f;
  for (int sp = 0; sp < S; ++sp) {
    const float* w = W + ((int64_t)sp * Mt + m) * Nt + n;
    const float4 a = *reinterpret_cast<const float4*>(w);
    const float4 b = *reinterpret_cast<const float4*>(w + 4);
    v[0] += a.x; v[1] += a.y; v[2] += a.z; v[3] += a.w;
    v[4] += b.x; v[5] += b.y; v[6] += b.z; v[7] += b.w;
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] *= alpha;
  if (beta != 0.f) {
    const half8 r = as_half8(ld16(R + m * ldr + n));
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += beta * (float)r[e];
  }
  if (bias) {
    const half8 bb = as_half8(ld16(bias + n));
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += (float)bb[e];
  }
  half8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (_Float16)v[e];
  *reinterpret_cast<half8*>(C + m * ldc + n) = o;
}

// one launch of one tile size; LDS stages: two of 64 KiB, three of 48, four of
// 32, eight of 16 (five of 32 and ten of 16, all that fit 160 KiB, are level to
// 7% slower: 1024 x 1024 x 4096 TN 20.4 us against 19.0)
template <bool TA, bool TB, int EPI>
hipError_t launch_tile(int tile, const GemmArgs& g, hipStream_t s) {
  switch (tile) {
    case kTile256: return launch<256, 256, 2, 2, 64, 2, TA, TB, EPI>(g, s);
    case kTile256x128: return launch<256, 128, 2, 2, 64, 3, TA, TB, EPI>(g, s);
    case kTile128x256: return launch<128, 256, 2, 2, 64, 3, TA, TB, EPI>(g, s);
    case kTile128: return launch<128, 128, 2, 2, 64, 4, TA, TB, EPI>(g, s);
    default: return launch<64, 64, 2, 2, 64, 8, TA, TB, EPI>(g, s);
  }
}

template <bool TA, bool TB, int EPI>
hipError_t dispatch_tile(const GemmArgs& g, hipStream_t s) {
  if constexpr (EPI == 0 && (!TA || TB)) {
    // K not a multiple of 8 with a K-contiguous operand: one launch of the
    // tiles with the last slice's fix-up (256x256 from about one wave of
    // them).  Weight gradients (both operands k-major) load whole k-rows and
    // need no fix-up.
    if (g.K & 7) {
      if (((g.M + 255) / 256) * ((g.N + 255) / 256) >= 192)
        return launch<256, 256, 2, 4, 64, 2, TA, TB, 0, true>(g, s);
      return launch<128, 128, 2, 2, 64, 2, TA, TB, 0, true>(g, s);
    }
  }
  const bool split_k = EPI == 0 && g.ws != nullptr && gemm_splitk_ws_bytes(g.M, g.N, g.K) <= g.ws_bytes;
  const GemmPlan p = gemm_plan(TA, g.M, EPI == 1 ? g.F : g.N, g.K, EPI, EPI == 0 && g.beta != 0.f, split_k,
                               ((g.lda | g.ldb) & 63) != 0);
  GemmArgs tail = g;
  if (p.split_at > 0) {
    GemmArgs head = g;
    if (!p.columns) {
      head.M = p.split_at;
      tail = row_part<TA, TB, EPI>(g, p.split_at);
    } else {
      if (EPI == 1) {
        head.pair_off = g.pair_off > 0 ? g.pair_off : g.F;
        head.F = p.split_at;
        head.N = 2 * p.split_at;
      } else {
        head.N = p.split_at;
      }
      tail = column_part<TA, TB, EPI>(g, p.split_at);
    }
    const hipError_t e = launch_tile<TA, TB, EPI>(p.head, head, s);
    if (e != hipSuccess) return e;
  }
  if constexpr (EPI == 0) {
    if (p.splits > 1) {
      // the tail's K split over p.splits workgroups per tile (FP32 partials in
      // the workspace), then the fixed-order sum with alpha, beta * R and bias
      GemmArgs part = tail;
      part.C = reinterpret_cast<lt_half*>(g.ws);
      part.ldc = tail.N;
      part.beta = 0.f;
      part.bias = nullptr;
      const hipError_t e = launch<256, 256, 2, 2, 64, 2, TA, TB, 3>(part, s, p.splits);
      if (e != hipSuccess) return e;
      const int64_t threads = tail.M * (tail.N / 8);
      hipLaunchKernelGGL(splitk_reduce_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0,
                         s, g.ws, p.splits, tail.M, tail.N, g.alpha, g.beta, tail.R, tail.ldr, tail.bias,
                         tail.C, tail.ldc);
      return hipGetLastError();
    }
  }
  return launch_tile<TA, TB, EPI>(p.tail, tail, s);
}

}  // namespace

hipError_t gemm_f16_launch(const GemmArgs& g, hipStream_t s) {
  if (g.epi == 1) return dispatch_tile<false, true, 1>(g, s);     // X Wgu^T
  if (g.epi == 2) return dispatch_tile<false, false, 2>(g, s);    // dY Wd
  if (g.transA) {
    return g.transB ? dispatch_tile<true, true, 0>(g, s) : dispatch_tile<true, false, 0>(g, s);
  }
  return g.transB ? dispatch_tile<false, true, 0>(g, s) : dispatch_tile<false, false, 0>(g, s);
}

}  // namespace lt
