// Reproducible fp32 GEMM with the contraction's blocks spread over the waves of
// a workgroup: products whose outputs are too few to fill the chip.
//
// The canonical contraction cuts k into 64-deep blocks.  A block's partial is a
// chain of fused multiply-adds that starts from +0, so the partials do not
// depend on each other; only their sum is ordered (left to right).  A kernel
// that walks k in one wave therefore runs K dependent matrix steps per output
// where 64 would do, and with few outputs most SIMDs hold no wave at all.
// Here wave w of a workgroup computes the partials of blocks w, w + KS, ... of
// the same output tile, leaves each in LDS, and after every round of KS blocks
// the workgroup's threads add the round's partials to the accumulators in block
// order.  Every output sees the operations of the one-wave walk in its order:
// the bits are the same.
//
// Operands go from global memory into registers, DEPTH slices (of 16 k steps)
// ahead of the steps that use them, with no barrier inside a block.  An operand
// stored along rows is one coalesced 4-byte load per lane and k step: a lane
// needs one row of A and one column of B.  One stored along k is loaded 64 bytes
// of a row by four lanes and turned through the wave's own piece of LDS (direct
// 16-byte loads, one row per lane, touch 64 cache lines each and took twice as
// long: 64 x 4096 outputs, k 14336, B transposed, 198 against 97 us).  The loads
// need 4-byte alignment only, whatever the leading dimensions; the block that K
// cuts short reads in bounds and takes +0 past the end.
//
// What bounds it: few outputs, the latency of one block (64 matrix steps), its
// loads and the launch; few rows, the reading of B from HBM; many outputs, the
// matrix units (counted busy 0.70 of the time at 4096 x 768 outputs and k 3072,
// 0.41 at 1000 x 999 x 1001: a round's partials pass through LDS behind a barrier,
// and a 32 x 64 tile reads three times the operand bytes per step of the 128 x 128
// tile, which is why the large tile stays the better one from about one tile per
// compute unit on).  Measured, graph-replayed, against the one-wave walk (64 x 64
// tiles): 256^3 18.2 -> 3.7 us, 512^3 31.6 -> 6.3, 1000 x 999 x 1001 75 -> 25,
// 4 x 14336 outputs with k 4096 283 -> 38.5 (6.1 TB/s of B), 128 x 3072 with k 768
// 44 -> 11.4, 128 x 768 with k 3072 161 -> 13.5.
//
// The matrix instruction is one of the single-term kinds
//   R = 32: v_mfma_f32_32x32x1_2b    two   32 x 32 blocks, 16 passes
//   R = 16: v_mfma_f32_16x16x1_4b    four  16 x 16 blocks,  8 passes
//   R =  4: v_mfma_f32_4x4x1_16b  sixteen   4 x  4 blocks,  2 passes
// whose blocks are independent products: MB x NB of them side by side make the
// output tile (R MB rows x R NB columns), and KB of them take KB consecutive k
// blocks of the same tile.  All three do 64 flops per clock, so the tile is
// chosen for the rows the product has and for how many workgroups it makes.
#include <hip/hip_runtime.h>

#include <cmath>
#include <type_traits>

#include "gemm_store.h"
#include "gemm_tiles.h"
#include "repops_internal.h"

#pragma clang fp contract(off)

namespace repops {
namespace {

constexpr int kBlock = 64;  // k block of the canonical order this kernel takes
constexpr int kSlice = 16;  // k steps whose operands are loaded together
constexpr int kSlices = kBlock / kSlice;

typedef float v4 __attribute__((ext_vector_type(4)));
// Four consecutive floats at any 4-byte aligned address.
typedef float v4_any __attribute__((ext_vector_type(4), aligned(4)));

typedef const __attribute__((address_space(1))) char* global_bytes;

template <int R>
struct Mfma;
template <>
struct Mfma<32> {
  static constexpr int V = 32;  // accumulator registers
  typedef float acc_t __attribute__((ext_vector_type(32)));
  template <int CBSZ, int ABID>
  __device__ static __forceinline__ acc_t step(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_32x32x1f32(a, b, c, CBSZ, ABID, 0);
  }
  // block, row and column inside the block of register r in lane l
  __device__ static __forceinline__ int block(int r, int) { return r / 16; }
  __device__ static __forceinline__ int row(int r, int l) {
    return 8 * ((r % 16) / 4) + 4 * (l / 32) + r % 4;
  }
  __device__ static __forceinline__ int col(int l) { return l % 32; }
};
template <>
struct Mfma<16> {
  static constexpr int V = 16;
  typedef float acc_t __attribute__((ext_vector_type(16)));
  template <int CBSZ, int ABID>
  __device__ static __forceinline__ acc_t step(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x1f32(a, b, c, CBSZ, ABID, 0);
  }
  __device__ static __forceinline__ int block(int r, int) { return r / 4; }
  __device__ static __forceinline__ int row(int r, int l) { return 4 * (l / 16) + r % 4; }
  __device__ static __forceinline__ int col(int l) { return l % 16; }
};
template <>
struct Mfma<4> {
  static constexpr int V = 4;
  typedef float acc_t __attribute__((ext_vector_type(4)));
  template <int CBSZ, int ABID>
  __device__ static __forceinline__ acc_t step(float a, float b, acc_t c) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, CBSZ, ABID, 0);
  }
  __device__ static __forceinline__ int block(int, int l) { return l / 4; }
  __device__ static __forceinline__ int row(int r, int) { return r; }
  __device__ static __forceinline__ int col(int l) { return l % 4; }
};

template <int R, int MB, int NB, int KB, int MI, int KS, int DEPTH, bool TA, bool TB>
struct SplitTile {
  using M = Mfma<R>;
  using acc_t = typename M::acc_t;
  static constexpr int V = M::V;
  static constexpr int NBLK = 64 / R;  // blocks of one instruction
  static_assert(MB * NB * KB == NBLK, "the instruction's blocks make the tile");
  static_assert(kSlices % DEPTH == 0, "a block is whole turns of the slice registers");
  // MI > 1: the lanes hold the rows of MI row blocks of A, and MI instructions
  // per k step each broadcast one of them to all blocks.
  static_assert(MI == 1 || (MI == NBLK && NB == NBLK), "a broadcast takes one block of A");
  static constexpr int TM = R * MB * MI, TN = R * NB;
  // Partials of KB blocks per wave and round: [slot][register][lane].
  static constexpr int SLOTS = KS * KB;
  static constexpr bool DOUBLE = 2 * KS * MI * V * 64 * 4 <= 64 * 1024;
  // Distinct (row, k place) pairs over the lanes: with MI = 1 the lanes of
  // different column blocks hold the same rows of A, and likewise for B.
  static constexpr int DA = MI > 1 ? 64 : R * MB * KB, DB = R * NB * KB;
  static constexpr bool SA = !TA && DA >= 16, SB = TB && DB >= 16;  // turned through LDS
  static constexpr int STAGE = ((SA ? DA : 0) + (SB ? DB : 0)) * kSlice;  // floats per wave
  static constexpr bool OWN_STAGE = STAGE > MI * V * 64;  // too large for a partial's slot
  struct Smem {
    float p[DOUBLE ? 2 : 1][KS][MI * V][64];
    float stage[OWN_STAGE ? KS : 1][OWN_STAGE ? STAGE : 1];
  };
  // Accumulators per thread.  Registers of the owners (block index along k 0)
  // are dealt to the waves; with R = 4 a register holds all blocks, one per
  // four lanes, and the lanes of k index 0 own.
  static constexpr int OWN = R == 4 ? MI * V : MI * V / KB;
  static constexpr int ACC = OWN >= KS ? OWN / KS : 1;

  // An instruction's block index -> (row block, k block, column block); column
  // blocks run fastest so that lanes of one k step read consecutive columns.
  __device__ static __forceinline__ int blk_m(int b) { return b / (NB * KB); }
  __device__ static __forceinline__ int blk_k(int b) { return (b / NB) % KB; }
  __device__ static __forceinline__ int blk_n(int b) { return b % NB; }

  // One operand's slices.  D distinct rows (columns); ALONG_K: stored along k.
  // Stored along rows, a lane loads its own 16 values, coalesced over the lanes.
  // Stored along k, neighbouring lanes' values lie ld apart, so a slice's D x 16
  // values are loaded 64 bytes of a row by four lanes and turned through LDS:
  // chunk c (of four values) of row d sits at chunk position c ^ (d / 4 % 4) of
  // its 64 bytes, which keeps both the writes and the reads free of bank
  // conflicts.
  template <bool ALONG_K, int D, bool STAGED>
  struct Side {
    static constexpr int NREG = STAGED ? D / 4 : kSlice;  // registers of a slice in flight
    struct Regs {
      float v[NREG];
    };
    int64_t ld;
    uint32_t off[STAGED ? D / 16 : 1];  // bytes from the slice's base to the lane's loads
    int own;                            // the lane's distinct row
    uint32_t wr, rd, swz;               // LDS places (floats) and the read's swizzle

    // place(d) gives the byte offset of row d's first value of a slice.
    template <class F>
    __device__ __forceinline__ void init(int64_t ld_, int lane, int mine, F place) {
      ld = ld_;
      own = mine;
      if constexpr (STAGED) {
#pragma unroll
        for (int i = 0; i < D / 16; ++i)
          off[i] = place(16 * i + lane / 4) + 16 * (lane % 4);
        wr = (lane / 4) * kSlice + 4 * ((lane % 4) ^ (lane / 16 % 4));
        rd = mine * kSlice;
        swz = mine / 4 % 4;
      } else {
        off[0] = place(mine);
      }
    }
    // Values of the slice at `base` (the tile's first row at its k index; uniform).
    __device__ __forceinline__ void load(const float* base, Regs& x) const {
      // The empty asm statements keep the addresses in the loads' form of a
      // scalar base and a 32-bit lane offset: the compiler would otherwise widen
      // the offsets outside the loop, and keep 16 multiples of ld there.
      global_bytes p = (global_bytes)(base);
      if constexpr (ALONG_K) {
#pragma unroll
        for (int i = 0; i < NREG / 4; ++i) {
          uint32_t o = off[STAGED ? i : 0];
          asm("" : "+v"(o));
          const v4_any y = *reinterpret_cast<const __attribute__((address_space(1))) v4_any*>(
              p + o + (STAGED ? 0 : 16 * i));
#pragma unroll
          for (int c = 0; c < 4; ++c) x.v[4 * i + c] = y[c];
        }
      } else {
        uint32_t o = off[0];
        asm("" : "+v"(o));
#pragma unroll
        for (int s = 0; s < kSlice; ++s) {
          x.v[s] = *reinterpret_cast<const __attribute__((address_space(1))) float*>(p + o);
          p += 4 * ld;
          asm("" : "+s"(p));
        }
      }
    }
    // The same with the values at k indices K and past it +0 (they add +0 to a
    // partial, which the accumulator cannot see).  The slice's k indices are
    // k + 64 kplace(d) + 0 .. 15 in row d; base as above at k.  Every address is
    // that of a k index below K in the same row (column).
    template <class F>
    __device__ __forceinline__ void load_cut(const float* base, int k, int K, int lane, F kplace,
                                             Regs& x) const {
      if constexpr (ALONG_K) {
#pragma unroll
        for (int i = 0; i < NREG / 4; ++i) {
          // four values from first <= K - 4 (or one by one where K < 4)
          const int d = STAGED ? 16 * i + lane / 4 : own;
          const int at = k + kplace(d) * kBlock + (STAGED ? 4 * (lane % 4) : 4 * i);
          const float* p = reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) +
                                                          off[STAGED ? i : 0]) +
                           (STAGED ? 0 : 4 * i);
          if (K >= 4) {
            const int past = at - (K - 4);
            const int sh = past > 0 ? past : 0;
            const v4_any y = *reinterpret_cast<const v4_any*>(p - sh);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              float v = c == 0 ? y[0] : (c == 1 ? y[1] : (c == 2 ? y[2] : y[3]));
#pragma unroll
              for (int d = 1; d < 4; ++d)
                if (c + d < 4) v = sh == d ? y[c + d] : v;
              x.v[4 * i + c] = c + sh < 4 ? v : 0.0f;
            }
          } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const int back = at + c - (K - 1);
              const float v = p[c - (back > 0 ? back : 0)];
              x.v[4 * i + c] = back > 0 ? 0.0f : v;
            }
          }
        }
      } else {
        const float* p = reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + off[0]);
        const int at = k + kplace(own) * kBlock;
#pragma unroll
        for (int s = 0; s < kSlice; ++s) {
          const int back = at + s - (K - 1);
          const float v = p[(s - (back > 0 ? back : 0)) * ld];
          x.v[s] = back > 0 ? 0.0f : v;
        }
      }
    }
    // The lane's 16 values of a slice out of the registers it was loaded into.
    __device__ __forceinline__ void turn(float* stage, const Regs& x, float (&v)[kSlice]) const {
      if constexpr (STAGED) {
#pragma unroll
        for (int i = 0; i < D / 16; ++i) {
          const v4 y = {x.v[4 * i], x.v[4 * i + 1], x.v[4 * i + 2], x.v[4 * i + 3]};
          *reinterpret_cast<v4*>(stage + 16 * i * kSlice + wr) = y;
        }
        // one wave: its LDS operations complete in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int q = 0; q < kSlice / 4; ++q) {
          const v4 y = *reinterpret_cast<const v4*>(stage + rd + 4 * (q ^ swz));
#pragma unroll
          for (int c = 0; c < 4; ++c) v[4 * q + c] = y[c];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      } else {
#pragma unroll
        for (int s = 0; s < kSlice; ++s) v[s] = x.v[s];
      }
    }
  };
  using SideA = Side<!TA, DA, SA>;
  using SideB = Side<TB, DB, SB>;

  template <int I>
  __device__ static __forceinline__ void step(float a, float b, bool open, acc_t (&P)[MI]) {
    const acc_t zero = {};
    constexpr int CBSZ = MI == 1 ? 0 : (MI == 2 ? 1 : (MI == 4 ? 2 : 4));
    P[I] = M::template step<CBSZ, MI == 1 ? 0 : I>(a, b, open ? zero : P[I]);
    if constexpr (I + 1 < MI) step<I + 1>(a, b, open, P);
  }
  // Matrix steps [LO, HI) of a slice; open: the slice starts a block.
  template <int LO, int HI>
  __device__ static __forceinline__ void steps(const float (&a)[kSlice], const float (&b)[kSlice],
                                               bool open, acc_t (&P)[MI]) {
#pragma unroll
    for (int s = LO; s < HI; ++s) step<0>(a[s], b[s], open && s == 0, P);
  }

  __device__ static void run(const GemmArgs& g, Smem& sm, int64_t b0, int64_t b1, int64_t m0,
                             int64_t n0) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float* A = g.A + b0 * g.sa0 + b1 * g.sa1;
    const float* B = g.B + b0 * g.sb0 + b1 * g.sb1;
    const int K = static_cast<int>(k_extent(g, m0, TM));  // below 2^31 (the host checks)
    const int nblocks = (K - 1) / kBlock + 1;             // K > 0
    const int rounds = (nblocks + SLOTS - 1) / SLOTS;

    // The lane's row of A, column of B and place along k inside its group of KB
    // blocks; rows and columns past the edge re-read the last one (they only
    // feed outputs that are never stored).
    const int blk = lane / R, idx = lane % R;
    const int ki = blk_k(blk);
    const int64_t arows = g.m - m0, bcols = g.n - n0;
    auto row_in = [&](int64_t r) { return r < arows ? r : arows - 1; };
    auto col_in = [&](int64_t c) { return c < bcols ? c : bcols - 1; };
    const float* A0 = A + (TA ? m0 : m0 * g.lda);
    const float* B0 = B + (TB ? n0 * g.ldb : n0);
    const int64_t astep = TA ? g.lda : 1, bstep = TB ? 1 : g.ldb;
    // Distinct row d: R consecutive lanes' rows, k places and row (column) blocks.
    auto a_kplace = [](int d) { return MI > 1 ? 0 : d / R % KB; };
    auto b_kplace = [](int d) { return d / (R * NB); };
    SideA sa;
    sa.init(g.lda, lane, MI > 1 ? lane : (blk_m(blk) * KB + ki) * R + idx, [&](int d) {
      const int64_t r = row_in(MI > 1 ? d : d / (R * KB) * R + d % R);
      return static_cast<uint32_t>(4 * (r * (TA ? 1 : g.lda) + a_kplace(d) * kBlock * astep));
    });
    SideB sb;
    sb.init(g.ldb, lane, (ki * NB + blk_n(blk)) * R + idx, [&](int d) {
      const int64_t c = col_in(d / R % NB * R + d % R);
      return static_cast<uint32_t>(4 * (c * (TB ? g.ldb : 1) + b_kplace(d) * kBlock * bstep));
    });

    float acc[ACC];
#pragma unroll
    for (int i = 0; i < ACC; ++i) acc[i] = 0.0f;

    // Group r of this wave: KB blocks from block (r KS + wave) KB.  In every
    // round but the last all groups are whole; there a wave's group may be
    // whole, hold the end of the contraction, or not exist.
    auto first_k = [&](int r) { return (r * KS + wave) * (KB * kBlock); };
    auto whole = [&](int r) { return first_k(r) <= K - KB * kBlock; };
    typename SideA::Regs ra[DEPTH];
    typename SideB::Regs rb[DEPTH];
    // slices stay in order: so do the waits for them
    auto load_a = [&](int t, int k) {
      sa.load(A0 + k * astep, ra[t % DEPTH]);
      __builtin_amdgcn_sched_barrier(0);
    };
    auto load_b = [&](int t, int k) {
      sb.load(B0 + k * bstep, rb[t % DEPTH]);
      __builtin_amdgcn_sched_barrier(0);
    };
    // Slices of the group that holds the end of the contraction.
    auto cut_a = [&](int t, int k) {
      if (k >= K) return;  // uniform; nothing reads the slice
      if (k + (KB - 1) * kBlock + kSlice <= K) load_a(t, k);
      else sa.load_cut(A0 + k * astep, k, K, lane, a_kplace, ra[t % DEPTH]);
    };
    auto cut_b = [&](int t, int k) {
      if (k >= K) return;
      if (k + (KB - 1) * kBlock + kSlice <= K) load_b(t, k);
      else sb.load_cut(B0 + k * bstep, k, K, lane, b_kplace, rb[t % DEPTH]);
    };
    // The round's partials join the accumulators in block order.
    auto publish = [&](int r, const acc_t (&P)[MI]) {
      float(*mine)[64] = sm.p[DOUBLE ? r & 1 : 0][wave];
#pragma unroll
      for (int v = 0; v < MI * V; ++v) mine[v][lane] = P[v / V][v % V];
    };
    auto combine = [&](int r, int count) {
      __syncthreads();
      if (OWN >= KS || wave < OWN) {
        auto add = [&](int s) {
          const int w = s / KB, k = s % KB;
          const float(*p)[64] = sm.p[DOUBLE ? r & 1 : 0][w];
#pragma unroll
          for (int i = 0; i < ACC; ++i) {
            const int v = wave * ACC + i;
            if constexpr (R == 4) acc[i] = acc[i] + p[v][(lane + k * NB * R) & 63];
            else acc[i] = acc[i] + p[own_reg(v) + k * NB * (V / NBLK)][lane];
          }
        };
        if (count == SLOTS) {
#pragma unroll
          for (int s = 0; s < SLOTS; ++s) add(s);
        } else {
#pragma unroll 1
          for (int s = 0; s < count; ++s) add(s);
        }
      }
      if constexpr (!DOUBLE) __syncthreads();
    };

    // A group of blocks from k0, its first DEPTH slices already in flight.  Each
    // register set is refilled with the slice DEPTH on as soon as it has been
    // read; a side turned through LDS is turned in the middle of the slice before.
    // MORE: past the group's end the slices of the next one, at kn, follow.
    // END: the group holds the end of the contraction; slices past it are left
    // out, and the others' values there are +0.
    constexpr int MORE = 0, LAST = 1, END = 2;
    auto block = [&](auto mode, int r, int k0, int kn) {
      constexpr int MODE = decltype(mode)::value;
      float* stage = OWN_STAGE ? sm.stage[wave] : sm.p[DOUBLE ? r & 1 : 0][wave][0];
      auto next_a = [&](int t) {
        if (t < kSlices) {
          if (MODE == END) cut_a(t, k0 + t * kSlice); else load_a(t, k0 + t * kSlice);
        } else if (MODE == MORE) {
          load_a(t, kn + (t - kSlices) * kSlice);
        }
      };
      auto next_b = [&](int t) {
        if (t < kSlices) {
          if (MODE == END) cut_b(t, k0 + t * kSlice); else load_b(t, k0 + t * kSlice);
        } else if (MODE == MORE) {
          load_b(t, kn + (t - kSlices) * kSlice);
        }
      };
      auto there = [&](int t) { return MODE != END || k0 + t * kSlice < K; };  // uniform
      acc_t P[MI];
      float a[2][kSlice], b[2][kSlice];
      auto turn = [&](int t) {
        if constexpr (SA) {
          sa.turn(stage, ra[t % DEPTH], a[t & 1]);
          next_a(t + DEPTH);
        }
        if constexpr (SB) {
          sb.turn(stage + (SA ? DA * kSlice : 0), rb[t % DEPTH], b[t & 1]);
          next_b(t + DEPTH);
        }
      };
      turn(0);
#pragma unroll
      for (int t = 0; t < kSlices; ++t) {
        if (!there(t)) continue;
        if constexpr (!SA) sa.turn(stage, ra[t % DEPTH], a[t & 1]);
        if constexpr (!SB) sb.turn(stage, rb[t % DEPTH], b[t & 1]);
        steps<0, kSlice / 2>(a[t & 1], b[t & 1], t == 0, P);
        if constexpr (SA || SB) {
          __builtin_amdgcn_sched_barrier(0);
          if (t + 1 < kSlices && there(t + 1)) turn(t + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
        steps<kSlice / 2, kSlice>(a[t & 1], b[t & 1], false, P);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (!SA) next_a(t + DEPTH);
        if constexpr (!SB) next_b(t + DEPTH);
      }
      publish(r, P);
    };

    if (whole(0)) {
#pragma unroll
      for (int t = 0; t < DEPTH; ++t) {
        load_a(t, first_k(0) + t * kSlice);
        load_b(t, first_k(0) + t * kSlice);
      }
    }
    for (int r = 0; r + 1 < rounds; ++r) {
      // without a whole group in the last round the loads repeat this one's (in
      // bounds; never used)
      block(std::integral_constant<int, MORE>{}, r, first_k(r),
            whole(r + 1) ? first_k(r + 1) : first_k(r));
      combine(r, SLOTS);
    }
    {
      const int r = rounds - 1;
      const int k0 = first_k(r);
      if (whole(r)) {
        block(std::integral_constant<int, LAST>{}, r, k0, 0);
      } else if (k0 < K) {
#pragma unroll
        for (int t = 0; t < DEPTH; ++t) {
          cut_a(t, k0 + t * kSlice);
          cut_b(t, k0 + t * kSlice);
        }
        block(std::integral_constant<int, END>{}, r, k0, 0);
      }
      combine(r, nblocks - r * SLOTS);
    }

    if (OWN < KS && wave >= OWN) return;
    float* C = g.C + b0 * g.sc0 + b1 * g.sc1;
    float* G = g.G ? g.G + b0 * g.sc0 + b1 * g.sc1 : nullptr;
    const float* X = g.gelu_in ? g.gelu_in + b0 * g.sc0 + b1 * g.sc1 : nullptr;
#pragma unroll
    for (int i = 0; i < ACC; ++i) {
      const int v = wave * ACC + i;
      const int reg = R == 4 ? v : own_reg(v);
      const int b = M::block(reg % V, lane);
      const int64_t row = m0 + ((reg / V) * MB + blk_m(b)) * R + M::row(reg % V, lane);
      const int64_t col = n0 + blk_n(b) * R + M::col(lane);
      if (blk_k(b) == 0 && row < g.m && col < g.n) gemm_store(g, C, G, X, row, col, acc[i]);
    }
  }

  // Register of the o-th owner: the registers of the blocks with k index 0.
  __device__ static __forceinline__ int own_reg(int o) {
    constexpr int PER = V / NBLK == 0 ? 1 : V / NBLK;  // registers of one block
    const int b = o / PER;                               // block among those of k index 0
    return ((b / NB) * NB * KB + b % NB) * PER + o % PER;
  }
};

template <int R, int MB, int NB, int KB, int MI, int KS, int DEPTH, int MINW, bool TA, bool TB>
__global__ __launch_bounds__(64 * KS, MINW) void gemm_split_kernel(GemmArgs g, uint32_t tiles_m,
                                                                   uint32_t tiles_n,
                                                                   uint32_t ntiles) {
  using T = SplitTile<R, MB, NB, KB, MI, KS, DEPTH, TA, TB>;
  __shared__ typename T::Smem sm;
  // tile_coords' mapping in 32-bit arithmetic (gemm_split_ok bounds the tiles):
  // panels of four tile rows, a contiguous share of them per XCD.  Lower-triangle
  // products launch every tile; those above the diagonal return.
  uint32_t t = blockIdx.x;
  if (ntiles % 8 == 0) t = (t % 8) * (ntiles / 8) + t / 8;
  const uint32_t per = tiles_m * tiles_n;
  const uint32_t bz = t / per, r = t % per;
  const uint32_t panel = r / (4 * tiles_n), in = r % (4 * tiles_n);
  const uint32_t rows = tiles_m - 4 * panel < 4 ? tiles_m - 4 * panel : 4;
  uint32_t tm = 4 * panel + in % rows;
  const uint32_t tn = in / rows;
  if (g.causal == 2) tm = tiles_m - 1 - tm;  // longest contraction first
  const uint32_t nb1 = static_cast<uint32_t>(g.batch1);
  const int64_t m0 = static_cast<int64_t>(tm) * T::TM, n0 = static_cast<int64_t>(tn) * T::TN;
  if (tile_above_diagonal(g, m0, T::TM, n0)) return;  // uniform over the workgroup
  T::run(g, sm, bz / nb1, bz % nb1, m0, n0);
}

struct SplitEntry {
  GemmConfig cfg;
  int ks, slots;
  // Time estimate in us: start + the larger of one tile alone (`round` per round
  // of blocks, `tile` for its first loads and its stores) and of the tiles a
  // compute unit gets (`work` per full round, a partly filled one saving `fill`
  // of what it leaves empty, and `tile`, each); and never less than the operands
  // and outputs at `gbs`, what the tile's access pattern reaches from HBM.  The
  // estimates are for ranking: over the 520 shapes of perf/gemm_choice.py those of
  // the entries near the fastest are 6 (ring) to 52% (smallest tiles) off, most of
  // them high together, and the chosen entry is 4% behind the fastest (geometric
  // mean; more than 10% behind on 71 shapes).
  float start, round, work, tile, fill, gbs;
  void (*kernel[4])(GemmArgs, uint32_t, uint32_t, uint32_t);  // [ta * 2 + tb]
};

#define REPOPS_SPLIT(NAME, R, MB, NB, KB, MI, KS, DEPTH, START, ROUND, WORK, TILE, FILL, GBS) \
  {{NAME, R * MB * MI, R * NB, kBlock}, KS, KS * KB, START, ROUND, WORK, TILE, FILL, GBS, \
   {gemm_split_kernel<R, MB, NB, KB, MI, KS, DEPTH, 2, false, false>,                    \
    gemm_split_kernel<R, MB, NB, KB, MI, KS, DEPTH, 2, false, true>,                     \
    gemm_split_kernel<R, MB, NB, KB, MI, KS, DEPTH, 2, true, false>,                     \
    gemm_split_kernel<R, MB, NB, KB, MI, KS, DEPTH, 2, true, true>}}

// Names: output tile x k block / waves, each with its own k blocks x k blocks per
// instruction.
const SplitEntry kSplit[] = {
    REPOPS_SPLIT("32x64x64/k4", 32, 1, 2, 1, 1, 4, 2, 2.6f, 2.0f, 2.55f, 1.7f, 0.7f, 4700),
    REPOPS_SPLIT("32x64x64/k8", 32, 1, 2, 1, 1, 8, 2, 2.6f, 0.3f, 5.1f, 2.2f, 0.7f, 5300),
    REPOPS_SPLIT("64x64x64/k4", 32, 1, 2, 1, 2, 4, 2, 5.2f, 1.8f, 4.6f, 2.0f, 0.6f, 4500),
    REPOPS_SPLIT("64x64x64/k8", 32, 1, 2, 1, 2, 8, 2, 2.6f, 2.6f, 9.2f, 3.0f, 0.7f, 4500),
    REPOPS_SPLIT("16x64x64/k8", 16, 1, 4, 1, 1, 8, 4, 2.3f, 0.2f, 3.05f, 2.0f, 0.7f, 6600),
    REPOPS_SPLIT("16x32x64/k8x2", 16, 1, 2, 2, 1, 8, 4, 2.2f, 2.5f, 3.4f, 2.2f, 0.7f, 5600),
    REPOPS_SPLIT("16x16x64/k8x4", 16, 1, 1, 4, 1, 8, 4, 2.0f, 1.2f, 5.1f, 2.3f, 0.7f, 5000),
    REPOPS_SPLIT("4x16x64/k8x4", 4, 1, 4, 4, 1, 8, 4, 2.6f, 1.4f, 3.3f, 1.0f, 0.7f, 6000),
    REPOPS_SPLIT("16x16x64/k4", 4, 4, 4, 1, 1, 4, 4, 3.0f, 1.1f, 0.75f, 0.5f, 0.7f, 5200),
};
constexpr int kSplitCount = sizeof(kSplit) / sizeof(kSplit[0]);

}  // namespace

int gemm_split_count() { return kSplitCount; }
const GemmConfig* gemm_split_config(int index) {
  return (index >= 0 && index < kSplitCount) ? &kSplit[index].cfg : nullptr;
}

bool gemm_split_ok(const GemmArgs& g, int index) {
  const SplitEntry& e = kSplit[index];
  const int64_t tiles_m = (g.m + e.cfg.bm - 1) / e.cfg.bm, tiles_n = (g.n + e.cfg.bn - 1) / e.cfg.bn;
  constexpr int64_t kLd = int64_t(1) << 22;  // lane offsets stay within 32 bits
  // one workgroup per tile; the tile arithmetic is 32-bit (4 tile rows at a time)
  const int64_t cap = max_workgroups(64 * e.ks);
  return g.fused && g.k_block == kBlock && g.k > 0 && g.k <= INT32_MAX / 2 && g.lda <= kLd && g.ldb <= kLd &&
         g.batch0 * g.batch1 <= cap &&
         static_cast<unsigned __int128>(tiles_m) * tiles_n * (g.batch0 * g.batch1) <= static_cast<uint64_t>(cap);
}

double gemm_split_us(const GemmArgs& g, int index, int cus) {
  const SplitEntry& e = kSplit[index];
  const int64_t tiles_m = (g.m + e.cfg.bm - 1) / e.cfg.bm, tiles_n = (g.n + e.cfg.bn - 1) / e.cfg.bn;
  const double batch = static_cast<double>(g.batch0) * static_cast<double>(g.batch1);
  double tiles = static_cast<double>(tiles_m) * static_cast<double>(tiles_n) * batch;
  const double blocks = static_cast<double>((g.k + kBlock - 1) / kBlock);
  // the part of the contraction (causal A) or of the tiles (causal output) left
  double part = 1.0;
  if (g.causal == 1 && tiles_n > 1) tiles *= 0.5 + 0.5 / static_cast<double>(tiles_n);
  if (g.causal == 2) part = 0.5 + 0.5 / std::ceil(blocks / e.slots);
  const double rounds = std::ceil(blocks / e.slots), per_cu = std::ceil(tiles / cus);
  // A partly filled round costs more than its share, and so does a short block.
  double full = e.fill * blocks / e.slots + (1.0 - e.fill) * rounds;
  if (blocks / e.slots < 0.3) full = 0.3;
  const double tile = e.tile + (g.k % kBlock != 0 ? 1.0 : 0.0);
  const double one = rounds * part * e.round + tile;
  const double all = per_cu * (full * part * e.work + tile);
  double us = e.start + (one > all ? one : all);
  if (g.causal == 2) us *= 1.1;  // row tiles of unequal length share the units unevenly
  if (g.tb && e.cfg.bn == 64) us *= 1.1;  // the wide operand turned through LDS
  const double m = static_cast<double>(g.m), n = static_cast<double>(g.n),
               k = static_cast<double>(g.k);
  const double moved = e.start + 4.0 * batch * (m * k + k * n + m * n) / (e.gbs * 1e3);
  return us > moved ? us : moved;
}

hipError_t launch_gemm_split(const GemmArgs& g, int index, hipStream_t s) {
  const SplitEntry& e = kSplit[index];
  const int64_t tiles_m = (g.m + e.cfg.bm - 1) / e.cfg.bm, tiles_n = (g.n + e.cfg.bn - 1) / e.cfg.bn;
  const int64_t ntiles = tiles_m * tiles_n * g.batch0 * g.batch1;
  hipLaunchKernelGGL(e.kernel[g.ta * 2 + g.tb], dim3(static_cast<unsigned>(ntiles)),
                     dim3(64 * e.ks), 0, s, g, static_cast<uint32_t>(tiles_m),
                     static_cast<uint32_t>(tiles_n), static_cast<uint32_t>(ntiles));
  return hipGetLastError();
}

}  // namespace repops
