// Tensor commitments for gfx950: SHA-256 (FIPS 180-4) and the RFC 6962 Merkle
// Tree Hash over fixed-size chunks of a tensor's bytes.
//
// The Verde protocol commits to checkpoints and to the tensors entering and
// leaving every graph node with a collision-resistant hash such as SHA-256,
// and combines node hashes in a binary Merkle tree (Sections 2.1 and 2.2).  A
// single SHA-256 stream is sequential, so a tensor is committed as a Merkle
// tree of its chunks: leaf = SHA-256(0x00 || chunk), node = SHA-256(0x01 ||
// left || right), the tree split at the largest power of two (RFC 6962).
//
// Schedule: one lane per leaf chunk (the chunk's blocks in sequence); then
// the tree level by level, pairs hashed and an odd last node carried up
// unchanged (which reproduces RFC 6962's split): one launch per level, eight
// levels per launch from LDS between 65536 and 16384 nodes, and the last 256 nodes
// in one workgroup, which writes the root as 32 bytes.  A level costs at least one
// two-block hash of latency, so a tensor's commitment has a floor of about that
// times the tree depth; wide levels and the leaves are integer-ALU bound.
//
// Digests travel between kernels as eight 32-bit words (SHA-256's big-endian
// word view); data bytes are read as little-endian dwords and reassembled into
// message words with byte permutes, the one-byte prefix shifting every word
// by a byte.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "commit_internal.h"

namespace repops {
namespace {

// First 32 bits of the fractional parts of the cube roots of the first 64
// primes, and of the square roots of the first 8 primes (FIPS 180-4, 4.2.2
// and 5.3.3).
constexpr uint32_t kK[64] = {
    0x428a2f98u, 0x71374491u, 0xb5c0fbcfu, 0xe9b5dba5u, 0x3956c25bu, 0x59f111f1u, 0x923f82a4u,
    0xab1c5ed5u, 0xd807aa98u, 0x12835b01u, 0x243185beu, 0x550c7dc3u, 0x72be5d74u, 0x80deb1feu,
    0x9bdc06a7u, 0xc19bf174u, 0xe49b69c1u, 0xefbe4786u, 0x0fc19dc6u, 0x240ca1ccu, 0x2de92c6fu,
    0x4a7484aau, 0x5cb0a9dcu, 0x76f988dau, 0x983e5152u, 0xa831c66du, 0xb00327c8u, 0xbf597fc7u,
    0xc6e00bf3u, 0xd5a79147u, 0x06ca6351u, 0x14292967u, 0x27b70a85u, 0x2e1b2138u, 0x4d2c6dfcu,
    0x53380d13u, 0x650a7354u, 0x766a0abbu, 0x81c2c92eu, 0x92722c85u, 0xa2bfe8a1u, 0xa81a664bu,
    0xc24b8b70u, 0xc76c51a3u, 0xd192e819u, 0xd6990624u, 0xf40e3585u, 0x106aa070u, 0x19a4c116u,
    0x1e376c08u, 0x2748774cu, 0x34b0bcb5u, 0x391c0cb3u, 0x4ed8aa4au, 0x5b9cca4fu, 0x682e6ff3u,
    0x748f82eeu, 0x78a5636fu, 0x84c87814u, 0x8cc70208u, 0x90befffau, 0xa4506cebu, 0xbef9a3f7u,
    0xc67178f2u};
constexpr uint32_t kH0[8] = {0x6a09e667u, 0xbb67ae85u, 0x3c6ef372u, 0xa54ff53au,
                             0x510e527fu, 0x9b05688cu, 0x1f83d9abu, 0x5be0cd19u};

constexpr int kTopNodes = 256;     // nodes one workgroup reduces to one (eight levels)
constexpr int kSplitLeaves = 128;  // leaves of a workgroup with two waves a leaf
// Leaves up to which they are hashed by two waves each: one workgroup of four
// waves per compute unit, so that no SIMD holds two waves (one lane a leaf takes
// 47.2 us just above this line, two waves a leaf 38.9 us at it).
constexpr uint64_t kFewLeaves = 256 * kSplitLeaves;
constexpr int kTopThreads = 256;   // two for each of the 128 pairs
// Levels of more nodes than the first and at most the second are reduced in
// slices, at most one workgroup per compute unit, whose SIMDs then hold one wave
// each.  A wider level fills the SIMDs by itself and takes a launch of its own; so
// does a narrower one, whose launch costs less than a level of slices (whole
// commitments of 64-byte leaves, slices against launches: 2000 leaves 76.9 and
// 69.7 us, 8192 87.8 and 88.1, 16384 93.2 and 89.7, 24000 97.6 and 97.3, 32768
// 97.2 and 98.1, 65536 99.7 and 105.9).
constexpr uint64_t kLevelNodes = 64 * kTopNodes;
constexpr uint64_t kSliceNodes = 256 * kTopNodes;

__device__ __forceinline__ uint32_t rotr(uint32_t x, int n) { return (x >> n) | (x << (32 - n)); }

// SHA-256's three-input bitwise functions, each one gfx950 three-input bitwise
// operation; the 8-bit table holds the output for input bits (a, b, c) at
// bit 4a + 2b + c.  Parity (0x96) for the Sigma / sigma functions, majority
// (0xE8), and choose -- b where a is set, else c -- (0xCA).  (The compiler
// otherwise splits each into two-input operations.)
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}
__device__ __forceinline__ uint32_t maj3(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xE8);
}
__device__ __forceinline__ uint32_t choose(uint32_t a, uint32_t b, uint32_t c) {
  return __builtin_amdgcn_bitop3_b32(a, b, c, 0xCA);
}

// Word t of the message schedule (t >= 16, t % 16 = j) into its place in the
// rolling words.
__device__ __forceinline__ void extend(uint32_t W[16], int j) {
  const uint32_t w15 = W[(j + 1) & 15], w2 = W[(j + 14) & 15];
  const uint32_t s0 = xor3(rotr(w15, 7), rotr(w15, 18), w15 >> 3);
  const uint32_t s1 = xor3(rotr(w2, 17), rotr(w2, 19), w2 >> 10);
  W[j] += s0 + W[(j + 9) & 15] + s1;
}

// One round on the working variables a .. h; kw is the round's constant plus its
// message word.
__device__ __forceinline__ void sha_round(uint32_t s[8], uint32_t kw) {
  const uint32_t S1 = xor3(rotr(s[4], 6), rotr(s[4], 11), rotr(s[4], 25));
  const uint32_t T1 = s[7] + S1 + choose(s[4], s[5], s[6]) + kw;
  const uint32_t S0 = xor3(rotr(s[0], 2), rotr(s[0], 13), rotr(s[0], 22));
  const uint32_t T2 = S0 + maj3(s[0], s[1], s[2]);
  s[7] = s[6];
  s[6] = s[5];
  s[5] = s[4];
  s[4] = s[3] + T1;
  s[3] = s[2];
  s[2] = s[1];
  s[1] = s[0];
  s[0] = T1 + T2;
}

// Sixteen rounds' words on their way through LDS from the thread that makes them
// to the one that runs the rounds: four 16-byte accesses a thread.
template <int THREADS>
struct Sched {
  uint4 w[4][THREADS];
  // Words W, the first of them word 16 t, with their round constants.
  __device__ __forceinline__ void put(int i, int t, const uint32_t W[16]) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t* k = kK + 16 * t + 4 * q;
      w[q][i] = make_uint4(W[4 * q] + k[0], W[4 * q + 1] + k[1], W[4 * q + 2] + k[2],
                           W[4 * q + 3] + k[3]);
    }
  }
  // The rounds.  All reads come first: the compiler otherwise puts each just
  // before its use and the wave waits out LDS's latency eight times.
  __device__ __forceinline__ void rounds(int i, uint32_t s[8]) const {
    uint4 x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = w[q][i];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sha_round(s, x[q].x);
      sha_round(s, x[q].y);
      sha_round(s, x[q].z);
      sha_round(s, x[q].w);
    }
  }
};

// The compression function on one block; W holds the block's 16 words and is
// consumed as the rolling message schedule.  Fully unrolled: every round
// constant is an immediate.
__device__ __forceinline__ void compress(uint32_t H[8], uint32_t W[16]) {
  uint32_t s[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) s[k] = H[k];
#pragma unroll
  for (int t = 0; t < 64; ++t) {
    if (t >= 16) extend(W, t & 15);
    sha_round(s, kK[t] + W[t & 15]);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) H[k] += s[k];
}

// Message word whose bytes are (top byte of prev, bytes 0..2 of cur): the
// stream shifted by the one-byte prefix, with prev/cur little-endian dwords.
// One byte permute; written as shifts and masks it took five instructions, 64 of
// a block's 1484 (leaves of 235 MB 192 -> 183 us).
__device__ __forceinline__ uint32_t shifted_word(uint32_t prev, uint32_t cur) {
  // byte i of the selector picks the result's byte i: 0-3 from cur, 4-7 from prev
  return __builtin_amdgcn_perm(prev, cur, 0x07000102u);
}

// Byte p of (prefix || data[0..len) || 0x80 || zeros || 64-bit bit length),
// padded to `blocks` blocks: the generic path for a short or unaligned chunk.
__device__ __forceinline__ uint32_t stream_byte(const uint8_t* data, uint64_t len, uint8_t prefix,
                                                uint64_t p, uint64_t total_len, uint64_t blocks) {
  if (p == 0) return prefix;
  if (p - 1 < len) return data[p - 1];
  if (p == len + 1) return 0x80u;
  const uint64_t end = blocks * 64;
  if (p >= end - 8) {
    const uint64_t bits = total_len * 8;
    const int shift = static_cast<int>(8 * (end - 1 - p));
    return static_cast<uint32_t>((bits >> shift) & 0xffu);
  }
  return 0u;
}

__device__ void sha_generic(const uint8_t* data, uint64_t len, uint8_t prefix, uint32_t H[8]) {
#pragma unroll
  for (int k = 0; k < 8; ++k) H[k] = kH0[k];
  const uint64_t total = len + 1;
  const uint64_t blocks = (total + 9 + 63) / 64;
  for (uint64_t b = 0; b < blocks; ++b) {
    uint32_t W[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const uint64_t p = b * 64 + 4 * j;
      W[j] = (stream_byte(data, len, prefix, p, total, blocks) << 24) |
             (stream_byte(data, len, prefix, p + 1, total, blocks) << 16) |
             (stream_byte(data, len, prefix, p + 2, total, blocks) << 8) |
             stream_byte(data, len, prefix, p + 3, total, blocks);
    }
    compress(H, W);
  }
}

// ---------------------------------------------------------------------------
// leaves: H = SHA-256(0x00 || chunk)
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void leaf_kernel(const uint8_t* data, uint64_t nbytes,
                                                   uint32_t chunk, uint64_t leaves, uint32_t* out,
                                                   int vec) {
  const uint64_t leaf = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (leaf >= leaves) return;
  const uint64_t off = leaf * chunk;
  const uint64_t len = (off + chunk <= nbytes) ? chunk : nbytes - off;
  uint32_t H[8];
  if (vec && len == chunk) {
    // Full chunk, 16-byte aligned, chunk a multiple of 64: chunk/64 blocks of
    // (prefix || data), then one block with the last data byte and padding.
#pragma unroll
    for (int k = 0; k < 8; ++k) H[k] = kH0[k];
    const uint4* p = reinterpret_cast<const uint4*>(data + off);
    uint32_t prev = 0;  // the prefix byte 0x00 sits in prev's top byte
    const uint32_t nb = chunk / 64;
    uint4 q0 = p[0], q1 = p[1], q2 = p[2], q3 = p[3];
    for (uint32_t b = 0; b < nb; ++b) {
      const uint32_t d[16] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w,
                              q2.x, q2.y, q2.z, q2.w, q3.x, q3.y, q3.z, q3.w};
      if (b + 1 < nb) {  // next block's loads in flight during this block's rounds
        q0 = p[4 * (b + 1)];
        q1 = p[4 * (b + 1) + 1];
        q2 = p[4 * (b + 1) + 2];
        q3 = p[4 * (b + 1) + 3];
      }
      uint32_t W[16];
      W[0] = shifted_word(prev, d[0]);
#pragma unroll
      for (int j = 1; j < 16; ++j) W[j] = shifted_word(d[j - 1], d[j]);
      prev = d[15];
      compress(H, W);
    }
    const uint64_t bits = (static_cast<uint64_t>(chunk) + 1) * 8;
    uint32_t W[16];
    W[0] = (prev & 0xff000000u) | 0x00800000u;
#pragma unroll
    for (int j = 1; j < 14; ++j) W[j] = 0;
    W[14] = static_cast<uint32_t>(bits >> 32);
    W[15] = static_cast<uint32_t>(bits);
    compress(H, W);
  } else {
    sha_generic(data + off, len, 0x00, H);
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) out[leaf * 8 + k] = H[k];
}

// The same for few leaves, two waves a leaf: with no more waves than half the
// SIMDs the rounds' instruction issue bounds the call and SIMDs are idle, so half
// of the threads make the message schedule (a third of the instructions) 16 words
// ahead of the rounds, as in the tree's slices below.  chunk is a multiple of 64
// and data 16-byte aligned.  32768 leaves of 1 KiB 47.2 -> 38.9 us; the whole
// commitment, its tree as below, of 48 leaves 81 -> 70 us, of 2000 113 -> 99, of
// 32768 139 -> 127.
__global__ __launch_bounds__(2 * kSplitLeaves) void leaf_split_kernel(const uint8_t* data,
                                                                      uint64_t nbytes,
                                                                      uint32_t chunk,
                                                                      uint64_t leaves,
                                                                      uint32_t* out) {
  __shared__ Sched<kSplitLeaves> sched[2];
  const int tid = threadIdx.x;
  const bool rounds = tid < kSplitLeaves;  // uniform over a wave
  const int i = rounds ? tid : tid - kSplitLeaves;
  const uint64_t leaf = static_cast<uint64_t>(blockIdx.x) * kSplitLeaves + i;
  const uint64_t off = leaf * chunk;
  const bool full = leaf < leaves && off + chunk <= nbytes;
  // Uniform over the workgroup: only the tensor's last leaf can be short, so the
  // workgroup has a whole leaf exactly if its first one is.  Without one no thread
  // has a block to make or to hash, and a chunk much longer than the tensor would
  // cost four empty barriers per block of the chunk (100 bytes with 1 MiB chunks:
  // 3140 us a call, 17 without the loop).
  const uint64_t first = static_cast<uint64_t>(blockIdx.x) * kSplitLeaves * chunk;
  const bool any_full = first + chunk <= nbytes;
  const uint4* p = reinterpret_cast<const uint4*>(data + off);
  const uint32_t nb = chunk / 64;
  uint32_t H[8], s[8];  // rounds: the chaining value and the working variables
  uint32_t W[16];       // schedule: the rolling message words
  uint4 q0 = {}, q1 = {}, q2 = {}, q3 = {};
  uint32_t prev = 0;  // the prefix byte 0x00 sits in prev's top byte
#pragma unroll
  for (int k = 0; k < 8; ++k) H[k] = s[k] = kH0[k];
  if (!rounds && full) {
    q0 = p[0];
    q1 = p[1];
    q2 = p[2];
    q3 = p[3];
  }
  // Block nb holds the last data byte and the padding.  Step (b, t) makes group t
  // of block b while the rounds take the group before it.
  for (uint32_t b = 0; any_full && b <= nb; ++b) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      if (rounds) {
        if (full && (t > 0 || b > 0)) {
          sched[(t + 1) & 1].rounds(i, s);
          if (t == 0) {
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k] = H[k] = H[k] + s[k];
          }
        }
      } else if (full) {
        if (t > 0) {
#pragma unroll
          for (int j = 0; j < 16; ++j) extend(W, j);
        } else if (b < nb) {
          const uint32_t d[16] = {q0.x, q0.y, q0.z, q0.w, q1.x, q1.y, q1.z, q1.w,
                                  q2.x, q2.y, q2.z, q2.w, q3.x, q3.y, q3.z, q3.w};
          W[0] = shifted_word(prev, d[0]);
#pragma unroll
          for (int j = 1; j < 16; ++j) W[j] = shifted_word(d[j - 1], d[j]);
          prev = d[15];
          if (b + 1 < nb) {
            q0 = p[4 * (b + 1)];
            q1 = p[4 * (b + 1) + 1];
            q2 = p[4 * (b + 1) + 2];
            q3 = p[4 * (b + 1) + 3];
          }
        } else {
          const uint64_t bits = (static_cast<uint64_t>(chunk) + 1) * 8;
          W[0] = (prev & 0xff000000u) | 0x00800000u;
#pragma unroll
          for (int j = 1; j < 14; ++j) W[j] = 0;
          W[14] = static_cast<uint32_t>(bits >> 32);
          W[15] = static_cast<uint32_t>(bits);
        }
        sched[t & 1].put(i, t, W);
      }
      __syncthreads();
    }
  }
  if (!rounds || leaf >= leaves) return;
  if (full) {
    sched[1].rounds(i, s);
#pragma unroll
    for (int k = 0; k < 8; ++k) H[k] += s[k];
  } else {
    sha_generic(data + off, nbytes - off, 0x00, H);  // the short last chunk
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) out[leaf * 8 + k] = H[k];
}

// ---------------------------------------------------------------------------
// nodes: H = SHA-256(0x01 || L || R), 65 bytes = two blocks
// ---------------------------------------------------------------------------

__device__ __forceinline__ void node_hash(const uint32_t L[8], const uint32_t R[8], uint32_t H[8]) {
#pragma unroll
  for (int k = 0; k < 8; ++k) H[k] = kH0[k];
  uint32_t W[16];
  W[0] = 0x01000000u | (L[0] >> 8);
#pragma unroll
  for (int j = 1; j < 8; ++j) W[j] = (L[j - 1] << 24) | (L[j] >> 8);
  W[8] = (L[7] << 24) | (R[0] >> 8);
#pragma unroll
  for (int j = 9; j < 16; ++j) W[j] = (R[j - 9] << 24) | (R[j - 8] >> 8);
  compress(H, W);
  W[0] = (R[7] << 24) | 0x00800000u;
#pragma unroll
  for (int j = 1; j < 15; ++j) W[j] = 0;
  W[15] = 65 * 8;
  compress(H, W);
}

__global__ __launch_bounds__(256) void node_kernel(const uint32_t* in, uint64_t n_in,
                                                   uint32_t* out) {
  const uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  const uint64_t n_out = (n_in + 1) / 2;
  if (i >= n_out) return;
  uint32_t H[8];
  if (2 * i + 1 < n_in) {
    uint32_t L[8], R[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      L[k] = in[(2 * i) * 8 + k];
      R[k] = in[(2 * i + 1) * 8 + k];
    }
    node_hash(L, R, H);
  } else {
#pragma unroll
    for (int k = 0; k < 8; ++k) H[k] = in[(2 * i) * 8 + k];  // odd last node carried up
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) out[i * 8 + k] = H[k];
}

// Aligned slices of kTopNodes nodes, one per workgroup, reduced to one node each,
// level by level in LDS (inside a slice the pairs (2i, 2i + 1) are those of the
// whole level, and only the last slice can hold the odd last node).
//
// Bound: instruction issue of the one wave that holds a lane's hash; a narrow
// level leaves the other SIMDs idle.  A third of a compression's instructions
// are the message schedule, which does not depend on the rounds, so the lower
// half of the threads runs the rounds and the upper half makes the schedule, 16
// words (round constants added) ahead of them, through LDS.  A workgroup's four
// waves sit on four SIMDs, and 128 nodes per level take two waves of each kind.
// All 16 levels of 64 MB's 65536 leaves take two launches of 48 us at most, where
// seven levels of a launch each and nine in one workgroup took 7 x 7.6 and 52 us:
// the commitment 151 -> 140 us, that of 235 MB 293 -> 279 us.  A round form with a
// shorter dependent chain and one more instruction was slower (140 -> 145 us):
// issue bounds the rounds' wave too.
__global__ __launch_bounds__(kTopThreads) void tree_kernel(const uint32_t* in, uint64_t n_in,
                                                           uint32_t* out, uint8_t* digest) {
  constexpr int kPairs = kTopNodes / 2;
  static_assert(kTopThreads == 2 * kPairs, "one thread of each kind per pair");
  // Node words (word-major: lanes read neighbouring nodes) and the words in flight.
  __shared__ uint32_t node[2][8][kTopNodes];
  __shared__ Sched<kPairs> sched[2];
  const int tid = threadIdx.x;
  const bool rounds = tid < kPairs;  // uniform over a wave
  const int i = rounds ? tid : tid - kPairs;
  const uint64_t first = static_cast<uint64_t>(blockIdx.x) * kTopNodes;
  const uint64_t left = n_in - first;
  int n = static_cast<int>(left < static_cast<uint64_t>(kTopNodes) ? left : kTopNodes);
  for (int w = tid; w < n * 8; w += kTopThreads) node[0][w % 8][w / 8] = in[first * 8 + w];
  __syncthreads();
  int cur = 0;
  while (n > 1) {
    const int n_out = (n + 1) / 2;
    const bool pair = 2 * i + 1 < n;
    uint32_t H[8], s[8];  // rounds: the chaining value and the working variables
    uint32_t W[16];       // schedule: the rolling message words
    if (rounds) {
#pragma unroll
      for (int k = 0; k < 8; ++k) H[k] = s[k] = kH0[k];
    }
    // The 65 bytes make two blocks of four 16-word groups; in step t the rounds
    // take group t - 1 while group t is made.
#pragma unroll
    for (int t = 0; t <= 8; ++t) {
      if (rounds) {
        if (t > 0 && pair) {
          sched[(t - 1) & 1].rounds(i, s);
          if (t % 4 == 0) {
#pragma unroll
            for (int k = 0; k < 8; ++k) s[k] = H[k] = H[k] + s[k];
          }
        }
      } else if (t < 8 && pair) {
        if (t == 0) {  // 0x01 || left || first 31 bytes of right
          uint32_t prev = 0x01u;
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const uint32_t x = node[cur][j % 8][2 * i + j / 8];
            W[j] = (prev << 24) | (x >> 8);
            prev = x;
          }
        } else if (t == 4) {  // right's last byte, padding and bit length
          W[0] = (node[cur][7][2 * i + 1] << 24) | 0x00800000u;
#pragma unroll
          for (int j = 1; j < 15; ++j) W[j] = 0;
          W[15] = 65 * 8;
        } else {
#pragma unroll
          for (int j = 0; j < 16; ++j) extend(W, j);
        }
        sched[t & 1].put(i, t % 4, W);
      }
      if (t < 8) __syncthreads();
    }
    if (rounds && i < n_out) {
      if (!pair) {  // odd last node carried up
#pragma unroll
        for (int k = 0; k < 8; ++k) H[k] = node[cur][k][2 * i];
      }
#pragma unroll
      for (int k = 0; k < 8; ++k) node[cur ^ 1][k][i] = H[k];
    }
    __syncthreads();
    cur ^= 1;
    n = n_out;
  }
  if (digest) {  // SHA-256's byte order
    if (tid < 32) digest[tid] = static_cast<uint8_t>(node[cur][tid / 4][0] >> (24 - 8 * (tid % 4)));
  } else if (tid < 8) {
    out[static_cast<uint64_t>(blockIdx.x) * 8 + tid] = node[cur][tid][0];
  }
}

// SHA-256 of the empty message (the commitment of zero bytes).
__global__ __launch_bounds__(64) void empty_kernel(uint8_t* digest) {
  uint32_t H[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) H[k] = kH0[k];
  uint32_t W[16];
  W[0] = 0x80000000u;
#pragma unroll
  for (int j = 1; j < 16; ++j) W[j] = 0;
  compress(H, W);
  const int tid = threadIdx.x;
  if (tid < 32) digest[tid] = static_cast<uint8_t>(H[tid / 4] >> (24 - 8 * (tid % 4)));
}

unsigned grid_for(uint64_t items, int threads) {
  return static_cast<unsigned>((items + threads - 1) / threads);
}

}  // namespace

uint64_t commit_leaves(uint64_t nbytes, uint32_t chunk) {
  return nbytes == 0 ? 0 : (nbytes + chunk - 1) / chunk;
}

uint64_t commit_workspace_bytes(uint64_t nbytes, uint32_t chunk) {
  const uint64_t leaves = commit_leaves(nbytes, chunk);
  return 32 * (leaves + (leaves + 1) / 2);
}

hipError_t launch_commit(const uint8_t* data, uint64_t nbytes, uint32_t chunk, uint8_t* digest,
                         uint32_t* ws, hipStream_t s) {
  const uint64_t leaves = commit_leaves(nbytes, chunk);
  if (leaves == 0) {
    hipLaunchKernelGGL(empty_kernel, dim3(1), dim3(64), 0, s, digest);
    return hipGetLastError();
  }
  const bool vec = reinterpret_cast<uintptr_t>(data) % 16 == 0 && chunk % 64 == 0;
  uint32_t* a = ws;                // leaf digests, then every second reduced level
  uint32_t* b = ws + leaves * 8;   // the other reduced levels
  if (vec && leaves <= kFewLeaves)
    hipLaunchKernelGGL(leaf_split_kernel, dim3(grid_for(leaves, kSplitLeaves)),
                       dim3(2 * kSplitLeaves), 0, s, data, nbytes, chunk, leaves, a);
  else
    hipLaunchKernelGGL(leaf_kernel, dim3(grid_for(leaves, 256)), dim3(256), 0, s, data, nbytes,
                       chunk, leaves, a, vec ? 1 : 0);
  hipError_t e = hipGetLastError();
  uint64_t n = leaves;
  while (e == hipSuccess && n > static_cast<uint64_t>(kTopNodes)) {
    if (n > kSliceNodes || n <= kLevelNodes) {
      hipLaunchKernelGGL(node_kernel, dim3(grid_for((n + 1) / 2, 256)), dim3(256), 0, s, a, n, b);
      n = (n + 1) / 2;
    } else {
      const unsigned slices = grid_for(n, kTopNodes);
      hipLaunchKernelGGL(tree_kernel, dim3(slices), dim3(kTopThreads), 0, s, a, n, b,
                         static_cast<uint8_t*>(nullptr));
      n = slices;
    }
    e = hipGetLastError();
    uint32_t* t = a;
    a = b;
    b = t;
  }
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(tree_kernel, dim3(1), dim3(kTopThreads), 0, s, a, n,
                     static_cast<uint32_t*>(nullptr), digest);
  return hipGetLastError();
}

}  // namespace repops
