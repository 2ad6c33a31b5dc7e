// Rules that choose between forms of a kernel, as plain functions of sizes: no runtime, no device, so that they can be checked anywhere.
#pragma once
#include <cmath>
#include <cstddef>

namespace br {
namespace rule {

// bf16 outputs of the kernels with one tile of 128x128 or more per workgroup, which take products of any size whose K the persistent
// kernel does not (hidden sizes of an odd multiple of 64).  Up to 160 MB they are stored plainly and the launch that reads them finds
// a part in the memory-side cache; larger ones go past the caches.  Velocity calls of hidden 192, 320, 576, 960, 1344 and 2880, samples of 93
// and 1101 rows, past the caches against plain, by the bytes of the MLP's first layer: 25 to 90 MB 0.960 to 1.066, mean 1.007; 130 and 170 MB
// 0.955 to 1.010, mean 0.996; 250 and 400 MB 0.951 to 1.000, mean 0.975.  (fp32 outputs, the gated residual: the same either way.)
inline bool tile_output_streams(size_t bytes) { return bytes > (size_t)160 << 20; }

// bf16 outputs of the persistent kernel: stored plainly, the launch that reads them finds them in the memory-side cache (256 MB, with the
// operands and the residual stream); else past the caches, which leaves those to the operands.  Below 32 MB the L2 caches of the dies count.  Above,
// a product of small K stores so fast that plain stores of more than the cache takes stall it, and the line lies where that begins.
// Velocity calls (samples of 93, 1101 and 4608 rows), plain against past the caches, mean (least to greatest):
//   hidden           256 to 640                768 to 1024               1280 to 3072
//   MLP's first layer (with GELU)
//     up to  75 MB   0.982 (0.949 to 1.010)    0.990 (0.944 to 1.011)    1.000 (0.938 to 1.021)   [with the QKV rows in front]
//      75 to 100     0.989 (0.953 to 1.011)    1.009 (0.981 to 1.025)    1.000 (0.989 to 1.015)
//     100 to 130     1.035 (1.001 to 1.104)    1.013 (0.993 to 1.037)    0.997 (0.981 to 1.003)
//     130 to 170     1.009 (0.990 to 1.048)    1.008 (0.989 to 1.033)    0.995 (0.987 to 1.002)
//   QKV rows
//      60 to  85     0.993 (0.979 to 1.002)    0.996 (0.985 to 1.004)    1.002 (0.994 to 1.014)
//      85 to 112     0.994 (0.979 to 1.007)    0.998 (0.981 to 1.023)    0.998 (0.992 to 1.004)
//     112 to 130     1.002 (0.988 to 1.015)    1.003 (0.992 to 1.015)    1.000 (0.997 to 1.007)
inline bool persistent_output_stays(size_t bytes, int K, bool gelu) {
  const size_t to = K > 1024 ? (size_t)160 << 20 : !gelu ? 112000000 : K <= 640 ? 100000000 : 75000000;
  return bytes >= (size_t)32 << 20 && bytes <= to;
}

// Parts, with 16 queries a wave instead of 32, that a bf16 attention cuts the last `left` tiles into, behind `whole` tiles in full rounds of the units (of
// one compute die where its pairs are grouped so).  A part takes about 0.6 of its tile's time at twice the workgroups.
// Head dim 128 (256 queries and one workgroup a unit), by the share of the units that the last round takes, us whole / in two / in four parts: 9 % (12 heads
// of 33 272 tokens) 5520 / 5230 / 5025; 16 % (8 of 1101) 28.6 / 19.5 / 15.0; 25 % behind a round (64 of 1101) 60.1 / 51.2 / 47.2; 38 % behind three (48 of
// 4608) 427 / 404 / 424; 42 % (54 of 458) 17.5 / 12.1 / 17.0; 50 % behind thirteen (192 of 4608) 1593 / 1587 / 1607; 69 % behind one (24 of 4608) 212 / 246 / 248.
// Head dim 64 (128 queries, three a unit, which share it): where units would stay empty, or have one workgroup or two, as long as the parts still start all at
// once.  140 to 4096 tokens, 4 and 16 heads, 128 launches, two parts against whole by tiles a unit: up to 0.5 0.85 to 1.01; 0.5 to 0.6 0.92 to 1.02 (16 heads of
// 1101 14.3 / 13.1 us); 0.6 to 0.9 0.98 to 1.05; 0.9 to 1 0.99 to 1.09; 1 to 1.13 0.91 to 0.99 (32 of 1101 19.7 / 18.3); 1.13 to 1.5 0.91 to 0.99 (36 of
// 1101 20.2 / 19.0); 1.5 to 2 1.16 to 1.24 (48 of 1101 21.2 / 25.1); 2 to 2.5 1.04 to 1.17; behind two rounds 950 / 975 us.
inline int attention_parts(int head_dim, bool brief, long long left, long long whole, int units) {
  if (brief) return left * 2 <= units ? 2 : 1;  // (up to 128 or 192 tokens: level within the launch's own time)
  if (head_dim == 128) return left * 4 <= units ? 4 : left * 2 <= units ? 2 : 1;
  return whole == 0 && (left * 5 <= units * 3LL || (left > units && left * 2 <= units * 3LL)) ? 2 : 1;
}

// bf16 attention of head dim 128: whether tiles of 128 queries, two workgroups a unit, take the place of 256 in one workgroup (up to 192 tokens: of 128 in the
// kernel that fetches all keys at once, one workgroup a unit from 129 on).  `tiles128` and `tiles256`, of all units or of one compute die and its.  27 sequences
// of 65 to 8192 tokens, 6 to 1536 pairs, us with 256 / 128, by the number of tiles of 128 a unit:
//   up to a half: 256, in parts (1101 tokens, 6 pairs 15.0 / 18.6).  Up to one: 128, in one round (513 tokens, 48 pairs 18.8 / 12.9; 4608, 6 pairs 67 / 61).
//   More, but one round of 256: 256 (2048 tokens, 24 pairs 51.0 / 53.7; 193, 192 pairs 12.9 / 13.9; not 129 to 192, 144 pairs 14.9 / 11.7).
//   Beyond: 128, whose workgroups hide one another's ends, up to 2048 tokens (192 tokens, 1536 pairs 109 / 74; 320, 768 pairs 92.8 / 57.8; 1101, 768 515 / 458; 210
//   launches of 193 to 2048 tokens, 40 to 1320 pairs 0.65 to 1.02 of the time, mean 0.91), but not where 256 have a last round of at most a quarter, which
//   is cut in four, and 128 begin a second of theirs, from 1025 tokens on (1101, 64 pairs 49.1 / 50.6; 1500, 48 62.5 / 64.6; 2048, 40 84.4 / 86.9).  Longer
//   loops have the bytes into LDS of 256 (2300, 48 pairs 121 / 126; 3000, 56 233 / 239; 4000, 32 to 80 1.03 to 1.06; 4608, 24 208 / 224; 8192, 48 1165 / 1204).
// Up to 128 tokens the short kernel has two workgroups a unit itself (128 tokens, 288 pairs 10.8 / 12.3).
inline bool attention_pair(int tokens, long long tiles128, long long tiles256, int units) {
  if (tokens <= 128 || tiles128 * 2 <= units) return false;
  if (tiles128 <= units || tokens <= 192) return true;
  if (tiles256 <= units || tokens > 2048) return false;
  return tokens <= 1024 || tiles128 <= 2 * units || tiles256 * 4 > units * 5LL;
}

// Whether a network's matrices (of the blocks and the modulation) stay in the memory-side cache (256 MB) from one evaluation to the next: then there is
// nothing to read ahead.  One sample, hidden 512 to 2048, 333 and 1101 tokens, read ahead against not: 58 to 236 MB 1.003 to 1.025; 264 to 278 MB 0.948
// to 1.011 (once 1.064), mean 0.987; 319 to 350 MB 0.909 to 0.995, mean 0.945.
inline bool weights_stay(double bytes) { return bytes <= 256e6; }

// Whether an attention that leaves compute units idle has them read the next products' weights: `room` bytes of a list of `bytes`.  Below a
// thirteenth what is read ahead does not pay for the memory that the attention shares meanwhile.  Velocity calls of one and two samples, with
// against without: hidden 2560 to 3072, 333 to 1101 tokens, 3 to 7 % of the list 1.001 to 1.008; hidden 2048, 200 tokens, 8 and 13 % 0.978 and 0.982;
// 2560, 10 and 11 % 0.978 and 0.982; 1536 and 2048, head dim 128, 20 to 45 % 0.967 to 0.996; 1024, head dims 64 and 128, 44 to 100 % 0.91 to 0.98.
inline bool read_ahead(size_t room, size_t bytes) { return room * 13 >= bytes; }

// fp32 products: the 32x32 tiles up to three a compute unit, whose four waves are faster there (599 x 768 x 768 11.8 us, 13.9 in the best tile of the ring
// kernel; 3833 x 192 x 768 15.1, 16.0; 24 x 64 x 256 by far); beyond, the ring kernel (1101 x 1024 x 4096 98 us, 91; 1624 x 768 x 3072 84, 70).
inline bool f32_small(int M, int N, int units) { return ((long long)M + 31) / 32 * ((N + 31) / 32) <= 3LL * units; }

// The cheapest tile of the ring kernel, 16 rb rows x 64 cb columns: whole rounds of tiles, each its products (a 16 x 64 block of them is K / 300 us
// of a compute unit) and half a block's time that they do not hide, and half a microsecond a tile for first stage and epilogue.  Fitted to 90 shapes
// (M 100 to 40 000, hidden sizes 64 to 1024) in all 22 tiles: 1.6 % slower on average than the best of each shape.  Where a sample
// (rps rows, 0: nothing is looked up per sample) is shorter than the tile, every row would look its gate up by itself.
// (The units come from the caller: asked of the runtime for every tile they cost a microsecond and more of each call.)
constexpr int F32_RING_MAX_RB = 12;
inline void f32_ring_tile(int M, int N, int K, int rps, int units, int* rb, int* cb) {
  double best = 0.0;
  *rb = 0;
  for (int c = 1; c <= 2; ++c)
    for (int r = 2; r <= F32_RING_MAX_RB; ++r) {
      if (r > 2 && rps > 0 && rps < 16 * r) break;
      const double n = (double)((M + 16LL * r - 1) / (16 * r)) * ((N + 64LL * c - 1) / (64 * c)) / units;
      const double cost = std::ceil(n) * (r * c + 0.47) * K / 300.0 + 0.5 * n;
      if (*rb == 0 || cost < best) {
        best = cost;
        *rb = r;
        *cb = c;
      }
    }
}

}  // namespace rule
}  // namespace br
