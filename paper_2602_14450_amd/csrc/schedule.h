// Block orders of the Wilson operator: which half sites a block takes.  Plain
// C++ (constexpr functions serve the host and the device), so that the orders
// can be enumerated without a GPU.
#pragma once

namespace qcd {

struct DslashSched {
  int mode, nsb, ntiles, Lz, Lt, bp, zc, sub, H;  // H: half-sites per parity per block
  int slice, Vh, grid;                            // half sites of a time slice and in all; blocks to launch
};
// orders that stand in for modes 1..3 where a plane does not hold whole blocks
// or Lz is no multiple of 8 (block_pos)
enum { kSchedChunk = 5, kSchedRagged = 6 };

// Whether the form that stages x and y neighbours in LDS applies to blocks of H
// half sites: they cover whole x rows (of at most max_lxh half sites) of one
// (z, t) plane.
constexpr bool lds_rows_apply(int lxh, int Ly, int H, int max_lxh) {
  return lxh <= max_lxh && H % lxh == 0 && Ly % (H / lxh) == 0;
}

struct BlockPos { int h0, tile, sb, cnt; };  // cnt: half sites of the block that exist, -1: no block
constexpr BlockPos block_pos(const DslashSched& sc, int b) {
  BlockPos p{};
  if (sc.mode == kSchedRagged) {
    // the half sites of one time slice are contiguous: each XCD owns an eighth
    // of every slice (a z slab, up to the rounding) and sweeps it in t order, as
    // mode 1, in bp blocks.  Where planes hold whole blocks the parts are whole
    // blocks too, each in one plane, and the last XCDs' may be empty; elsewhere
    // the last block of a part is short and blocks are not aligned to the 64-site
    // layout blocks.  An empty block still writes its partial sums
    const int xcd = b & 7, j = b >> 3;
    p.tile = j % sc.ntiles;
    const int js = j / sc.ntiles;
    const int t = js / sc.bp, k = js - t * sc.bp;
    const int first = xcd * sc.zc + k * sc.H;
    const int end = (xcd + 1) * sc.zc < sc.slice ? (xcd + 1) * sc.zc : sc.slice;
    const int left = end - first < sc.H ? end - first : sc.H;
    p.h0 = t * sc.slice + first;
    p.cnt = left > 0 ? left : 0;
    p.sb = (t * 8 + xcd) * sc.bp + k;
    return p;
  }
  if (sc.mode == kSchedChunk) {
    // each XCD takes its own eighth of the blocks in index order: t slabs, whose
    // z neighbours stay in its L2 and whose t neighbours do where three slices fit
    const int xcd = b & 7, j = b >> 3;
    p.tile = j % sc.ntiles;
    p.sb = xcd * sc.zc + j / sc.ntiles;
    p.h0 = p.sb * sc.H;
    p.cnt = p.sb >= sc.nsb ? -1 : (sc.Vh - p.h0 < sc.H ? sc.Vh - p.h0 : sc.H);
    return p;
  }
  if (sc.mode == 4) {
    // XCD xcd owns time slices [xcd*zc, (xcd+1)*zc) and sweeps them in z
    // order, all slices of one z plane (and all right-hand-side tiles) back
    // to back: z-neighbours stay in its L2 from the previous step, t-neighbours
    // are in the same step, and only the two slab faces in t are foreign
    const int xcd = b & 7, j = b >> 3;
    p.tile = j % sc.ntiles;
    const int js = j / sc.ntiles;
    const int per_z = sc.zc * sc.bp;
    const int z = js / per_z, rem = js - z * per_z;
    const int tl = rem / sc.bp, yb = rem - tl * sc.bp;
    p.sb = ((xcd * sc.zc + tl) * sc.Lz + z) * sc.bp + yb;
  } else if (sc.mode >= 1) {
    // XCD xcd owns z planes [xcd*zc, (xcd+1)*zc), swept as `sub` thinner
    // slabs one after the other, each in t order
    const int xcd = b & 7, j = b >> 3;
    p.tile = j % sc.ntiles;
    const int js = j / sc.ntiles;
    const int zs = sc.zc / sc.sub;            // z planes per sub-slab
    const int per_t = zs * sc.bp;
    const int per_sub = per_t * sc.Lt;
    const int sub = js / per_sub, r1 = js - sub * per_sub;
    const int t = r1 / per_t, rem = r1 - t * per_t;
    const int zl = rem / sc.bp, yb = rem - zl * sc.bp;
    p.sb = (t * sc.Lz + xcd * sc.zc + sub * zs + zl) * sc.bp + yb;
  } else {
    p.tile = b % sc.ntiles;
    p.sb = b / sc.ntiles;
  }
  p.h0 = p.sb * sc.H;
  p.cnt = sc.Vh - p.h0 < sc.H ? sc.Vh - p.h0 : sc.H;
  return p;
}

// The order of mode `mode` (0..4, as qcd_set_dslash_tuning's sched) for n
// right-hand sides, T of them in a block's adjacent lanes; eo: one parity.
constexpr DslashSched make_sched(int lxh, int Ly, int Lz, int Lt, int mode, int T, int n, bool eo) {
  DslashSched s{};
  const int plane = lxh * Ly;
  s.slice = plane * Lz;
  s.Vh = s.slice * Lt;
  s.H = (eo ? 256 : 128) / T;  // half sites of one parity (eo) or of each parity per block
  s.nsb = (s.Vh + s.H - 1) / s.H;
  s.ntiles = n / T;
  s.mode = 0;
  s.Lz = Lz;
  s.Lt = Lt;
  s.bp = 1;
  s.zc = 1;
  s.sub = 1;
  s.grid = s.nsb * s.ntiles;
  if (mode == 4) {
    // XCD slabs of Lt/8 time slices, each swept in z order
    if (plane % s.H == 0 && Lt % 8 == 0) {
      s.mode = 4;
      s.bp = plane / s.H;
      s.zc = Lt / 8;
    }
    return s;
  }
  // mode m = 1..3: XCD slabs of Lz/8 planes, each swept as 2^(m-1) sub-slabs in t order
  const int sub = mode >= 1 ? 1 << (mode - 1) : 1;
  if (mode >= 1 && plane % s.H == 0 && Lz % (8 * sub) == 0) {
    s.mode = mode;
    s.bp = plane / s.H;
    s.zc = Lz / 8;
    s.sub = sub;
    return s;
  }
  if (mode == 0) return s;
  // Planes that do not hold whole blocks, or Lz not a multiple of 8: eighths of
  // each time slice where the short block at the end of each leaves at most an
  // eighth of the lanes idle and three slices are past an XCD's L2, else t slabs
  // (index order, 8 blocks per XCD in turn / eighths of a slice / t slabs, us:
  // D at 24^3 x 48 FP64 172 / 125 / 143, FP16 36.8 / 26.3 / 25.2; at 20^3 x 40
  // FP16 19.4 / 14.7 / 13.8; at 40^4 FP64 666 / 498 / 551; at 18 x 22 x 16 x 30
  // FP16, 29 % idle, 12.1 / 11.1 / 9.0; the one-parity operators at 24^3 x 48
  // FP64, 19 % idle, 195 / 170 / 167, at 30^3 x 60 FP16, 6 %, 116 / 112 / 123).
  // Where a plane holds whole blocks an XCD's part is rounded up to whole
  // blocks: the LDS forms need every block to be x rows of one plane (index order
  // / eighths of whole blocks, us: D at 32 x 24 x 18 x 64 FP16 50.4 / 35.0, FP32
  // 108 / 76, FP64 226 / 176; at 32 x 32 x 20 x 64 55.2 / 50.7, 122 / 116, 277 /
  // 249; the one-parity operators at 32 x 16 x 30 x 64 77.9 / 68.3, 134 / 117, 267
  // / 241).
  const int part = (s.slice + 7) / 8, bp = (part + s.H - 1) / s.H;
  if ((bp * s.H - part) * 8 <= part && s.slice >= 6144) {
    s.mode = kSchedRagged;
    s.zc = plane % s.H == 0 ? bp * s.H : part;
    s.bp = bp;
    s.nsb = 8 * Lt * bp;
    s.grid = s.nsb * s.ntiles;
  } else {
    s.mode = kSchedChunk;
    s.zc = (s.nsb + 7) / 8;
    s.grid = 8 * s.zc * s.ntiles;
  }
  return s;
}

}  // namespace qcd
