// Geometry of the two-step kernel: two time steps in one pass over the
// populations.
//
// A block owns a tile of one x-block (64 nodes) by TY span rows and marches
// up its range of z planes. For each plane it makes the first step on the
// tile and the ring of nodes around it (TY + 2 row waves; the ring's two
// columns in x share one further wave) and hands the results to the second
// step through LDS: each first-step population p of node n belongs to the
// second step's pull at n + c_p, so it is written where that node, in its own
// place, reads it (population opp(p) of n itself when n + c_p is beyond a
// wall: the half-way bounce-back). A population with c_z = +1 is needed one
// plane later than one with c_z = 0, one with c_z = -1 one plane earlier: the
// tile keeps the downward populations of one plane, the resting ones of one
// plane and the upward ones of two.
//
// Everything here runs on the host as well, where the addressing is checked.
#pragma once

#include "lattice.h"

namespace lbm {

// both lattices of a model as one list: flow populations first, then scalar
template <class LF, class LS>
struct Pops {
  static constexpr int Q = LF::Q + LS::Q;
  static constexpr bool flow(int a) { return a < LF::Q; }
  static constexpr int cx(int a) { return flow(a) ? LF::cx[a] : LS::cx[a - LF::Q]; }
  static constexpr int cy(int a) { return flow(a) ? LF::cy[a] : LS::cy[a - LF::Q]; }
  static constexpr int cz(int a) { return flow(a) ? LF::cz[a] : LS::cz[a - LF::Q]; }
  static constexpr int opposite(int a) {
    return flow(a) ? opp<LF>(a) : LF::Q + opp<LS>(a - LF::Q);
  }
  static constexpr int count(int s) {
    int n = 0;
    for (int a = 0; a < Q; ++a) n += cz(a) == s;
    return n;
  }
  // place of population a among those of its c_z
  static constexpr int rank(int a) {
    int n = 0;
    for (int b = 0; b < a; ++b) n += cz(b) == cz(a);
    return n;
  }
  static constexpr int kDown = count(-1), kRest = count(0), kUp = count(1);
  // LDS slots, each TY rows of kPitch elements: the downward populations, the
  // upward ones of even and of odd planes, the resting ones
  static constexpr int kSlots = kDown + 2 * kUp + kRest;
};

// one LDS row: a pad, 64 nodes, a pad (a push across the tile's edge in x
// lands in a pad and is never read)
constexpr int kPitch = kXB + 2;

// tiles of a launch: x-blocks by groups of ty rows by chunks of zc planes
struct TwoStep {
  int ntx, nty, zc, nblocks;
};

// rows of a tile by element size: what 168 (FP32, 3 waves per SIMD) and 256
// (FP64, 2 waves) registers and the LDS allow
constexpr int two_step_rows(int bytes) { return bytes == 8 ? 5 : 8; }

// The split into chunks that takes the fewest plane iterations: blocks run in
// rounds of one per CU, and each costs its planes, the two first-step planes
// at its ends and about one more to fill and drain. Returns that number.
inline int64_t two_step_plan(const Grid& g, int ty, int cus, TwoStep& s) {
  s.ntx = g.nxb;
  s.nty = (g.ny + ty - 1) / ty;
  const int64_t tiles = (int64_t)s.ntx * s.nty;
  int64_t best = INT64_MAX;
  for (int c = 1; c <= g.nz; ++c) {
    const int zc = (g.nz + c - 1) / c;
    if ((g.nz + zc - 1) / zc != c) continue;
    const int64_t cost = (tiles * c + cus - 1) / cus * (zc + 3);
    if (cost < best) {
      best = cost;
      s.zc = zc;
      s.nblocks = (int)(tiles * c);
    }
  }
  return best;
}

// Plane iterations that a pair may spend per one that the grid needs and still be
// no slower than two single steps, by collision. Break-even is the gain of a pair
// (40 steps, single / paired) times spent / work, measured on some 45 grids each on
// both sides of the line: cumulant with unit rates + D3Q7 FP32 2.0 to 2.9, FP64 2.1 to
// 2.9, + D3Q27 FP32 1.9 to 2.5; parametrised 1.9 to 2.7, 1.9 to 3.2 and 1.7 to 2.2; BGK
// FP64 1.8 to 2.7 (the least of them on large grids, which the other condition of
// two_step_pays holds to less). The given rates transform forward as well and have
// less to gain: FP32 + D3Q7 1.5 to 2.2, + D3Q27 1.5 to 1.9; FP64 1.9 to 2.9 where memory
// feeds the single steps, 1.7 to 2.1 where the last-level cache does. What a line at
// 1.6 work + 2 alone cost them: 655 x 27 x 93 + D3Q27 127 us per step single, 148 paired;
// 962 x 19 x 90 + D3Q7 85 / 92; FP64 372 x 29 x 32 31.6 / 35.4.
enum class Rates { kUnit, kParametrised, kGiven };
inline double two_step_limit(int qt, int bytes, Rates rates, size_t state_bytes) {
  if (rates == Rates::kGiven) {
    if (bytes == 4) return qt == 54 ? 1.5 : 1.67;
    return state_bytes > ((size_t)128 << 20) ? 2.0 : 1.7;
  }
  if (qt == 25) return 1.9;
  return qt == 54 && rates == Rates::kParametrised ? 1.9 : 2.05;
}

// Two steps at a time halve the traffic but need a grid whose tiles keep every
// CU busy, and one that the caches do not hold anyway: `work` is the tile planes
// per CU if nothing were lost to ragged tiles, chunk ends and a part-filled last
// round, `spent` those that the plan takes. Single against paired, us per step:
// cumulant + D3Q7 FP32 277 x 23 x 41 (work 2.0, spent 6) 13.8 / 15.1, 427 x 23 x 47 (3.5,
// 7) 20.3 / 18.8, 512 x 32 x 64 (8, 11) 55 / 38, 1024 x 64 x 128 (64, 67) 394 / 255; FP64
// 186 x 33 x 40 (3.0, 7) 21.9 / 22.6, 372 x 29 x 32 (4.2, 8) 30.6 / 28.2, 1024 x 64 x 128 819 /
// 560; cumulant + D3Q27 FP32 389 x 11 x 106 (3.5, 9) 34.3 / 35.8, 423 x 33 x 56 (6.0, 11)
// 61.9 / 53.5, 1024 x 64 x 128 656 / 401; BGK FP64 335 x 40 x 25 (4.1, 8) 22.0 / 22.6, 381 x 13
// x 105 (6.4, 11) 33.0 / 31.1, 1024 x 64 x 128 599 / 443. A pull reaches over three planes
// with 32-bit offsets, which bounds their size.
inline bool two_step_pays(const Grid& g, int qt, int bytes, int cus, Rates rates, size_t state_bytes) {
  const int64_t plane = (int64_t)g.ny * g.nxb * kXB * qt * bytes;
  if (3 * plane >= ((int64_t)1 << 31)) return false;
  const int ty = two_step_rows(bytes);
  TwoStep s;
  const double spent = (double)two_step_plan(g, ty, cus, s);
  const double work = (double)g.n / ((double)kXB * ty * cus);
  return spent <= 1.6 * work + 2.0 && spent <= two_step_limit(qt, bytes, rates, state_bytes) * work;
}

struct Tile {
  int xb, y0, rows, z0, z1;  // rows of the tile (ty, fewer at the span's end); planes z0 .. z1 - 1
};

// Blocks go round-robin to the 8 XCDs; each XCD takes a contiguous run of
// tiles, y fastest, so that the ring rows that neighbouring tiles share are
// read through one L2.
LBM_HD Tile tile_of(const Grid& g, const TwoStep& s, int ty, int b) {
  int l = xcd_run_order(b, s.nblocks);
  Tile t;
  const int yt = l % s.nty;
  l /= s.nty;
  t.xb = l % s.ntx;
  const int c = l / s.ntx;
  t.y0 = yt * ty;
  t.rows = g.ny - t.y0 < ty ? g.ny - t.y0 : ty;
  t.z0 = c * s.zc;
  t.z1 = t.z0 + s.zc < g.nz ? t.z0 + s.zc : g.nz;
  return t;
}

// The first step's node of a lane: wave w < ty + 2 takes the row t = w - 1 of
// the tile (-1 and rows: the ring), wave ty + 2 the ring's columns.
struct Lane {
  int x, t, y;  // node column, tile row, span position
  int side;     // 0: a row wave; +1 / -1: ring column left / right of the tile (the c_x it pushes)
  bool active;  // the node exists
};

LBM_HD Lane lane_of(const Grid& g, const Tile& tile, int ty, int w, int lane) {
  Lane l;
  int t;
  if (w < ty + 2) {
    l.side = 0;
    l.x = tile.xb * kXB + lane;
    t = w;
  } else {
    const bool right = lane >= ty + 2;
    l.side = right ? -1 : 1;
    l.x = right ? tile.xb * kXB + kXB : tile.xb * kXB - 1;
    t = right ? lane - (ty + 2) : lane;
  }
  l.active = l.x >= 0 && l.x < g.nx && t < tile.rows + 2;
  // a lane without a node addresses the tile's first one
  if (!l.active) {
    l.x = tile.xb * kXB;
    t = 1;
  }
  l.t = t - 1;
  const int y = tile.y0 + l.t;
  l.y = y < 0 ? g.ny - 1 : (y >= g.ny ? y - g.ny : y);
  return l;
}

// byte offsets, inside one z plane, of the sources of a node's pulls:
// off[c_y + 1][c_x + 1] is the node at (x - c_x, y - c_y), with x held at the
// walls (the bounce-back replaces those values). A plane is below 4 GiB.
template <int QT, typename ST>
LBM_HD void plane_offsets(const Grid& g, int x, int y, uint32_t (&off)[3][3]) {
  const int ym = y == 0 ? g.ny - 1 : y - 1, yp = y == g.ny - 1 ? 0 : y + 1;
  const int ys[3] = {yp, y, ym};  // c_y = -1, 0, 1
  const int xs[3] = {x == g.nx - 1 ? x : x + 1, x, x == 0 ? x : x - 1};
#pragma unroll
  for (int j = 0; j < 3; ++j)
#pragma unroll
    for (int i = 0; i < 3; ++i)
      off[j][i] = (uint32_t)(elem_index<QT>(g, 0, ys[j], xs[i]) * (int64_t)sizeof(ST));
}

// A lane's own place in an LDS row: its node, or, for a ring column, the tile
// column that it pushes to.
LBM_HD int lds_lane(const Lane& l, int lane) {
  return l.t * kPitch + 1 + (l.side == 0 ? lane : (l.side > 0 ? 0 : kXB - 1));
}

// first element of the LDS slots of class CZ for the second step's plane z
template <class P, int TY>
LBM_HD int class_base(int cz, int z) {
  constexpr int kSlot = TY * kPitch;
  return cz < 0 ? 0 : (cz > 0 ? (P::kDown + (z & 1) * P::kUp) * kSlot : (P::kDown + 2 * P::kUp) * kSlot);
}

// element, from a class's base at the lane's own place, of population a at the
// node (cx, cy) away
template <class P, int TY>
constexpr int class_offset(int a, int cx, int cy) {
  return P::rank(a) * (TY * kPitch) + cy * kPitch + cx;
}

// Pushes of the first step's populations with c_z = CZ to their places in LDS:
// put(a, index). base: the class's base plus the lane's place. row: the wave is
// a row wave (uniform; its tile row tw is uniform too), else it holds the
// ring's columns, whose pushes off the tile go to a pad instead.
template <class P, int TY, int CZ, class Put>
LBM_HD void push_class(const Lane& l, bool row, int tw, int rows, int base, int at, Put&& put) {
  if (row) {
    static_for<0, 3>([&](auto jc) {
      constexpr int cy = decltype(jc)::value - 1;
      if ((unsigned)(tw + cy) < (unsigned)rows)
        static_for<0, P::Q>([&](auto ac) {
          constexpr int a = decltype(ac)::value;
          if constexpr (P::cz(a) == CZ && P::cy(a) == cy)
            put(ac, base + class_offset<P, TY>(a, P::cx(a), cy));
        });
    });
  } else {
    static_for<0, 6>([&](auto jc) {
      constexpr int cy = decltype(jc)::value / 2 - 1, cx = decltype(jc)::value % 2 ? 1 : -1;
      int t = l.t;
#ifdef __HIP_DEVICE_COMPILE__
      asm volatile("" : "+v"(t));  // tested here, not kept over the planes
#endif
      const bool ok = l.side == cx && (unsigned)(t + cy) < (unsigned)rows;
      const int to = base - at + (ok ? at + cy * kPitch : 0);
      static_for<0, P::Q>([&](auto ac) {
        constexpr int a = decltype(ac)::value;
        if constexpr (P::cz(a) == CZ && P::cy(a) == cy && P::cx(a) == cx)
          put(ac, to + class_offset<P, TY>(a, 0, 0));
      });
    });
  }
}

// Bounce-back pushes of plane k by a row wave of the tile's own rows: a
// population bound for a wall comes back to its own node as the opposite one.
// base[c_z + 1]: the bases of plane k's classes plus the lane's place.
template <class P, int TY, class Put>
LBM_HD void push_bounce(const Grid& g, const Lane& l, const int (&base)[3], int k, Put&& put) {
  static_for<0, 9>([&](auto jc) {
    constexpr int cx = decltype(jc)::value / 3 - 1, cz = decltype(jc)::value % 3 - 1;
    if constexpr (cx != 0 || cz != 0) {
      bool wall = false;
      if constexpr (cz != 0) wall = k == (cz > 0 ? g.nz - 1 : 0);
      if constexpr (cx != 0) wall = wall || l.x == (cx > 0 ? g.nx - 1 : 0);
      if (wall)
        static_for<0, P::Q>([&](auto ac) {
          constexpr int a = decltype(ac)::value;
          if constexpr (P::cx(a) == cx && P::cz(a) == cz)
            put(ac, base[1 - cz] + class_offset<P, TY>(P::opposite(a), 0, 0));
        });
    }
  });
}

}  // namespace lbm
