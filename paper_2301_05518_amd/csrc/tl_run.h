// Whole-run kernel: all n smearing steps of a plan in one launch (step variant 9).
//
// What bounds the step kernels on lattices up to 64^3 is not the arithmetic: below 48^3 a
// launch costs about 5 us whatever it does, and on 64^3 every step streams the two-links
// again although they never change.  Here a workgroup keeps its share of the two-links in
// registers (forward and backward ones of one site per thread: 108 VGPRs in FP32) for the
// whole run, its colour vectors in LDS, and exchanges only the outer sites of its tile.
//
// Hops of two sites decouple a slice into cells: the sites of one parity in every direction
// of even extent (a direction of odd extent is one chain 0, 2, 4, ... around the ring; a
// one-link field is one cell).  Inside a cell the hops are nearest-neighbour and periodic.
// A unit of work is one cell of one RHS group; it is cut into tiles, one per workgroup, and a
// team of workgroups runs the unit's n steps together.
//
// Exchange.  A thread whose site has a neighbour in another tile publishes its vector in the
// team's scratch memory as 16-byte words of 12 payload bytes and a 4-byte tag that names the
// step; a reader loads a word until it holds the tag it waits for.  So there is no flag, no
// fence and no barrier between workgroups: one store-to-load latency per step (about 1.3 us,
// against 4 us with separate flags, and 40 us with the agent-scope fences that plain loads
// would need).  The loads are device-scope: they bypass the per-CU caches and are coherent.
// The stores are device-scope where a reader sits on another XCD, plain otherwise (they then
// stay in the L2 both share; device-scope stores write through to memory, which alone took a
// 48^3 FP32 step from 4.1 to 5.6 us).  A lane's aligned 16-byte word is one request, so a
// tag never arrives without its payload.  Two scratch planes alternate; a tile overwrites
// step s - 1 with step s + 1 only after it has read step s of all its neighbour tiles, each
// of which published step s after it had read step s - 1 completely.  Tags never repeat
// within a launch, and every launch begins at a new epoch (kept in device memory, advanced
// by the launch's last workgroup), so a graph replay never takes an old word for a new one.
//
// Progress.  Nothing assumes that the whole grid is resident.  A team is made of workgroups
// that run: each enrols when it starts, the first one closes the team when all expected
// members have come or after a wait in proportion to the launch (about what it should take),
// later ones leave.  An incomplete team leaves too if complete ones can take its work; else it
// runs the same exchange with several tiles per workgroup and the two-links read from memory
// each step (run_slow).  Teams take their shares of the
// units from a common counter.  Microseconds per run with 1 and with 16 CUs held by another
// stream: with 2 ms of waiting, no leaving, and run_slow one RHS and neighbour at a time; now; and
// the step kernels.  32^3 FP64 3 RHS, 40 steps: 548 and 1537; 300 and 1030; 2090.  64^3 FP32 6
// RHS, 20 steps: 607 and 5265; 608 and 2140; 1000.  64^3 FP32 24 RHS, 60 steps: 29900 and 17500;
// 5790 and 19900; 12000.  96^3 BF16 3 RHS (a team of most CUs), 20 steps: 10030 and 10360; 3710
// and 3910; 990.  run_slow reads every neighbour from memory, so where every team lacks a member
// and the lattice is large it is behind the step kernels.
// Every wait is bounded; where one runs out the kernel sets *fail, leaves NaNs in the results
// of the tile concerned (in run_slow: takes them for the words that did not come), and ends.
//
// Measured, microseconds per step with everything a run does once spread over its steps, before
// (the tuned step kernels in a graph) and now: 8^3 FP64 1 RHS 5.2 -> 1.2; 32^3 FP64 3 RHS
// 8.9 -> 4.0; 48^3 3 RHS FP32 11.1 -> 3.4, F16S 9.3 -> 3.8; 24^3 + 32^3 + 48^3 BF16 21 RHS
// 24 -> 18.4; 64^3 FP32 24 RHS 104 -> 51 to 55 (about 50 a step and 300 once).  At 64^3 the vector
// units issue 92% of the cycles the kernel runs (1.45 M instructions of 4 cycles per SIMD in 6.27 M
// cycles), so what is left there is the instruction count: 251 per site and RHS, the fetch waves'
// included, 222 of them FMAs.  A copy that does not wait for its neighbours takes 41.5 instead of
// 50 us a step there, 3.0 instead of 3.3 at 48^3 FP32, and 2.2 instead of 4.0 at 32^3 FP64, which is
// the one that the exchange bounds.
#pragma once

#include <type_traits>

#include "tl_step.h"

namespace tl {

namespace {

// Raw storage words of a colour vector and their exchange form.
template <int P> struct Exch;
template <> struct Exch<F64> {
  static constexpr int ND = 12, NW = 4;   // dwords, tagged words
  static __device__ __forceinline__ void load(const char* b, int64_t Vp, int64_t i, uint32_t (&d)[ND]) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
      const v4u w = ldg<v4u>(b + (c * Vp + i) * 16);
      d[4 * c] = w.x; d[4 * c + 1] = w.y; d[4 * c + 2] = w.z; d[4 * c + 3] = w.w;
    }
  }
  static __device__ __forceinline__ void decode(const uint32_t (&d)[ND], double (&v)[6]) {
#pragma unroll
    for (int c = 0; c < 6; c++) v[c] = __hiloint2double((int)d[2 * c + 1], (int)d[2 * c]);
  }
  static __device__ __forceinline__ void encode(const double (&v)[6], uint32_t (&d)[ND]) {
#pragma unroll
    for (int c = 0; c < 6; c++) {
      d[2 * c] = (uint32_t)__double2loint(v[c]);
      d[2 * c + 1] = (uint32_t)__double2hiint(v[c]);
    }
  }
};
template <> struct Exch<F32> {
  static constexpr int ND = 6, NW = 2;
  static __device__ __forceinline__ void load(const char* b, int64_t Vp, int64_t i, uint32_t (&d)[ND]) {
    const v4u a = ldg<v4u>(b + i * 16);
    const v2u c = ldg<v2u>(b + 16 * Vp + i * 8);
    d[0] = a.x; d[1] = a.y; d[2] = a.z; d[3] = a.w; d[4] = c.x; d[5] = c.y;
  }
  static __device__ __forceinline__ void decode(const uint32_t (&d)[ND], float (&v)[6]) {
#pragma unroll
    for (int c = 0; c < 6; c++) v[c] = __uint_as_float(d[c]);
  }
  static __device__ __forceinline__ void encode(const float (&v)[6], uint32_t (&d)[ND]) {
#pragma unroll
    for (int c = 0; c < 6; c++) d[c] = __float_as_uint(v[c]);
  }
};
template <> struct Exch<F16S> {
  static constexpr int ND = 4, NW = 2;
  static __device__ __forceinline__ void load(const char* b, int64_t, int64_t i, uint32_t (&d)[ND]) {
    const v4u a = ldg<v4u>(b + i * 16);
    d[0] = a.x; d[1] = a.y; d[2] = a.z; d[3] = a.w;
  }
  static __device__ __forceinline__ void decode(const uint32_t (&d)[ND], float (&v)[6]) {
    f16s_decode(v4u{d[0], d[1], d[2], d[3]}, v);
  }
  static __device__ __forceinline__ void encode(const float (&v)[6], uint32_t (&d)[ND]) {
    const v4u a = f16s_encode(v);
    d[0] = a.x; d[1] = a.y; d[2] = a.z; d[3] = a.w;
  }
};
template <> struct Exch<BF16> {
  static constexpr int ND = 3, NW = 1;
  static __device__ __forceinline__ void load(const char* b, int64_t Vp, int64_t i, uint32_t (&d)[ND]) {
    const v2u a = ldg<v2u>(b + i * 8);
    d[0] = a.x; d[1] = a.y; d[2] = ldg<uint32_t>(b + 8 * Vp + i * 4);
  }
  static __device__ __forceinline__ void decode(const uint32_t (&d)[ND], float (&v)[6]) {
#pragma unroll
    for (int c = 0; c < 3; c++) {
      v[2 * c] = bf16_to_f32(d[c] & 0xffffu);
      v[2 * c + 1] = bf16_to_f32(d[c] >> 16);
    }
  }
  static __device__ __forceinline__ void encode(const float (&v)[6], uint32_t (&d)[ND]) {
#pragma unroll
    for (int c = 0; c < 3; c++) d[c] = pack_bf16(v[2 * c], v[2 * c + 1]);
  }
};

// The exchange words of one plane pair entry: word q of a vector holds dwords 3q .. 3q + 2.
template <int P>
__device__ __forceinline__ v4u exch_word(const uint32_t (&d)[Exch<P>::ND], int q, uint32_t tag) {
  constexpr int ND = Exch<P>::ND;
  return v4u{d[3 * q], 3 * q + 1 < ND ? d[3 * q + 1] : 0u, 3 * q + 2 < ND ? d[3 * q + 2] : 0u, tag};
}
template <int P>
__device__ __forceinline__ void exch_dwords(const v4u (&w)[Exch<P>::NW], uint32_t (&d)[Exch<P>::ND]) {
#pragma unroll
  for (int k = 0; k < Exch<P>::ND; k++) d[k] = w[k / 3][k % 3];
}

// What a reader of run_slow that gives up takes for a word: NaNs in every format (all exponent bits set).
__device__ __forceinline__ v4u exch_nan() { return v4u{~0u, ~0u, ~0u, ~0u}; }

// A site's R vectors in LDS: one record, so that every access of a neighbour is one address
// plus an immediate offset (run_record bytes; the odd multiple of 8 for four RHS keeps the
// 16 lanes of an 8-byte access phase on different banks).
template <int R>
__device__ __forceinline__ void rec_put(unsigned char* p, int r, const float (&v)[6]) {
#pragma unroll
  for (int c = 0; c < 3; c++) *reinterpret_cast<v2f*>(p + 24 * r + 8 * c) = v2f{v[2 * c], v[2 * c + 1]};
}
template <int R>
__device__ __forceinline__ void rec_get(const unsigned char* p, int r, float (&v)[6]) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    const v2f w = *reinterpret_cast<const v2f*>(p + 24 * r + 8 * c);
    v[2 * c] = w.x;
    v[2 * c + 1] = w.y;
  }
}
template <int R>
__device__ __forceinline__ void rec_put(unsigned char* p, int r, const double (&v)[6]) {
#pragma unroll
  for (int c = 0; c < 3; c++) *reinterpret_cast<v2d*>(p + 48 * r + 16 * c) = v2d{v[2 * c], v[2 * c + 1]};
}
template <int R>
__device__ __forceinline__ void rec_get(const unsigned char* p, int r, double (&v)[6]) {
#pragma unroll
  for (int c = 0; c < 3; c++) {
    const v2d w = *reinterpret_cast<const v2d*>(p + 48 * r + 16 * c);
    v[2 * c] = w.x;
    v[2 * c + 1] = w.y;
  }
}

constexpr int kDeviceScope = 16;   // sc1 in a buffer instruction's cache policy

// The word's offset goes into the instruction's vector offset alone.  A store of 128 bits reads its
// data registers after it is issued, and what overwrites them needs a wait state, which the
// compiler inserts only where the scalar offset is not a register.  With part of the offset in one
// the data registers were reused in the next instruction, and under load a store has been seen to
// write the next word's payload under this word's tag, four lanes at a time.
// tests/test_run_stores.py looks for both in the built code.
template <int Scope>
__device__ __forceinline__ void exch_store(v4u w, __amdgpu_buffer_rsrc_t rs, int off) {
  __builtin_amdgcn_raw_buffer_store_b128(w, rs, off, 0, Scope);
}
// The XCD this wave runs on (hardware register XCC_ID).
__device__ __forceinline__ uint32_t xcd_id() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)); }

__device__ __forceinline__ uint32_t ctl_load(const uint32_t* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void ctl_store(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint32_t ctl_add(uint32_t* p, uint32_t v) {
  return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void run_failed(uint32_t* fail) {
  __hip_atomic_store(fail, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Barrier of a workgroup over LDS only: global loads and stores in flight stay in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A value every lane of a wave holds, as a scalar: the compiler cannot see that what comes from
// LDS or from threadIdx / np is the same in all lanes.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

constexpr uint32_t kTeamClosed = 0x40000000u;
constexpr uint32_t kTeamAway = 0x20000000u;   // size of a team that leaves the work to others
// An incomplete team leaves its shares to the complete ones if those then take at most this many
// each: about what a share costs an incomplete team more (run_slow).
constexpr uint32_t kAwayShares = 3;

// Where a workgroup stands: its team and its place there; `expect` workgroups of the grid
// belong to the team.  Workgroups are dispatched round-robin over the XCDs, so a team of up
// to a grid's workgroups per XCD sits on one XCD (its exchange then stays in one L2), a
// larger one on neighbouring XCDs, in equal parts, so that the workgroups it does not need are
// spare on each of them; only speed depends on that.
struct RunPlace {
  int team, rank, expect;
};
__device__ __forceinline__ RunPlace run_place(int team_size) {
  const int per = (int)gridDim.x / kXcds, k = (int)blockIdx.x % kXcds, j = (int)blockIdx.x / kXcds;
  if (j >= per) return {0, 1 << 20, 0};
  if (per >= team_size) {
    const int tpx = per / team_size, q = j / team_size;
    return {q < tpx ? q * kXcds + k : 0, q < tpx ? j - q * team_size : 1 << 20, team_size};
  }
  int xpt = 2;
  while (xpt < kXcds && xpt * per < team_size) xpt *= 2;
  const int expect = min(team_size, xpt * per), part = (expect + xpt - 1) / xpt;
  const int r = (k % xpt) * part + j;
  return {k / xpt, j < part && r < expect ? r : 1 << 20, expect};
}

// A tile of a unit: origin and extent in cell coordinates.
struct RunTile {
  int o[3], e[3];
};
__device__ __forceinline__ RunTile run_tile(const RunUnit& g, int tile) {
  const int ix = tile % g.t[0], iyz = tile / g.t[0], iy = iyz % g.t[1], iz = iyz / g.t[1];
  RunTile r;
  r.o[0] = ix * g.b[0];
  r.o[1] = iy * g.b[1];
  r.o[2] = iz * g.b[2];
#pragma unroll
  for (int d = 0; d < 3; d++) r.e[d] = min(g.b[d], g.c[d] - r.o[d]);
  return r;
}

// Lattice site index of a cell coordinate.
__device__ __forceinline__ int run_site(const RunUnit& g, int hop, int cx, int cy, int cz) {
  int x = g.p[0] + hop * cx, y = g.p[1] + hop * cy, z = g.p[2] + hop * cz;
  x = x >= g.Lx ? x - g.Lx : x;
  y = y >= g.Ly ? y - g.Ly : y;
  z = z >= g.Lz ? z - g.Lz : z;
  return (z * g.Ly + y) * g.Lx + x;
}

// Scratch slot of a cell coordinate: np slots per tile, the tile's sites in x, y, z order.
__device__ __forceinline__ int run_slot(const RunUnit& g, int np, int cx, int cy, int cz) {
  const int ix = cx / g.b[0], iy = cy / g.b[1], iz = cz / g.b[2];
  const int lx = cx - ix * g.b[0], ly = cy - iy * g.b[1], lz = cz - iz * g.b[2];
  return ((iz * g.t[1] + iy) * g.t[0] + ix) * np + (lz * g.b[1] + ly) * g.b[0] + lx;
}

__device__ __forceinline__ int ring(int c, int n) { return c < 0 ? c + n : c >= n ? c - n : c; }

template <int P, typename T>
__device__ __forceinline__ void run_load_w(bool w12, const char* b, int64_t Vp, int64_t i, T (&m)[18]) {
  if (w12) Fmt<P | W12>::load_w(b, Vp, i, m);
  else Fmt<P>::load_w(b, Vp, i, m);
}

// One unit by a team smaller than its tile count: member `me` of `size` takes the tiles me,
// me + size, ... of every step in turn; vectors live in the scratch words, two-links are read
// each step.  Every tile of a step is published before any of the next, so no wait is circular.
// A step costs the latencies of its loads, so a direction's links and the words of all RHS are
// requested together (RC of them at a time, and FP64 one neighbour's, as registers allow).
template <int P, int R>
__device__ void run_slow(const RunArgs& a, const RunUnit& g, int me, int size, uint32_t tag0, int par0, int team,
                         typename Fmt<P>::real alpha, typename Fmt<P>::real beta) {
  using real = typename Fmt<P>::real;
  using X = Exch<P>;
  constexpr int NW = X::NW, RC = R == 4 ? 2 : P == F64 && R == 3 ? 1 : R;
  const int sub = uniform((int)threadIdx.x / a.np), i = (int)threadIdx.x - sub * a.np;
  const int n_tiles = g.t[0] * g.t[1] * g.t[2], bvol = g.b[0] * g.b[1] * g.b[2];
  const int slots = a.team_size * a.np;
  const int64_t plane = (int64_t)a.subs * R * NW * slots * 16;
  char* const base = a.scratch + team * 2 * plane;
  bool dead = false;
  int rr0 = 0;   // first of the RHS in hand
  for (int s = -1; s < a.n_steps; s++) {   // s = -1 publishes the input
    const uint32_t tag = tag0 + (uint32_t)s;
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base + ((par0 + s) & 1) * plane, 0, (int)plane, 0x00027000);
    const __amdgpu_buffer_rsrc_t ws = __builtin_amdgcn_make_buffer_rsrc(base + ((par0 + s + 1) & 1) * plane, 0, (int)plane, 0x00027000);
    auto request = [&](int slot, int r, v4u(&w)[NW]) {
#pragma unroll
      for (int q = 0; q < NW; q++)
        w[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, slot * 16, ((rr0 + r) * NW + q) * slots * 16, kDeviceScope);
    };
    auto request_all = [&](int slot, v4u(&w)[RC][NW]) {
#pragma unroll
      for (int r = 0; r < RC; r++) request(slot, r, w[r]);
    };
    auto settle = [&](int slot, v4u(&w)[RC][NW]) {
      for (int spin = 0;; spin++) {
        bool late = false, miss[RC];
#pragma unroll
        for (int r = 0; r < RC; r++) {
          miss[r] = false;
#pragma unroll
          for (int q = 0; q < NW; q++) miss[r] = miss[r] || w[r][q].w != tag;
          late = late || miss[r];
        }
        if (!late) break;
        const bool give_up = dead || spin >= a.spins;
        if (give_up && !dead) run_failed(a.fail);
        dead = dead || give_up;
        asm volatile("" ::: "memory");
#pragma unroll
        for (int r = 0; r < RC; r++) {
          if (!miss[r]) continue;
          if (!give_up) request(slot, r, w[r]);
#pragma unroll
          for (int q = 0; q < NW; q++) w[r][q] = give_up ? exch_nan() : w[r][q];
        }
        if (give_up) break;
      }
    };
    auto vector = [&](const v4u(&w)[NW], real(&v)[6]) {
      uint32_t e[X::ND];
      exch_dwords<P>(w, e);
      X::decode(e, v);
    };
    for (int tile = me; tile < n_tiles; tile += size) {
      const RunTile tl = run_tile(g, tile);
      const int lx = i % g.b[0], lyz = i / g.b[0], ly = lyz % g.b[1], lz = lyz / g.b[1];
      if (i >= bvol || lx >= tl.e[0] || ly >= tl.e[1] || lz >= tl.e[2]) continue;
      const int cx = tl.o[0] + lx, cy = tl.o[1] + ly, cz = tl.o[2] + lz;
      const int site = run_site(g, a.hop, cx, cy, cz);
      const int own = tile * a.np + i;
#pragma nounroll
      for (rr0 = sub * R; rr0 < (sub + 1) * R; rr0 += RC) {
        auto publish = [&](int r, const uint32_t(&d)[X::ND]) {
#pragma unroll
          for (int q = 0; q < NW; q++)
            exch_store<kDeviceScope>(exch_word<P>(d, q, tag + 1), ws, (own + ((rr0 + r) * NW + q) * slots) * 16);
        };
        if (s < 0) {
          for (int r = 0; r < RC; r++) {
            uint32_t d[X::ND];
            X::load(a.in + g.psi_off + (int64_t)min(rr0 + r, g.nr - 1) * g.rhs_stride, g.Vp, site, d);
            publish(r, d);
          }
          continue;
        }
        real acc[RC][6], v[6];
#pragma unroll
        for (int r = 0; r < RC; r++)
#pragma unroll
          for (int c = 0; c < 6; c++) acc[r][c] = (real)0;
        auto add = [&](const real(&m)[18], const v4u(&w)[RC][NW], bool forward) {
#pragma unroll
          for (int r = 0; r < RC; r++) {
            vector(w[r], v);
            if (forward) mv_acc(m, v, acc[r]);
            else mdv_acc(m, v, acc[r]);
          }
        };
#pragma nounroll
        for (int mu = 0; mu < 3; mu++) {
          const int dx = mu == 0, dy = mu == 1, dz = mu == 2;
          const int bx = ring(cx - dx, g.c[0]), by = ring(cy - dy, g.c[1]), bz = ring(cz - dz, g.c[2]);
          const int fs = run_slot(g, a.np, ring(cx + dx, g.c[0]), ring(cy + dy, g.c[1]), ring(cz + dz, g.c[2]));
          const int bs = run_slot(g, a.np, bx, by, bz);
          const char* W = g.W + mu * g.w_mu_stride;
          v4u f[RC][NW];
          real m[18];
          request_all(fs, f);
          run_load_w<P>(a.w12, W, g.Vp, site, m);
          if constexpr (P == F64) {
            settle(fs, f);
            add(m, f, true);
            request_all(bs, f);
            run_load_w<P>(a.w12, W, g.Vp, run_site(g, a.hop, bx, by, bz), m);
            settle(bs, f);
            add(m, f, false);
          } else {
            v4u b[RC][NW];
            real mb[18];
            request_all(bs, b);
            run_load_w<P>(a.w12, W, g.Vp, run_site(g, a.hop, bx, by, bz), mb);
            settle(fs, f);
            add(m, f, true);
            settle(bs, b);
            add(mb, b, false);
          }
        }
        v4u w[RC][NW];
        request_all(own, w);
        settle(own, w);
#pragma unroll
        for (int r = 0; r < RC; r++) {
          vector(w[r], v);
          real o[6];
#pragma unroll
          for (int c = 0; c < 6; c++) o[c] = fma_(beta, acc[r][c], alpha * v[c]);
          if (s + 1 < a.n_steps) {
            uint32_t d[X::ND];
            X::encode(o, d);
            publish(r, d);
          } else if (rr0 + r < g.nr) {
            Fmt<P>::template store_v<real, false>(a.out + g.psi_off + (int64_t)(rr0 + r) * g.rhs_stride, g.Vp, site, o);
          }
        }
      }
    }
  }
}

// Geometry of a workgroup's tile that its compute and fetch waves share.
struct RunFaces {
  int f[3];    // sites of a face across direction d (0: the direction is not cut, its ends meet)
  int hb[3];   // LDS entry of the first halo site of direction d: faces d-, then d+
};
__device__ __forceinline__ RunFaces run_faces(const RunUnit& g, int np) {
  RunFaces q;
  q.f[0] = g.t[0] > 1 ? g.b[1] * g.b[2] : 0;
  q.f[1] = g.t[1] > 1 ? g.b[0] * g.b[2] : 0;
  q.f[2] = g.t[2] > 1 ? g.b[0] * g.b[1] : 0;
  q.hb[0] = 2 * np;
  q.hb[1] = q.hb[0] + 2 * q.f[0];
  q.hb[2] = q.hb[1] + 2 * q.f[1];
  return q;
}

// Scratch slot of halo site h of a tile (h counts from the first halo entry), -1 for an entry
// past the halo or past a ragged tile's edge.
__device__ __forceinline__ int halo_slot(const RunUnit& g, const RunTile& tl, const RunFaces& fc, int np, int h) {
  int d = -1, q = 0;
  bool plus = false;
#pragma unroll
  for (int e = 0; e < 3; e++) {
    const int u = h - (fc.hb[e] - 2 * np);
    if (fc.f[e] > 0 && u >= 0 && u < 2 * fc.f[e]) {
      d = e;
      plus = u >= fc.f[e];
      q = plus ? u - fc.f[e] : u;
    }
  }
  if (d < 0) return -1;
  const int w = d == 0 ? g.b[1] : g.b[0];   // fast extent of the face
  const int u = q % w, v = q / w;
  const int l[3] = {d == 0 ? 0 : u, d == 0 ? u : d == 1 ? 0 : v, d == 2 ? 0 : v};
  int c[3];
  bool ok = true;
#pragma unroll
  for (int e = 0; e < 3; e++) {
    ok = ok && (d == e || l[e] < tl.e[e]);
    c[e] = e == d ? ring(plus ? tl.o[e] + tl.e[e] : tl.o[e] - 1, g.c[e]) : min(tl.o[e] + l[e], g.c[e] - 1);
  }
  return ok ? run_slot(g, np, c[0], c[1], c[2]) : -1;
}

// What both kinds of waves of run_tile know of the exchange.
struct RunExch {
  char* base;                      // the team's two scratch planes, one after the other
  int plane_bytes;
  int stride;                      // bytes between the word planes of a scratch plane
  uint32_t tag0;                   // tag of the input; step s: tag0 + s
  int par0;                        // scratch plane of the input
  int ne;                          // LDS entries per RHS subset
  __device__ __forceinline__ __amdgpu_buffer_rsrc_t plane(int s) const {
    return __builtin_amdgcn_make_buffer_rsrc(base + (int64_t)((par0 + s) & 1) * plane_bytes, 0, plane_bytes, 0x00027000);
  }
};

// The compute waves: np threads per RHS subset, one site each; the RHS of a subset take turns.
// FP32 arithmetic keeps both two-links of every direction in registers; FP64 keeps the
// backward ones in LDS (27 planes of np 16-byte words, shared by the subsets).  Inside the
// step loop these waves wait for LDS and the barrier only: loads in their own instruction
// stream would make every wait for a halo word wait for their stores as well.
template <int P, int R, bool CUT>
__device__ __forceinline__ void run_compute(const RunArgs& a, const RunUnit& g, const RunExch& x, int tile,
                                            const uint8_t* xcc, bool full, unsigned char* lds,
                                            typename Fmt<P>::real alpha, typename Fmt<P>::real beta) {
  using real = typename Fmt<P>::real;
  using X = Exch<P>;
  constexpr bool kLdsW = P == F64;
  constexpr int REC = run_record(P, R);
  const int np = a.np;
  const int sub = uniform((int)threadIdx.x / np), i = (int)threadIdx.x - sub * np;
  const RunTile tl = run_tile(g, tile);
  const RunFaces fc = run_faces(g, np);
  const int bx = g.b[0], by = g.b[1], bz = g.b[2];
  const bool in = i < bx * by * bz;
  const int i0 = in ? i : 0;
  const int lx = i0 % bx, lyz = i0 / bx, ly = lyz % by, lz = lyz / by;
  const bool active = in && lx < tl.e[0] && ly < tl.e[1] && lz < tl.e[2];
  // threads without a site compute the tile's first one and publish and store nothing
  const int ax = active ? lx : 0, ay = active ? ly : 0, az = active ? lz : 0;
  const int cx = tl.o[0] + ax, cy = tl.o[1] + ay, cz = tl.o[2] + az;
  const int site = run_site(g, a.hop, cx, cy, cz);
  const int64_t Vp = g.Vp;
  unsigned char* const wl = lds + (int64_t)a.subs * x.ne * REC;
  unsigned char* const vl = lds + (int64_t)sub * x.ne * REC;
  int nb[6];   // LDS offset of the neighbour x+, x-, y+, y-, z+, z- (own entries: those of even steps)
  {
    const int l[3] = {ax, ay, az}, st[3] = {1, bx, bx * by};
    const int face[3] = {az * by + ay, az * bx + ax, ay * bx + ax};
    const int me = (az * by + ay) * bx + ax;
#pragma unroll
    for (int d = 0; d < 3; d++) {
      nb[2 * d] = l[d] + 1 < tl.e[d] ? me + st[d] : fc.f[d] ? fc.hb[d] + fc.f[d] + face[d] : me - l[d] * st[d];
      nb[2 * d + 1] = l[d] > 0 ? me - st[d] : fc.f[d] ? fc.hb[d] + face[d] : me + (tl.e[d] - 1) * st[d];
    }
  }
  // readers of this site's words: tiles on this XCD see a plain store through their common L2
  // (loads of the words bypass the per-CU caches), tiles on another one need a device-scope store
  bool pub = false, far = false;
  if constexpr (CUT) {
    const int it[3] = {tile % g.t[0], tile / g.t[0] % g.t[1], tile / g.t[0] / g.t[1]};
    const int ts[3] = {1, g.t[0], g.t[0] * g.t[1]};
#pragma unroll
    for (int d = 0; d < 6; d++) {
      const int e = d / 2, n = ring(it[e] + (d % 2 ? -1 : 1), g.t[e]);
      const bool away = !full || (fc.f[e] > 0 && xcc[tile + (n - it[e]) * ts[e]] != xcc[tile]);
      if (nb[d] >= 2 * np) {
        pub = true;
        far = far || away;
      }
    }
    // One kind of store per 128-byte cache line (eight slots): a line that holds both written-through
    // and held-back words costs a probe of its owner's L2 for every reader on another XCD (one-link
    // 45x26x38 FP32 24 RHS: 40.8 us per step with mixed lines, 16.5 without).
    const uint64_t away = __ballot(far && active);
    far = pub && active && ((away >> ((int)__lane_id() & ~7)) & 0xff) != 0;
    pub = pub && active && !far;
  }
#pragma unroll
  for (int d = 0; d < 6; d++) nb[d] *= REC;
  real wf[3][18], wb[kLdsW ? 1 : 3][18];
#pragma unroll
  for (int mu = 0; mu < 3; mu++) {
    const char* W = g.W + mu * g.w_mu_stride;
    const int bs = run_site(g, a.hop, ring(cx - (mu == 0), g.c[0]), ring(cy - (mu == 1), g.c[1]), ring(cz - (mu == 2), g.c[2]));
    run_load_w<P>(a.w12, W, Vp, site, wf[mu]);
    if constexpr (kLdsW) {
      if (sub == 0) {
        real m[18];
        run_load_w<P>(a.w12, W, Vp, bs, m);
#pragma unroll
        for (int c = 0; c < 9; c++) reinterpret_cast<v2d*>(wl)[(9 * mu + c) * np + i] = v2d{m[2 * c], m[2 * c + 1]};
      }
    } else {
      run_load_w<P>(a.w12, W, Vp, bs, wb[mu]);
    }
  }
  const int mine = sub * R * X::NW * x.stride + (tile * np + i) * 16;
  auto publish = [&](int r, int s, const uint32_t (&d)[X::ND]) {
    const __amdgpu_buffer_rsrc_t rs = x.plane(s);
    if (pub) {
#pragma unroll
      for (int q = 0; q < X::NW; q++)
        exch_store<0>(exch_word<P>(d, q, x.tag0 + (uint32_t)s), rs, mine + (r * X::NW + q) * x.stride);
    }
    if (far) {
#pragma unroll
      for (int q = 0; q < X::NW; q++)
        exch_store<kDeviceScope>(exch_word<P>(d, q, x.tag0 + (uint32_t)s), rs, mine + (r * X::NW + q) * x.stride);
    }
  };
#pragma unroll
  for (int r = 0; r < R; r++) {
    uint32_t d[X::ND];
    X::load(a.in + g.psi_off + (int64_t)min(sub * R + r, g.nr - 1) * g.rhs_stride, Vp, site, d);
    if constexpr (CUT) publish(r, 0, d);
    real v[6];
    X::decode(d, v);
    rec_put<R>(vl + i * REC, r, v);
  }
  __builtin_amdgcn_s_waitcnt(0);   // the two-links have arrived: no wait for them in the loop
  for (int s = 0; s < a.n_steps; s++) {
    const int own = (s & 1) ? np * REC : 0;
    const int hal = R == 1 && (s & 1) ? a.halo * REC : 0;
    const bool last = s + 1 == a.n_steps;
#pragma unroll
    for (int r = 0; r < R; r++) {
      lds_barrier();
      real acc[6];
#pragma unroll
      for (int c = 0; c < 6; c++) acc[c] = (real)0;
#pragma unroll
      for (int mu = 0; mu < 3; mu++) {
        const unsigned char* const ef = vl + nb[2 * mu] + (nb[2 * mu] < np * REC ? own : hal);
        const unsigned char* const eb = vl + nb[2 * mu + 1] + (nb[2 * mu + 1] < np * REC ? own : hal);
        real u[6];
        rec_get<R>(ef, r, u);
        mv_acc(wf[mu], u, acc);
        rec_get<R>(eb, r, u);
        if constexpr (kLdsW) {
          real m[18];
#pragma unroll
          for (int c = 0; c < 9; c++) {
            const v2d w = reinterpret_cast<const v2d*>(wl)[(9 * mu + c) * np + i];
            m[2 * c] = w.x;
            m[2 * c + 1] = w.y;
          }
          mdv_acc(m, u, acc);
        } else {
          mdv_acc(wb[mu], u, acc);
        }
      }
      real o[6], w[6];
      rec_get<R>(vl + own + i * REC, r, w);
#pragma unroll
      for (int c = 0; c < 6; c++) o[c] = fma_(beta, acc[c], alpha * w[c]);
      if (!last) {
        uint32_t d[X::ND];
        X::encode(o, d);
        if constexpr (CUT) {
          publish(r, s + 1, d);
          if constexpr (R == 1) __builtin_amdgcn_s_barrier();   // the fetch waves start here (see run_fetch)
        }
        X::decode(d, w);
        rec_put<R>(vl + (np * REC - own) + i * REC, r, w);
      } else if (active && sub * R + r < g.nr) {
        Fmt<P>::template store_v<real, false>(a.out + g.psi_off + (int64_t)(sub * R + r) * g.rhs_stride, Vp, site, o);
      }
    }
  }
}

// The fetch waves: they collect the halo of each phase, E entries a thread, and write it to LDS
// before the barrier that opens the phase.  A phase's words were published R - 1 phases ago (by
// the phase before, where a thread has one RHS), so with several RHS per thread the store's and
// the load's latency run behind arithmetic.  (Requesting them a phase earlier still finds most
// of them not published yet and asks again: 70 instead of 60 us per step at 64^3 FP32 24 RHS.)
template <int P, int R, int E>
__device__ __forceinline__ bool run_fetch(const RunArgs& a, const RunUnit& g, const RunExch& x, int tile,
                                          unsigned char* lds) {
  using real = typename Fmt<P>::real;
  using X = Exch<P>;
  constexpr int REC = run_record(P, R);
  const int np = a.np;
  const int lane = (int)threadIdx.x - np * a.subs, lanes = (int)blockDim.x - np * a.subs;
  const RunTile tl = run_tile(g, tile);
  const RunFaces fc = run_faces(g, np);
  int src[E];            // byte offset of the first word; outside the plane (read as zeros) without an entry
  bool has[E];
  unsigned char* dst[E];
#pragma unroll
  for (int k = 0; k < E; k++) {
    const int e = lane + k * lanes;
    const int sub = e / a.halo, h = e - sub * a.halo;
    const int slot = sub < a.subs ? halo_slot(g, tl, fc, np, h) : -1;
    has[k] = slot >= 0;
    src[k] = has[k] ? sub * R * X::NW * x.stride + slot * 16 : x.plane_bytes;
    dst[k] = lds + ((int64_t)(sub < a.subs ? sub : 0) * x.ne + 2 * np + h) * REC;
  }
  bool dead = false;
  // loads of phase (s, r); unconditional, so that the number of loads in flight is known
  auto load = [&](int k, int s, int r, v4u(&w)[X::NW]) {
    const __amdgpu_buffer_rsrc_t rs = x.plane(s);
#pragma unroll
    for (int q = 0; q < X::NW; q++)
      w[q] = __builtin_amdgcn_raw_buffer_load_b128(rs, src[k], (r * X::NW + q) * x.stride, kDeviceScope);
  };
  auto take = [&](int s, int r, v4u(&hw)[E][X::NW]) {
    const uint32_t tag = x.tag0 + (uint32_t)s;
#pragma unroll
    for (int k = 0; k < E; k++) {
      int spin = 0;
      while (true) {
        bool ok = true;
#pragma unroll
        for (int q = 0; q < X::NW; q++) ok = ok && hw[k][q].w == tag;
        if (ok || !has[k] || dead) break;
        if (++spin > a.spins) {
          run_failed(a.fail);
          dead = true;
        }
        asm volatile("" ::: "memory");
        load(k, s, r, hw[k]);
      }
      uint32_t d[X::ND];
      exch_dwords<P>(hw[k], d);
      real u[6];
      X::decode(d, u);
      if (has[k]) rec_put<R>(dst[k] + (R == 1 && (s & 1) ? a.halo * REC : 0), r, u);
    }
  };
  __builtin_amdgcn_s_setprio(3);   // few instructions, on which every wave of the workgroup waits
  for (int s = 0; s < a.n_steps; s++) {
#pragma unroll
    for (int r = 0; r < R; r++) {
      // One RHS per thread: its words are published when the neighbours' phase ends, about when
      // this workgroup's does; polling from the phase's start would only load the caches.
      if (R == 1 && s > 0) __builtin_amdgcn_s_barrier();
      v4u hw[E][X::NW];
#pragma unroll
      for (int k = 0; k < E; k++) load(k, s, r, hw[k]);
      take(s, r, hw);
      lds_barrier();
    }
  }
  __builtin_amdgcn_s_setprio(0);
  return dead;
}

// One unit, one tile per workgroup: `tile` of this workgroup.  True in a thread that gave up a wait.
template <int P, int R, bool CUT>
__device__ __forceinline__ bool run_tile_steps(const RunArgs& a, const RunUnit& g, int tile, uint32_t tag0, int par0,
                                               int team, const uint8_t* xcc, bool full, unsigned char* lds,
                                               typename Fmt<P>::real alpha, typename Fmt<P>::real beta) {
  RunExch x;
  x.stride = a.team_size * a.np * 16;
  const int64_t plane = (int64_t)a.subs * R * Exch<P>::NW * x.stride;
  x.base = a.scratch + team * 2 * plane + (int64_t)g.first * a.np * 16;   // the unit's own slots
  x.plane_bytes = (int)plane;
  x.tag0 = tag0;
  x.par0 = par0;
  x.ne = 2 * a.np + (R == 1 ? 2 : 1) * a.halo;
  if (CUT && uniform((int)threadIdx.x) >= a.np * a.subs) {
    const int lanes = (int)blockDim.x - a.np * a.subs, entries = a.subs * a.halo;
    if (entries <= lanes) return run_fetch<P, R, 1>(a, g, x, tile, lds);
    if (entries <= 2 * lanes) return run_fetch<P, R, 2>(a, g, x, tile, lds);
    return run_fetch<P, R, kFetch>(a, g, x, tile, lds);
  }
  run_compute<P, R, CUT>(a, g, x, tile, xcc + g.first, full, lds, alpha, beta);
  return false;
}

// The result of a tile whose halo did not come: NaNs at its first site, so that no one takes the
// field for valid (a launch that goes on from it spreads them).
template <int P>
__device__ __forceinline__ void run_poison(const RunArgs& a, const RunUnit& g, int tile) {
  using real = typename Fmt<P>::real;
  const RunTile tl = run_tile(g, tile);
  real v[6];
  for (int c = 0; c < 6; c++) v[c] = (real)__builtin_nanf("");
  for (int r = 0; r < g.nr; r++)
    Fmt<P>::template store_v<real, false>(a.out + g.psi_off + (int64_t)r * g.rhs_stride, g.Vp,
                                          run_site(g, a.hop, tl.o[0], tl.o[1], tl.o[2]), v);
}

template <int P, int R, bool CUT>
__global__ __launch_bounds__(run_max_threads(P)) void smear_run(RunArgs a, typename Fmt<P>::real alpha, typename Fmt<P>::real beta) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  // messages between the workgroup's threads, the XCD of each member of the team, then the vectors
  uint32_t* const sh = reinterpret_cast<uint32_t*>(lds_raw);
  uint8_t* const xcc = lds_raw + 16;
  unsigned char* const lds = lds_raw + kRunMsgBytes;
  const RunPlace pl = run_place(a.team_size);
  RunTeam* const tm = a.ctl->team + pl.team;
  if (threadIdx.x == 0) {
    uint32_t e = 1u << 20, size = 0;
    if (pl.rank < pl.expect) {
      if constexpr (CUT) {
        ctl_store(a.ctl->xcc + pl.team * a.team_size + pl.rank, xcd_id());
        __builtin_amdgcn_s_waitcnt(0);   // there before this workgroup counts as enrolled
      }
      e = ctl_add(&tm->enrolled, 1u);
      if (e == 0) {
        for (int k = 0; k < a.patience && ctl_load(&tm->enrolled) < (uint32_t)pl.expect; k++) __builtin_amdgcn_s_sleep(2);
        size = __hip_atomic_fetch_or(&tm->enrolled, kTeamClosed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (size == (uint32_t)pl.expect) ctl_add(&a.ctl->full, 1u);
        else if (ctl_load(&a.ctl->full) * kAwayShares >= (uint32_t)a.n_shares) size = kTeamAway;
        ctl_store(&tm->size, size);
      } else if (e < kTeamClosed) {
        for (int k = 0; k < kSpinLimit && (size = ctl_load(&tm->size)) == 0; k++) __builtin_amdgcn_s_sleep(1);
        if (size == 0) run_failed(a.fail);
      }
    }
    if (size == kTeamAway) size = 0;
    sh[0] = size;
    sh[1] = size == (uint32_t)pl.expect ? (uint32_t)pl.rank : e;   // a full team's members take their places' tiles
    sh[2] = ctl_load(&a.ctl->epoch);
    sh[3] = e;
  }
  __syncthreads();
  const int size = uniform((int)sh[0]), me = uniform((int)sh[1]);
  const uint32_t epoch = (uint32_t)uniform((int)sh[2]);
  const bool leader = uniform((int)sh[3]) == 0;
  const bool full = size == pl.expect;
  if (CUT && full && me < size)
    for (int k = (int)threadIdx.x; k < size; k += (int)blockDim.x)
      xcc[k] = (uint8_t)ctl_load(a.ctl->xcc + pl.team * a.team_size + k);
  __syncthreads();
  if (me < size) {
    uint32_t barriers = 0, seq = 0;   // team barriers passed, rounds begun (a round: the units that run at once)
    // Every member has finished what came before: needed before scratch slots change their readers.
    auto team_barrier = [&] {
      barriers++;
      if (size > 1 && threadIdx.x == 0) {
        __builtin_amdgcn_s_waitcnt(0);
        ctl_add(&tm->arrived, 1u);
        int k = 0;
        while (ctl_load(&tm->arrived) < barriers * (uint32_t)size && ++k < kSpinLimit) {}
        if (k >= kSpinLimit) run_failed(a.fail);
      }
      __syncthreads();
    };
    int shape = -1;   // of the unit before, -1: a barrier has to come first
    // A team takes shares of the units (every n_shares-th one) until none is left.
    for (uint32_t take = 1;; take++) {
      if (threadIdx.x == 0) {
        uint32_t u = (uint32_t)a.n_shares;
        if (leader) {
          u = min(ctl_add(&a.ctl->next_share, 1u), (uint32_t)a.n_shares);
          if (size > 1) __hip_atomic_store(&tm->mail, (uint64_t)take << 32 | u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else {
          uint64_t m = 0;
          int k = 0;
          while (((m = __hip_atomic_load(&tm->mail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >> 32) != take &&
                 ++k < kSpinLimit) {}
          if (k >= kSpinLimit) run_failed(a.fail);
          else u = (uint32_t)m;
        }
        sh[0] = u;
      }
      __syncthreads();
      const int share = uniform((int)sh[0]);
      __syncthreads();
      if (share >= a.n_shares) break;
      for (int u = share; u < a.n_units; u += a.n_shares) {
        const RunUnit& g = a.units[u];
        const int tile = me - g.first;
        const bool fast = size >= g.span;
        // The units of a round have members, scratch slots and tags of their own place in the team,
        // so they share the round's tags; a team too small for the round runs them one by one.
        if (g.first == 0 || !fast) seq++;
        // Units of one shape follow each other without a barrier: a workgroup that starts the next
        // one overwrites words of step n - 2, which its readers have read before they published the
        // step n - 1 it has read; and words of step n - 1 once those readers have published the
        // next unit's input.
        if (seq > 1 && (!fast || g.shape != shape)) team_barrier();
        shape = fast ? g.shape : -1;
        const uint32_t pubs = (seq - 1) * (uint32_t)a.n_steps;
        bool gave_up = false;
        if (fast) {
          if (tile >= 0 && tile < g.t[0] * g.t[1] * g.t[2])
            gave_up = run_tile_steps<P, R, CUT>(a, g, tile, epoch + 1u + pubs, (int)(pubs & 1), pl.team, xcc, full, lds, alpha, beta);
        } else if constexpr (CUT) {
          if ((int)threadIdx.x < a.np * a.subs)
            run_slow<P, R>(a, g, me, size, epoch + 1u + pubs, (int)(pubs & 1), pl.team, alpha, beta);
        }
        __syncthreads();   // LDS is free for the next unit
        if (CUT && gave_up) run_poison<P>(a, g, tile);
      }
      shape = -1;
      team_barrier();
    }
  }
  // the launch's last workgroup leaves the control block ready for the next launch
  if (threadIdx.x == 0) {
    __builtin_amdgcn_s_waitcnt(0);
    sh[0] = ctl_add(&a.ctl->finished, 1u) == gridDim.x - 1;
  }
  __syncthreads();
  if (!sh[0]) return;
  for (int k = (int)threadIdx.x; k < a.n_teams; k += (int)blockDim.x) {
    RunTeam* const t = a.ctl->team + k;
    ctl_store(&t->enrolled, 0);
    ctl_store(&t->size, 0);
    ctl_store(&t->arrived, 0);
    __hip_atomic_store(&t->mail, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x == 0) {
    ctl_store(&a.ctl->next_share, 0);
    ctl_store(&a.ctl->full, 0);
    ctl_store(&a.ctl->finished, 0);
    ctl_store(&a.ctl->epoch, epoch + (uint32_t)a.n_units * (uint32_t)a.n_steps + 1u);
  }
}

template <int P, int R>
hipError_t launch_run_k(const RunConfig& c, const RunArgs& a, double alpha, double beta, hipStream_t s) {
  using real = typename Fmt<P>::real;
  const real al = (real)alpha, be = (real)beta;
  const int threads = a.np * a.subs + 64 * c.fetch;
  if (c.fetch == 0) smear_run<P, R, false><<<c.grid, threads, (size_t)c.lds, s>>>(a, al, be);
  else smear_run<P, R, true><<<c.grid, threads, (size_t)c.lds, s>>>(a, al, be);
  return hipGetLastError();
}

template <int P>
hipError_t launch_run_p(const RunConfig& c, const RunArgs& a, double alpha, double beta, hipStream_t s) {
  if (a.np < 64 || a.np % 64 || a.np * a.subs + 64 * c.fetch > run_max_threads(P) || c.lds > kMaxLds || c.grid % kXcds ||
      (c.fetch > 0) != (a.halo > 0) || a.subs * a.halo > 64 * c.fetch * kFetch)
    return hipErrorInvalidValue;
  switch (c.width) {
    case 1: return launch_run_k<P, 1>(c, a, alpha, beta, s);
    case 2: return launch_run_k<P, 2>(c, a, alpha, beta, s);
    case 3: return launch_run_k<P, 3>(c, a, alpha, beta, s);
    case 4: return launch_run_k<P, 4>(c, a, alpha, beta, s);
    default: return hipErrorInvalidValue;
  }
}

template <int P, int R>
hipError_t run_allow_lds() {
  for (const void* f : {reinterpret_cast<const void*>(&smear_run<P, R, false>),
                        reinterpret_cast<const void*>(&smear_run<P, R, true>)}) {
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxLds);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <int P>
hipError_t run_attributes() {
  hipError_t e = hipSuccess;
  for (hipError_t r : {run_allow_lds<P, 1>(), run_allow_lds<P, 2>(), run_allow_lds<P, 3>(), run_allow_lds<P, 4>()})
    if (r != hipSuccess) e = r;
  return e;
}

}  // namespace

}  // namespace tl
