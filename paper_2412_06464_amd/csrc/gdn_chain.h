// Sequential inter-chunk state passes in bf16 (gfx950) of the chunkwise gated
// delta rule (Sec. 3.3; state stored dk x dv).  Every wave is a chain of its
// own: it holds all dk rows of the state (or of its gradient) over 16 NC
// columns of dv in MFMA accumulators and walks a sequence's chunks in order.
// The accumulator tiles, rounded to bf16, are directly the operands of the
// next product (no exchange between waves), so a chunk costs one barrier:
// the one that hands over the chunk's k and q rows, which the waves of a
// workgroup share through LDS.
//
// With T = (I + A)^-1 and P from the prep kernel, b = beta, g the cumulative
// log gate of the chunk:
//   forward   R = V - diag(e^g) (K S),  V' = (T diag(b)) R,
//             O = diag(e^g) (Q S) + P V',
//             S <- e^{g_n} S + K^T (diag(e^{g_n - g}) V')
//   backward  (reverse order; dS = gradient of the chunk's exit state)
//             dV' = P^T dO + diag(e^{g_n - g}) (K dS),  dX = T^T dV',
//             dv = b dX,
//             dS <- e^{g_n} dS + Q^T (diag(e^g) dO) - K^T (diag(b e^g) dX)
// These are the UT transform's equations with W~ = T diag(b e^g) K and
// U~ = T diag(b) V multiplied out: the passes read q, k, v (or dO) and two
// 64 x 64 matrices per chunk and head, and W~, U~, Kbar^T, (e^g Q)^T never
// exist in memory.
//
// Layouts.  k and q rows lie in LDS row-major with 16-byte units permuted
// inside a row (unit u of row t at u ^ sw(t)), so that both reads are free of
// bank conflicts: the row operands (A of K S: lane = row, 8 consecutive d,
// ds_read_b128, 256 B/cycle measured) and the transposed ones (A of K^T V':
// lane = d, 4 rows per ds_read_b64_tr_b16, 128 B/cycle).  State tile 2 kt + p
// holds in accumulator row 4 g + e the state row d = 32 kt + 8 g + 4 p + e, so
// that a lane's eight rows of a k-step are the eight consecutive d of the row
// operands; with NC = 2, column c of tile j is 8 (c >> 2) + 4 j + (c & 3) of
// the wave's 32, so that a transposed product leaves eight consecutive columns
// in a lane, one 16-byte store.  Contractions over t use the order of
// kperm<bf16>, as the prep kernel stores T and P.  The state, V' and dS go out
// transposed by a product with a 0/1 matrix, which needs no LDS and is exact
// where they are finite.  Where one is not, 0 Inf = NaN reaches the other 31
// rows of its own column in the stored copy, which only the gradient kernel
// reads; that column's V' (or dX) is then not finite in any row of the chunk
// either, since K S contracts over the state's rows, and with it none of the
// gradients that the copy enters.  v and dO, whose columns stay apart through
// the whole recurrence, are turned by transposed LDS reads instead, which
// move values and keep a non-finite one in its column.
#pragma once
#include "gdn_device.h"
#include "gdn_kernels.h"
#include "gdn_seq_common.h"

namespace gdn {

namespace {

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) u32x4 lds_u32x4;
using M = Mfma<bf16>;
using frag = bf16x8;

// XOR of a row's 16-byte units (of U units): the three low bits of the row
// reversed into the three high bits of a 16-unit index.
__device__ inline unsigned row_swizzle(unsigned t, unsigned U) {
  return ((t & 1) << 3 | (t & 2) << 1 | (t & 4) >> 1) & (U - 1);
}

__device__ inline frag pack8(f32x4 a, f32x4 b) {
  return frag{(bf16)a[0], (bf16)a[1], (bf16)a[2], (bf16)a[3],
              (bf16)b[0], (bf16)b[1], (bf16)b[2], (bf16)b[3]};
}

// Keeps the products that form x where they stand: they have no side effects,
// and the compiler would otherwise collect them (and with them the operands
// they read) at the end of the chunk.
template <int N>
__device__ inline void pin(f32x4 (&x)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(x[i]));
}

// Nothing is scheduled across this point.
__device__ inline void phase() { __builtin_amdgcn_sched_barrier(0); }

// A store of data that this kernel does not read back.  Non-temporal at
// dk = 256 (the chunk states are several times the last-level cache: stored
// plainly, the saving forward took 437 us instead of 453, but the gradient
// kernel behind it 610 instead of 565); plain at dk <= 128 (65,536 packed
// tokens, 16 heads, 128/128: saving forward 649 -> 625 us, reverse pass
// 716 -> 675, gradient kernel the same).
template <bool STREAM, class T>
__device__ inline void put_out(void* p, const T& v) {
  if constexpr (STREAM) store_stream_small(p, v);
  else *reinterpret_cast<T*>(p) = v;
}

__device__ inline frag select8(int lane_k0, int target) {
  frag f;
#pragma unroll
  for (int j = 0; j < 8; ++j) f[j] = (bf16)(lane_k0 + j == target ? 1.f : 0.f);
  return f;
}

// A uniform base and a 32-bit lane offset in bytes (a chunk's rows span less
// than 4 GiB: at most 65,535 heads fit the prep kernel's grid).
template <class T>
__device__ inline T ld(const void* base, unsigned off) {
  return *reinterpret_cast<const T*>((const char*)base + off);
}

// The shared k / q rows of a workgroup: NT tiles of 64 rows x DK, two buffers.
template <int DK, int NT, int NTH>
struct Rows {
  static constexpr int U = DK / 8;         // 16-byte units per row
  static constexpr int RB = DK * 2;        // bytes per row
  static constexpr int TILE = CH * RB;     // bytes of a tile
  static constexpr int BUF = NT * TILE;    // bytes of a buffer
  static constexpr int PER = CH * U / NTH; // 16-byte loads per lane and tile
  static_assert(CH * U % NTH == 0, "rows do not divide over the threads");
  static constexpr int RSTEP = NTH / U;    // rows between a lane's loads
  u32x4 r[NT][PER];

  // pieces X0 .. X1 - 1 of a chunk's rows (src: its first row and head, row
  // stride rs bytes), clamped to its last row
  template <int X0, int X1>
  __device__ inline void load(const bf16* const (&src)[NT], unsigned rs, int len, int tid) {
    const unsigned u = (unsigned)tid % U * 16, lim = (len - 1) * rs + u;
#pragma unroll
    for (int x = X0; x < X1; ++x) {
      const unsigned off = min((unsigned)tid / U * rs + u + x * RSTEP * rs, lim);
#pragma unroll
      for (int m = 0; m < NT; ++m) r[m][x] = ld<u32x4>(src[m], off);
    }
  }
  // this lane's addresses in the buffer at LDS byte address buf: its rows are
  // RSTEP apart, and the permutation of a row's units repeats every 8 rows
  static constexpr int NAT = RSTEP < 8 ? 8 / RSTEP : 1;
  struct At {
    unsigned a[NAT];
    __device__ inline At(unsigned buf, int tid) {
#pragma unroll
      for (int x = 0; x < NAT; ++x) {
        const unsigned t = (unsigned)tid / U + x * RSTEP, u = (unsigned)tid % U;
        a[x] = buf + t * RB + (u ^ row_swizzle(t, U)) * 16;
      }
    }
    __device__ inline void move(int by) {
#pragma unroll
      for (int x = 0; x < NAT; ++x) a[x] += by;
    }
    __device__ inline unsigned of(int x) const { return a[x % NAT] + x / NAT * (NAT * RSTEP * RB); }
  };
  // the pieces into the buffer of lane addresses at
  template <int X0, int X1>
  __device__ inline void store(const At& at) const {
#pragma unroll
    for (int x = X0; x < X1; ++x)
#pragma unroll
      for (int m = 0; m < NT; ++m) *(lds_u32x4*)(uintptr_t)(at.of(x) + m * TILE) = r[m][x];
  }
  // zeros in place of the rows past the chunk's end (after store, by the
  // same lanes)
  static __device__ inline void zero_tail(const At& at, int len, int tid) {
    if (len < CH) {
#pragma unroll
      for (int x = 0; x < PER; ++x)
        if (tid / U + x * RSTEP >= len) {
#pragma unroll
          for (int m = 0; m < NT; ++m)
            *(lds_u32x4*)(uintptr_t)(at.of(x) + m * TILE) = u32x4{0u, 0u, 0u, 0u};
        }
    }
  }
};

// Operand reads from the tiles of the current buffer.  The lane addresses
// are carried from chunk to chunk (moved to the other buffer by a step of one
// buffer) and every read is one of them plus a constant that fits the
// instruction; formed from the buffer's address in each chunk, the compiler
// keeps one register per read.
template <int DK>
struct RowOps {
  static constexpr int U = DK / 8, RB = DK * 2, NKD = DK / 32;
  unsigned row[NKD], col[NKD];
  __device__ inline RowOps(unsigned buf) {
    const unsigned l = lane_id(), g = l >> 4, t = l & 15, r = (l >> 2) & 3, q = l & 3;
    const unsigned sr = row_swizzle(t, U), sc = row_swizzle(4 * (g & 1) + r, U);
#pragma unroll
    for (int k = 0; k < NKD; ++k) {
      row[k] = buf + t * RB + ((4 * k + g) ^ sr) * 16;
      col[k] = buf + (4 * g + r) * RB + ((4 * k + q) ^ sc) * 16;
    }
  }
  __device__ inline void move(int by) {
#pragma unroll
    for (int k = 0; k < NKD; ++k) {
      row[k] += by;
      col[k] += by;
    }
  }
  // A (or B) operand: rows 16 i + (l & 15) of the tile, k-step kt over d
  template <int TILE>
  __device__ inline frag rows(int i, int kt) const {
    return __builtin_bit_cast(frag, *(const lds_u32x4*)(uintptr_t)(row[kt] + (TILE + i * 16 * RB)));
  }
  // A operand of the transpose: state tile i (rows d), k-step kt over t
  template <int TILE>
  __device__ inline frag cols(int i, int kt) const {
    constexpr int HALF = 16 * RB;
    const int o = TILE + 8 * (i & 1) + 32 * kt * RB;
    const s16x4 lo =
        __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(col[i >> 1] + o));
    const s16x4 hi =
        __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(col[i >> 1] + (o + HALF)));
    return __builtin_bit_cast(frag, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// The six nonzero 16 x 32 operand tiles of a lower- (LOW) or upper-triangular
// 64 x 64 matrix in A-buffer order: tile (i, kt) of row block i, k-step kt.
constexpr bool tri_has(bool low, int i, int kt) { return low ? kt <= (i >> 1) : kt >= (i >> 1); }
constexpr int tri_slot(bool low, int i, int kt) {
  int n = 0;
  for (int x = 0; x < i; ++x)
    for (int y = 0; y < 2; ++y) n += tri_has(low, x, y);
  for (int y = 0; y < kt; ++y) n += tri_has(low, i, y);
  return n;
}

// Two triangular matrices of a chunk, shared by the waves of a workgroup
// through LDS (two buffers): a wave loads every NW-th of their tiles.  Loaded
// by every wave instead, they were a third of the bytes on the path from L2.
template <bool LOW, int NM, int NW>
struct Tri {
  static constexpr int TILES = 6 * NM, BUF = TILES * 1024, PER = (TILES + NW - 1) / NW;
  u32x4 r[PER];
  __device__ inline void load(const bf16* m0, const bf16* m1, int w) {
#pragma unroll
    for (int x = 0; x < PER; ++x) {
      const int t = min(w + NW * x, TILES - 1), s = t < 6 ? t : t - 6;
      const int at = LOW ? (s < 2 ? 2 * s : s + 2) : (s < 4 ? s : 2 * s - 3);  // 2 i + kt
      r[x] = ld<u32x4>((t < 6 ? m0 : m1) + at * 512, lane_id() * 16u);
    }
  }
  // at: the buffer's address and 16 lane_id()
  __device__ inline void store(unsigned at, int w) const {
#pragma unroll
    for (int x = 0; x < PER; ++x)
      if (w + NW * x < TILES) *(lds_u32x4*)(uintptr_t)(at + (w + NW * x) * 1024) = r[x];
  }
  template <int MAT>
  static __device__ inline frag get(unsigned at, int i, int kt) {
    return __builtin_bit_cast(
        frag, *(const lds_u32x4*)(uintptr_t)(at + (6 * MAT + tri_slot(LOW, i, kt)) * 1024));
  }
};

// Columns of a wave: NC tiles of 16 from v0; see the head of the file.
template <int NC, bool STREAM = true>
struct Cols {
  static constexpr int W = 16 * NC;
  int v0;  // first column
  __device__ inline Cols(int first) : v0(first) {}
  __device__ static inline int at(int j) {  // column of this lane in tile j, from v0
    const int c = lane_id() & 15;
    return NC == 2 ? 8 * (c >> 2) + 4 * j + (c & 3) : c;
  }
  // Transposed tiles (rows = the wave's columns, columns = the rows of row
  // tile i) to rows of a row-major matrix (base: the chunk's first row and
  // head, stride rs bytes), through LDS (row_put, then row_out); or (frag_out)
  // to fragment order over dv (tile: the row tile's first fragment).
  template <class B>
  __device__ inline void row_put(const f32x4 (&t)[NC], const B& b) const {
    if constexpr (NC == 2) {
      B::put(b.op, __builtin_bit_cast(typename B::vec, pack8(t[0], t[1])));
    } else {
      const bf16x4 x = {(bf16)t[0][0], (bf16)t[0][1], (bf16)t[0][2], (bf16)t[0][3]};
      B::put(b.op, __builtin_bit_cast(typename B::vec, x));
    }
  }
  template <class B>
  __device__ inline void row_out(bf16* base, unsigned rs, int i, int len, const B& b) const {
    const typename B::vec x = B::get(b.mem);
    const int l = lane_id(), r = 16 * i + (l >> 2);
    if (r < len) put_out<STREAM>((char*)(base + v0) + (r * rs + (l & 3) * (8u * NC)), x);
  }
  __device__ inline void frag_out(bf16* tile, const f32x4 (&t)[NC]) const {
    const int l = lane_id(), g = l >> 4;
    bf16* f = tile + (size_t)(v0 >> 5) * 512;
    if constexpr (NC == 2) {
      put_out<STREAM>((char*)f + l * 16u, pack8(t[0], t[1]));
    } else {
      const bf16x4 x = {(bf16)t[0][0], (bf16)t[0][1], (bf16)t[0][2], (bf16)t[0][3]};
      f += ((v0 >> 4) & 1) * 256;
      put_out<STREAM>((char*)f + ((l & 15) * 16u + (g >> 1) * 256u + (g & 1) * 8u), x);
    }
  }
};

// One 16-row tile of a wave's columns, 64 lanes of 8 NC bytes, passed through
// LDS between memory order (lane 4 r + p holds piece p of row r: four lanes
// cover a row's 32 NC bytes, which the memory path takes as one access) and
// the lane orders of the products: operand order (lane 16 p + r) for the rows
// that go out, and accumulator tiles (transposed reads) for those that come
// in.  In operand order straight from or to memory every lane of a quad is
// another row, four times the accesses: with v and O so, a chunk at dk = 128
// took 9.2k cycles and 6.6k / 6.9k without the loads of v / the stores of O.
// The unit of (r, p) is permuted so that all sides are free of bank conflicts.
template <int NC>
struct Bounce {
  typedef unsigned vec __attribute__((ext_vector_type(2 * NC)));
  typedef __attribute__((address_space(3))) vec lds_vec;
  static constexpr int BYTES = 64 * 8 * NC;  // one tile
  unsigned mem, op;  // lane addresses
  __device__ inline Bounce(unsigned base) {
    const unsigned l = lane_id();
    mem = base + unit(l >> 2, l & 3) * (8 * NC);
    op = base + unit(l & 15, l >> 4) * (8 * NC);
  }
  __device__ static inline unsigned unit(unsigned r, unsigned p) {
    return 4 * r + (p ^ ((r >> 2) & 3));
  }
  __device__ static inline void put(unsigned at, vec v) { *(lds_vec*)(uintptr_t)at = v; }
  __device__ static inline vec get(unsigned at) { return *(const lds_vec*)(uintptr_t)at; }
  // rows 4 (l >> 4) .. + 3 of this lane's column in tile c: a lane points at
  // its piece of the 16 lanes' 4 rows, which in memory order is its own unit
  __device__ inline s16x4 column(int c) const {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(uintptr_t)(mem + 8 * c));
  }
};

// Rows of v or dO as accumulator tiles (tile i, rows t; tile c, the wave's
// columns), zero past the chunk's end.
template <int NC>
struct VRows {
  using B = Bounce<NC>;
  typename B::vec r[4];  // as loaded
  s16x4 t[4][NC];        // turned
  // x: the chunk's first row and head at the wave's first column
  __device__ inline void load(const bf16* x, unsigned rs, int len) {
    const unsigned l = lane_id(), u = (l & 3) * (8 * NC), lim = (len - 1) * rs + u;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      r[i] = ld<typename B::vec>(x, min((l >> 2) * rs + u + 16 * i * rs, lim));
  }
  __device__ inline void turn(const B& b, int len) {
    if (len < CH) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (16 * i + (lane_id() >> 2) >= len) r[i] = typename B::vec{};
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      B::put(b.mem, r[i]);
#pragma unroll
      for (int c = 0; c < NC; ++c) t[i][c] = b.column(c);
    }
  }
  __device__ inline f32x4 tile(int i, int c) const {
    f32x4 x;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = (float)__builtin_bit_cast(bf16, (short)t[i][c][e]);
    return x;
  }
  // row tiles 2 kt, 2 kt + 1 as an operand over t
  __device__ inline frag over_t(int kt, int c) const {
    return __builtin_bit_cast(
        frag, __builtin_shufflevector(t[2 * kt][c], t[2 * kt + 1][c], 0, 1, 2, 3, 4, 5, 6, 7));
  }
};

// The wave's columns of a dk x dv fp32 state in memory (base: row 0 at the
// wave's first column).  State row of tile i, element e:
// 32 (i >> 1) + 8 g + 4 (i & 1) + e.
template <int DV, int NC>
__device__ inline float* state_at(float* base, int i, int j, int e) {
  const unsigned off = ((lane_id() >> 4) * 8u * DV + Cols<NC>::at(j)) * 4u;
  return (float*)((char*)(base + (32 * (i >> 1) + 4 * (i & 1) + e) * DV) + off);
}
template <int DV, int MT, int NC>
__device__ inline void load_state(float* base, f32x4 (&S)[MT][NC]) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j) S[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  if (base) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NC; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) S[i][j][e] = *state_at<DV, NC>(base, i, j, e);
  }
}
template <int DV, int MT, int NC>
__device__ inline void store_state(float* base, const f32x4 (&S)[MT][NC]) {
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) *state_at<DV, NC>(base, i, j, e) = S[i][j][e];
}

}  // namespace

// Between phase() marks: operand reads one by one between the products,
// instead of in a block before them (an LDS read holds a wave's path to LDS
// for 16 cycles, as long as a product holds the matrix core).
template <int MFMA, int READS>
__device__ inline void interleave() {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, MFMA, 0);
    __builtin_amdgcn_sched_group_barrier(0x100, READS, 0);
  }
}

template <int I>
using int_c = std::integral_constant<int, I>;

// Order of the forward's row-operand groups: k of k-step kt, and q of k-step
// kt behind k of k-step kt + lag.
constexpr int group_pos(int kt, bool q, int nkd, int lag) {
  if (!q) return kt < lag ? kt : 2 * kt - lag;
  return kt < nkd - lag ? lag + 2 * kt + 1 : nkd + kt;
}
struct GroupAt {
  bool q;
  int kt;
};
constexpr GroupAt group_at(int pos, int nkd, int lag, bool has_q) {
  if (!has_q) return {false, pos};
  for (int kt = 0; kt < nkd; ++kt) {
    if (group_pos(kt, false, nkd, lag) == pos) return {false, kt};
    if (group_pos(kt, true, nkd, lag) == pos) return {true, kt};
  }
  return {false, 0};
}

// Waves per SIMD the registers are sized for: one where LDS holds one
// four-wave workgroup per CU (dk >= 128), else two.
template <int DK, int NW>
constexpr int chain_occ() { return DK >= 128 && NW == 4 ? 1 : 2; }

// ------------------------------------------------------------------ forward / recompute

template <int DK, int DV, int MODE, int NC, int NW>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * NW, 64 * NW),
                          amdgpu_waves_per_eu(chain_occ<DK, NW>(), chain_occ<DK, NW>())))
void k_fwd_chain(Args a) {
  constexpr bool OUT = MODE != SEQ_STORE, STORE = MODE != SEQ_FWD;
  constexpr int NTH = 64 * NW, BV = 16 * NC * NW, NKD = DK / 32, MT = DK / 16;
  constexpr bool AFTER = STORE && NC == 2;
  using R = Rows<DK, OUT ? 2 : 1, NTH>;
  __shared__ __align__(16) unsigned char sRows[2 * R::BUF];
  __shared__ __align__(16) float sGate[2][2][CH];  // by chunk parity: e^g, e^{g_n - g}
  __shared__ __align__(16) unsigned char sBounce[NW][Bounce<NC>::BYTES];
  __shared__ __align__(16) unsigned char sTri[2 * Tri<true, OUT ? 2 : 1, NW>::BUF];

  int unit, tile;
  if (!map_unit_tile(DV / BV, a.N * a.H, unit, tile)) return;
  const int n = unit / a.H, h = unit - n * a.H, H = a.H;
  const int tid = threadIdx.x, l = lane_id(), g = l >> 4;
  const int w = __builtin_amdgcn_readfirstlane(wave_id());
  const Cols<NC, DK == 256> cols(tile * BV + w * 16 * NC);
  const unsigned rows0 = (unsigned)(uintptr_t)sRows;
  const Bounce<NC> bounce((unsigned)(uintptr_t)sBounce[w]);
  RowOps<DK> ops(rows0);              // reads the chunk's buffer
  typename R::At put(rows0, tid);     // writes the next one's
  unsigned tri = (unsigned)(uintptr_t)sTri + l * 16;  // T and P of the chunk
  const int s0 = a.cu ? a.cu[n] : n * a.T;
  const int L = a.cu ? a.cu[n + 1] - s0 : a.T;
  const int c0 = seq_first_chunk(a, n), nch = (L + CH - 1) / CH;
  frag selD[2], selT[2];
  if constexpr (STORE) {
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      selD[p] = select8(8 * g, 16 * p + (l & 15));
#pragma unroll
      for (int j = 0; j < 8; ++j)
        selT[p][j] = (bf16)(kperm<bf16>(0, g, j) == 16 * p + (l & 15) ? 1.f : 0.f);
    }
  }

  f32x4 S[MT][NC];
  const size_t sbase = ((size_t)n * H + h) * DK * DV + cols.v0;
  load_state<DV>(a.h0 ? const_cast<float*>(a.h0) + sbase : nullptr, S);

  R rows;
  VRows<NC> vr;
  using TP = Tri<true, OUT ? 2 : 1, NW>;  // T diag(b), P
  TP tp;
  float gl = 0.f;
  auto load_rows = [&](int j, auto x0, auto x1) {
    constexpr int X0 = decltype(x0)::value, X1 = decltype(x1)::value;
    const size_t row0 = (size_t)(s0 + j * CH) * H + h;
    const int len = min(CH, L - j * CH);
    if constexpr (OUT)
      rows.template load<X0, X1>({(const bf16*)a.k + row0 * DK, (const bf16*)a.q + row0 * DK},
                                 H * DK * 2, len, tid);
    else
      rows.template load<X0, X1>({(const bf16*)a.k + row0 * DK}, H * DK * 2, len, tid);
  };
  auto load_v = [&](int j) {
    const size_t row0 = (size_t)(s0 + j * CH) * H + h;
    vr.load((const bf16*)a.v + row0 * DV + cols.v0, H * DV * 2, min(CH, L - j * CH));
  };
  auto chunk = [&](int j) { return (size_t)(c0 + j) * H + h; };
  auto load_tp = [&](int j) {
    const size_t at = chunk(j) * CH * CH;
    tp.load((const bf16*)a.Wf + at, (const bf16*)a.Pf + at, w);
  };
  auto load_g = [&](int j) { gl = ld<float>(a.g + chunk(j) * CH, l * 4u); };
  auto put_gates = [&](int j) {  // from gl, by one wave
    if (w == 0) {
      sGate[j & 1][0][l] = __expf(gl);
      sGate[j & 1][1][l] = __expf(__shfl(gl, CH - 1, 64) - gl);
    }
  };

  // the loads in the order of the loop, so that its waits (which have to hold
  // on entry too) stay partial
  if (nch > 0) {
    load_rows(0, int_c<0>{}, int_c<R::PER>{});
    load_tp(0);
    rows.template store<0, R::PER>(put);
    tp.store(tri, w);
    R::zero_tail(put, min(CH, L), tid);
    put.move(R::BUF);
    load_g(0);
    put_gates(0);
    load_rows(min(1, nch - 1), int_c<0>{}, int_c<R::PER>{});
    load_tp(min(1, nch - 1));
    load_g(min(1, nch - 1));
    load_v(0);
    lds_barrier();
  }
  int step = R::BUF, step_tri = TP::BUF;  // to the other buffer
  for (int j = 0; j < nch; ++j) {
    const int len = min(CH, L - j * CH), jn = min(j + 1, nch - 1);
    const size_t ch = chunk(j);
    const float(&gate)[2][CH] = sGate[j & 1];
    const float egn = gate[0][CH - 1];  // pads repeat g of the last token

    // Operands from LDS, in groups of four tiles read D - 1 groups ahead of
    // the products: the row operands of k for each k-step over d, those of q
    // LAG k-steps later (so that the last of (Q S)^T overlap R), then the
    // transposed ones of k, two state tiles at a time.
    constexpr int LAG = OUT ? (NC == 1 && NKD == 8 ? 1 : NKD / 2) : 0, NA = (OUT ? 2 : 1) * NKD, NC_ = MT / 2;
    constexpr int D = NC == 1 ? 3 : 2;
    frag f[D][4];
    auto fetch = [&](auto pc) {
      constexpr int P = decltype(pc)::value;
      if constexpr (P < NA) {
        constexpr GroupAt at = group_at(P, NKD, LAG, OUT);
#pragma unroll
        for (int i = 0; i < 4; ++i) f[P % D][i] = ops.template rows<at.q ? R::TILE : 0>(i, at.kt);
      } else if constexpr (P < NA + NC_) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
          f[P % D][i] = ops.template cols<0>(2 * (P - NA) + (i >> 1), i & 1);
      }
    };
    static_for<0, D - 1>(fetch);
    phase();

    f32x4 X[4][NC], O[4][NC];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < NC; ++c) X[i][c] = O[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The state rounded to bf16 (also the chunk's entry state, which goes
    // out transposed); the state decays in place.
    frag Sb[NKD][NC];
    auto round_state = [&](auto kc) {
      constexpr int kt = decltype(kc)::value;
      if constexpr (kt < NKD) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          Sb[kt][c] = pack8(S[2 * kt][c], S[2 * kt + 1][c]);
          S[2 * kt][c] *= egn;
          S[2 * kt + 1][c] *= egn;
        }
        pin(S[2 * kt]);
        pin(S[2 * kt + 1]);
      }
    };
    auto store_state_step = [&](auto kc) {
      constexpr int kt = decltype(kc)::value;
      if constexpr (STORE) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          f32x4 t[NC];
#pragma unroll
          for (int c = 0; c < NC; ++c)
            t[c] = M::mma(Sb[kt][c], selD[p], f32x4{0.f, 0.f, 0.f, 0.f});
          cols.frag_out((bf16*)a.Sc + ch * DK * DV + (size_t)(2 * kt + p) * DV * 16, t);
        }
      }
    };
    auto qs = [&](auto kc) {  // (Q S)^T over k-step kt
      constexpr int kt = decltype(kc)::value, P = group_pos(kt, true, NKD, LAG);
      fetch(int_c<P + D - 1>{});
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) O[i][c] = M::mma(Sb[kt][c], f[P % D][i], O[i][c]);
#pragma unroll
      for (int i = 0; i < 4; ++i) pin(O[i]);
    };
    round_state(int_c<0>{});
    static_for<0, NKD>([&](auto kc) {
      constexpr int kt = decltype(kc)::value;
      constexpr int P = OUT ? group_pos(kt, false, NKD, LAG) : kt;
      fetch(int_c<P + D - 1>{});
      // the next chunk's rows into the other buffer (its readers passed the
      // barrier), and the loads of the one after
      if constexpr (!AFTER) {
        constexpr int X0 = kt * R::PER / NKD, X1 = (kt + 1) * R::PER / NKD;
        rows.template store<X0, X1>(put);
        load_rows(min(j + 2, nch - 1), int_c<X0>{}, int_c<X1>{});
        if constexpr (kt == NKD - 1) {
          tp.store(tri + step_tri, w);
          load_tp(min(j + 2, nch - 1));
        }
      }
      // K S
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) X[i][c] = M::mma(f[P % D][i], Sb[kt][c], X[i][c]);
#pragma unroll
      for (int i = 0; i < 4; ++i) pin(X[i]);
      store_state_step(kc);
      round_state(int_c<kt + 1>{});
      interleave<NC, 1>();
      phase();
      if constexpr (OUT && kt >= LAG) {
        qs(int_c<kt - LAG>{});
        interleave<NC, 1>();
        phase();
      }
    });
    // v's turn: ahead of the tail and the gates in the plain forward (48 x 4096,
    // 256/512: 314 -> 311 us), behind them where the rows are still to be stored
    // (training step 1,497 us, ahead of them 1,510)
    if constexpr (!STORE) vr.turn(bounce, len);
    if constexpr (AFTER) {
      rows.template store<0, R::PER>(put);
      load_rows(min(j + 2, nch - 1), int_c<0>{}, int_c<R::PER>{});
      tp.store(tri + step_tri, w);
      load_tp(min(j + 2, nch - 1));
    }
    R::zero_tail(put, min(CH, L - jn * CH), tid);
    put_gates(j + 1);
    load_g(min(j + 2, nch - 1));
    if constexpr (STORE) vr.turn(bounce, len);

    // R = V - e^g (K S), beside the last products of (Q S)^T
    f32x4 egr[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) egr[i] = *reinterpret_cast<const f32x4*>(&gate[0][16 * i + 4 * g]);
    auto residual = [&](int i) {
#pragma unroll
      for (int c = 0; c < NC; ++c) X[i][c] = vr.tile(i, c) - egr[i] * X[i][c];
    };
    if constexpr (OUT) {
      static_for<0, LAG>([&](auto qc) {
        constexpr int n = decltype(qc)::value;
        qs(int_c<NKD - LAG + n>{});
#pragma unroll
        for (int i = 4 * n / LAG; i < 4 * (n + 1) / LAG; ++i) residual(i);
        phase();
      });
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) residual(i);
    }
    frag tT[6];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
        if (tri_has(true, i, kt)) tT[tri_slot(true, i, kt)] = TP::template get<0>(tri, i, kt);
    f32x4 dec[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) dec[i] = *reinterpret_cast<const f32x4*>(&gate[1][16 * i + 4 * g]);
    frag Rb[2][NC];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int c = 0; c < NC; ++c) Rb[kt][c] = pack8(X[2 * kt][c], X[2 * kt + 1][c]);
    // V' = T diag(b) R
    frag Vb[2][NC], Vd[2][NC];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      f32x4 V[2][NC];
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          V[p][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int k = 0; k < 2; ++k)
            if (tri_has(true, 2 * kt + p, k))
              V[p][c] = M::mma(tT[tri_slot(true, 2 * kt + p, k)], Rb[k][c], V[p][c]);
        }
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        Vb[kt][c] = pack8(V[0][c], V[1][c]);
        Vd[kt][c] = pack8(V[0][c] * dec[2 * kt], V[1][c] * dec[2 * kt + 1]);
      }
    }
    phase();
    // S += K^T (e^{g_n - g} V'), and beside it O^T = (e^g Q S)^T + V'^T P^T,
    // V' for the backward, and the loads of the next chunk's operands
    const size_t row0 = (size_t)(s0 + j * CH) * H + h;
    float egc[4];
    if constexpr (OUT) {
#pragma unroll
      for (int i = 0; i < 4; ++i) egc[i] = gate[0][16 * i + (l & 15)];
    }
    auto out_tile = [&](int i) {
      if constexpr (OUT) {
        frag p[2];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
          if (tri_has(true, i, kt)) p[kt] = TP::template get<1>(tri, i, kt);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          O[i][c] *= egc[i];
#pragma unroll
          for (int kt = 0; kt < 2; ++kt)
            if (tri_has(true, i, kt)) O[i][c] = M::mma(Vb[kt][c], p[kt], O[i][c]);
        }
        cols.row_put(O[i], bounce);
      }
      if constexpr (STORE) {
        f32x4 t[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
          t[c] = M::mma(Vb[i >> 1][c], selT[i & 1], f32x4{0.f, 0.f, 0.f, 0.f});
        cols.frag_out((bf16*)a.Vp + ch * CH * DV + (size_t)i * DV * 16, t);
      }
    };
    auto out_row = [&](int i) {
      if constexpr (OUT) cols.row_out((bf16*)a.o + row0 * DV, H * DV * 2, i, len, bounce);
    };
    load_v(jn);
    static_for<0, NC_>([&](auto gc) {
      constexpr int G = decltype(gc)::value, P = NA + G;
      fetch(int_c<P + D - 1>{});
      // the tile put in the group before (a group of several: see below)
      if constexpr (G > 0 && 4 * (G - 1) / NC_ < 4 * G / NC_) out_row(4 * G / NC_ - 1);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          f32x4& s = S[2 * G + (i >> 1)][c];
          s = M::mma(f[P % D][i], Vd[i & 1][c], s);
        }
      pin(S[2 * G]);
      pin(S[2 * G + 1]);
      interleave<NC, 2>();
#pragma unroll
      for (int i = 4 * G / NC_; i < 4 * (G + 1) / NC_; ++i) {
        out_tile(i);
        if (i + 1 < 4 * (G + 1) / NC_) out_row(i);
      }
      phase();
    });
    out_row(3);
    ops.move(step);
    put.move(-step);
    step = -step;
    tri += step_tri;
    step_tri = -step_tri;
    lds_barrier();
  }

  if (OUT && a.ht) store_state<DV>(a.ht + sbase, S);
}

// ------------------------------------------------------------------ backward state pass

template <int DK, int DV, int NC, int NW>
__global__ __attribute__((amdgpu_flat_work_group_size(64 * NW, 64 * NW),
                          amdgpu_waves_per_eu(chain_occ<DK, NW>(), chain_occ<DK, NW>())))
void k_bwd_chain(Args a) {
  constexpr int NTH = 64 * NW, BV = 16 * NC * NW, NKD = DK / 32, MT = DK / 16;
  constexpr bool AFTER = NC == 2;
  using R = Rows<DK, 2, NTH>;
  __shared__ __align__(16) unsigned char sRows[2 * R::BUF];
  __shared__ __align__(16) float sGate[2][3][CH];  // by chunk parity: e^g, e^{g_n - g}, b
  __shared__ __align__(16) unsigned char sBounce[NW][Bounce<NC>::BYTES];
  __shared__ __align__(16) unsigned char sTri[2 * Tri<false, 2, NW>::BUF];

  int unit, tile;
  if (!map_unit_tile(DV / BV, a.N * a.H, unit, tile)) return;
  const int n = unit / a.H, h = unit - n * a.H, H = a.H;
  const int tid = threadIdx.x, l = lane_id(), g = l >> 4;
  const int w = __builtin_amdgcn_readfirstlane(wave_id());
  const Cols<NC, DK == 256> cols(tile * BV + w * 16 * NC);
  const unsigned rows0 = (unsigned)(uintptr_t)sRows;
  const Bounce<NC> bounce((unsigned)(uintptr_t)sBounce[w]);
  RowOps<DK> ops(rows0);              // reads the chunk's buffer
  typename R::At put(rows0, tid);     // writes the next one's
  unsigned tri = (unsigned)(uintptr_t)sTri + l * 16;  // T and P of the chunk
  const int s0 = a.cu ? a.cu[n] : n * a.T;
  const int L = a.cu ? a.cu[n + 1] - s0 : a.T;
  const int c0 = seq_first_chunk(a, n), nch = (L + CH - 1) / CH;
  frag selD[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) selD[p] = select8(8 * g, 16 * p + (l & 15));

  f32x4 dS[MT][NC];
  const size_t sbase = ((size_t)n * H + h) * DK * DV + cols.v0;
  load_state<DV>(a.dht ? const_cast<float*>(a.dht) + sbase : nullptr, dS);

  R rows;
  VRows<NC> dor;
  using TP = Tri<false, 2, NW>;  // P^T, T^T
  TP tp;
  float gl = 0.f, bl = 0.f;
  auto chunk = [&](int j) { return (size_t)(c0 + j) * H + h; };
  auto len_of = [&](int j) { return min(CH, L - j * CH); };
  auto load_rows = [&](int j, auto x0, auto x1) {
    const size_t row0 = (size_t)(s0 + j * CH) * H + h;
    rows.template load<decltype(x0)::value, decltype(x1)::value>(
        {(const bf16*)a.k + row0 * DK, (const bf16*)a.q + row0 * DK}, H * DK * 2, len_of(j), tid);
  };
  auto put_gates = [&](int j) {  // from gl and bl, by one wave
    if (w == 0) {
      sGate[j & 1][0][l] = __expf(gl);
      sGate[j & 1][1][l] = __expf(__shfl(gl, CH - 1, 64) - gl);
      sGate[j & 1][2][l] = l < len_of(j) ? bl : 0.f;
    }
  };
  auto load_tp = [&](int j) {
    const size_t at = chunk(j) * CH * CH;
    tp.load((const bf16*)a.PTf + at, (const bf16*)a.TTf + at, w);
  };
  auto load_do = [&](int j) {
    const size_t row0 = (size_t)(s0 + j * CH) * H + h;
    dor.load((const bf16*)a.dO + row0 * DV + cols.v0, H * DV * 2, len_of(j));
  };
  auto load_gates = [&](int j) {
    const size_t row0 = (size_t)(s0 + j * CH) * H + h;
    gl = ld<float>(a.g + chunk(j) * CH, l * 4u);
    bl = a.beta[row0 + (size_t)min(l, len_of(j) - 1) * H];
  };

  // the loads in the order of the loop, as in the forward
  if (nch > 0) {
    const int j = nch - 1;
    load_rows(j, int_c<0>{}, int_c<R::PER>{});
    load_tp(j);
    rows.template store<0, R::PER>(put);
    tp.store(tri, w);
    R::zero_tail(put, len_of(j), tid);
    put.move(R::BUF);
    load_gates(j);
    put_gates(j);
    load_rows(max(j - 1, 0), int_c<0>{}, int_c<R::PER>{});
    load_tp(max(j - 1, 0));
    load_gates(max(j - 1, 0));
    load_do(j);
    lds_barrier();
  }
  int step = R::BUF, step_tri = TP::BUF;  // to the other buffer
  for (int j = nch - 1; j >= 0; --j) {
    const int len = len_of(j), jn = max(j - 1, 0);
    const size_t ch = chunk(j), row0 = (size_t)(s0 + j * CH) * H + h;
    const float(&gate)[3][CH] = sGate[j & 1];
    const float egn = gate[0][CH - 1];  // pads repeat g of the last token
    // Operands from LDS in groups, as in the forward: the row operands of k,
    // then the transposed ones of q and of k.
    constexpr int NA = NKD, NC_ = MT / 2, NB = NA + NC_;
    constexpr int D = NC == 1 ? 3 : 2;
    frag f[D][4];
    auto fetch = [&](auto pc) {
      constexpr int P = decltype(pc)::value;
      if constexpr (P < NA) {
#pragma unroll
        for (int i = 0; i < 4; ++i) f[P % D][i] = ops.template rows<0>(i, P);
      } else if constexpr (P < NB + NC_) {
        constexpr int G = P < NB ? P - NA : P - NB;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          f[P % D][i] = ops.template cols<(P < NB ? R::TILE : 0)>(2 * G + (i >> 1), i & 1);
      }
    };
    static_for<0, D - 1>(fetch);
    phase();
    // K dS, from dS rounded to bf16 (stored, transposed, for the gradient
    // kernel); dS decays in place
    f32x4 X[4][NC];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int c = 0; c < NC; ++c) X[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    frag Sb[2][NC];
    auto round_state = [&](auto kc) {
      constexpr int kt = decltype(kc)::value;
      if constexpr (kt < NKD) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          Sb[kt & 1][c] = pack8(dS[2 * kt][c], dS[2 * kt + 1][c]);
          dS[2 * kt][c] *= egn;
          dS[2 * kt + 1][c] *= egn;
        }
        pin(dS[2 * kt]);
        pin(dS[2 * kt + 1]);
      }
    };
    round_state(int_c<0>{});
    static_for<0, NKD>([&](auto kc) {
      constexpr int kt = decltype(kc)::value;
      fetch(int_c<kt + D - 1>{});
      if constexpr (!AFTER) {
        constexpr int X0 = kt * R::PER / NKD, X1 = (kt + 1) * R::PER / NKD;
        rows.template store<X0, X1>(put);
        load_rows(max(j - 2, 0), int_c<X0>{}, int_c<X1>{});
        if constexpr (kt == NKD - 1) {
          tp.store(tri + step_tri, w);
          load_tp(max(j - 2, 0));
        }
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) X[i][c] = M::mma(f[kt % D][i], Sb[kt & 1][c], X[i][c]);
#pragma unroll
      for (int i = 0; i < 4; ++i) pin(X[i]);
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        f32x4 t[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c)
          t[c] = M::mma(Sb[kt & 1][c], selD[p], f32x4{0.f, 0.f, 0.f, 0.f});
        cols.frag_out((bf16*)a.dSc + ch * DK * DV + (size_t)(2 * kt + p) * DV * 16, t);
      }
      round_state(int_c<kt + 1>{});
      interleave<NC, 1>();
      phase();
    });
    if constexpr (AFTER) {
      rows.template store<0, R::PER>(put);
      load_rows(max(j - 2, 0), int_c<0>{}, int_c<R::PER>{});
      tp.store(tri + step_tri, w);
      load_tp(max(j - 2, 0));
    }
    R::zero_tail(put, len_of(jn), tid);
    if (j > 0) put_gates(j - 1);
    load_gates(max(j - 2, 0));
    dor.turn(bounce, len);
    // dO and e^g dO as B operands over t
    frag dOb[2][NC], dOg[2][NC];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {
      const f32x4 e0 = *reinterpret_cast<const f32x4*>(&gate[0][32 * kt + 4 * g]);
      const f32x4 e1 = *reinterpret_cast<const f32x4*>(&gate[0][32 * kt + 16 + 4 * g]);
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        dOb[kt][c] = dor.over_t(kt, c);
        dOg[kt][c] = pack8(dor.tile(2 * kt, c) * e0, dor.tile(2 * kt + 1, c) * e1);
      }
    }
    phase();
    load_do(jn);
    // dS += Q^T (e^g dO), and beside it the chain from K dS to b e^g dX:
    // dV' = P^T dO + e^{g_n - g} (K dS) (row tiles 2 s, 2 s + 1 in step s),
    // dX = T^T dV' as B operand over t, times -b e^g (steps 2, 3)
    frag dVb[2][NC], dRb[2][NC];
    auto chain_step = [&](int st) {
      if (st < 2) {
#pragma unroll
        for (int i = 2 * st; i < 2 * st + 2; ++i) {
          const f32x4 dec = *reinterpret_cast<const f32x4*>(&gate[1][16 * i + 4 * g]);
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            X[i][c] *= dec;
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
              if (tri_has(false, i, kt))
                X[i][c] = M::mma(TP::template get<0>(tri, i, kt), dOb[kt][c], X[i][c]);
          }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) dVb[st][c] = pack8(X[2 * st][c], X[2 * st + 1][c]);
      } else {
        const int s2 = st - 2;
        f32x4 d[2][NC];
#pragma unroll
        for (int p = 0; p < 2; ++p) {
          const int i = 2 * s2 + p;
          const f32x4 be = -*reinterpret_cast<const f32x4*>(&gate[0][16 * i + 4 * g]) *
                           *reinterpret_cast<const f32x4*>(&gate[2][16 * i + 4 * g]);
#pragma unroll
          for (int c = 0; c < NC; ++c) {
            d[p][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
              if (tri_has(false, i, kt))
                d[p][c] = M::mma(TP::template get<1>(tri, i, kt), dVb[kt][c], d[p][c]);
            d[p][c] *= be;
          }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) dRb[s2][c] = pack8(d[0][c], d[1][c]);
      }
    };
    static_for<0, NC_>([&](auto gc) {
      constexpr int G = decltype(gc)::value, P = NA + G;
      fetch(int_c<P + D - 1>{});
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          f32x4& s = dS[2 * G + (i >> 1)][c];
          s = M::mma(f[P % D][i], dOg[i & 1][c], s);
        }
      pin(dS[2 * G]);
      pin(dS[2 * G + 1]);
      interleave<NC, 2>();
#pragma unroll
      for (int st = 4 * G / NC_; st < 4 * (G + 1) / NC_; ++st) chain_step(st);
      phase();
    });
    // dS -= K^T (b e^g dX), and beside it dX, transposed, for dX and dv = b dX
    auto out_tile = [&](int i) {
      f32x4 d[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        d[c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
          if (tri_has(false, i, kt)) d[c] = M::mma(dVb[kt][c], TP::template get<1>(tri, i, kt), d[c]);
      }
      cols.frag_out((bf16*)a.dXb + ch * CH * DV + (size_t)i * DV * 16, d);
      const float b = gate[2][16 * i + (l & 15)];
#pragma unroll
      for (int c = 0; c < NC; ++c) d[c] *= b;
      cols.row_put(d, bounce);
    };
    auto out_row = [&](int i) {
      cols.row_out((bf16*)a.dv + row0 * DV, H * DV * 2, i, len, bounce);
    };
    static_for<0, NC_>([&](auto gc) {
      constexpr int G = decltype(gc)::value, P = NB + G;
      fetch(int_c<P + D - 1>{});
      if constexpr (G > 0 && 4 * (G - 1) / NC_ < 4 * G / NC_) out_row(4 * G / NC_ - 1);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          f32x4& s = dS[2 * G + (i >> 1)][c];
          s = M::mma(f[P % D][i], dRb[i & 1][c], s);
        }
      pin(dS[2 * G]);
      pin(dS[2 * G + 1]);
      interleave<NC, 2>();
#pragma unroll
      for (int i = 4 * G / NC_; i < 4 * (G + 1) / NC_; ++i) {
        out_tile(i);
        if (i + 1 < 4 * (G + 1) / NC_) out_row(i);
      }
      phase();
    });
    out_row(3);
    ops.move(step);
    put.move(-step);
    step = -step;
    tri += step_tri;
    step_tri = -step_tri;
    lds_barrier();
  }

  if (a.dh0) store_state<DV>(a.dh0 + sbase, dS);
}

}  // namespace gdn
