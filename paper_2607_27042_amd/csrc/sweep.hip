// The GPTQ-2D rounding sweep on 64 x 64 tiles (Sec. 4.2-4.3).
//
// Tile (I, J) holds rows 64I.. and columns 64J.. of X. An error at (i, j)
// reaches only rows >= i and columns >= j (Eq. rank-one-update), so tiles on
// one tile anti-diagonal I + J = s are independent and are swept together in
// launch s (s = 0 .. MT + NT - 2). Inside a tile the workgroup runs
// Algorithm 3 restricted to the tile; everything that crosses a tile edge is
// deferred, as in Algorithm 4's lazy block update, and delivered as dense
// products on MFMA:
//   down : P[I'][J] += L[I'][I]  E[I][J]      (completes C = L E below, and Y)
//   right: R[I][J'] += C[I][J]  U[J][J']      (right pushes of C = L E)
// With P the accumulated down feedback and R the accumulated right feedback,
// the corrected value of entry (i, j) when it is rounded is
//   y = X + R + (P + in-tile pushes down) + in-tile pushes right,
// which equals X + (L E U)_ij over earlier entries (proof of Theorem 2).
//
// Delivery: the sweeping workgroup of tile (I, J) itself pulls the
// contributions of its two immediate predecessors (I-1, J) and (I, J-1)
// (rank-64 products); everything older is delivered by GEMM tasks that run in
// the same launches as the sweeps, batched over g consecutive tile
// anti-diagonals (rank up to 64 g), never later than the launch before the
// target is swept. Each (target, direction) gets at most one task per launch,
// so accumulation needs no atomics and the result is deterministic.
#include <hip/hip_ext.h>
#include <math.h>

#include <algorithm>
#include <cstring>
#include <functional>
#include <queue>
#include <vector>

#include "device.hpp"
#include "internal.hpp"

namespace g2d {

struct StageArgs {
  int m, n, mp, np, MT, NT;
  const double* L;
  const double* U;
  const double* dL;
  const double* dU;
  // X, Z, Y at element (i, j) of the problem the sweep runs on: base + i ld +
  // j cstep. In the forward order cstep = 1 and the bases are the matrices';
  // in reverse order the problem is the index-reversed one, so each base is
  // the matrix's last element, ld its negated row stride and cstep = -1.
  const void* X;
  int64_t ldx;
  int32_t* Z;
  int64_t ldz;
  void* Y;
  int64_t ldy;
  int cstep;
  double* P;
  double* R;
  double* E;
  double* C;
  double* objp;
  double* obj;        // the objective (nullable), summed by the last launch's tile
  int* flags;
  const int4* tasks;  // this launch's deliveries, grouped by bin
  const int4* bins;   // this launch's bins (one work group each)
  int stage, ilo, nsweep;
  int set_flags;      // this launch sets the error word instead of adding to it
  // batched rounding: the problem's per-stage table {first task, first bin,
  // bins, 0}; tasks and bins then point at the problem's whole plan
  const int4* stab;
};

// A work group of a stage launch: eight waves, two per SIMD.
constexpr int ST = 512;

// The sweep of one tile: 16 x 16 blocks of 4 x 4 entries in four bands.
constexpr int BS = 4;              // block edge
constexpr int NB = TB / BS;        // blocks per tile edge
constexpr int BANDS = ST / 128;    // bands, each with a pair of waves
constexpr int BANDB = NB / BANDS;  // block rows of a band
constexpr int STEPS = NB + BANDB - 1;
constexpr int PAD = BS * (BANDB - 1);
// LDS row strides (doubles), at least TB + PAD. LDS serves 16 lanes of a 64-bit
// access at a time (4.2 cycles per wave instruction without conflicts): 76 has
// none in either layout of Et and Xs and for U's blocks, 80 takes 16 cycles for
// the chain layout; the transposed accesses of Ct take 8 at 78, 16 at 76 or 80.
constexpr int TE = TB + PAD;       // Et, Xs and Us
constexpr int TC = TE + 2;         // Ct
constexpr int TEN = TB * TE + PAD;
constexpr int TCN = TB * TC + PAD;

// LDS of a sweeping work group. A row of the arrays starts with 12 columns of
// zeros (the row before ends in them): a bank whose block column is still to
// come or already past the tile's edge reads and writes zeros there.
//   Xs: X plus the right feedback so far, then the corrected values
//   Ct: the down feedback so far, then C = L E
//   Et: the errors, as the blocks finish
//   Us: U_JJ, unit upper. Block row J' is read up to block column J' + 15: past
//     a row's end follow its 12 zeros and the lower triangle of the next rows.
//     What is read in front of Us (Ct) or behind it (Et) belongs to blocks
//     outside the tile and meets a zero; like everything here it is finite if X
//     is. (A NaN or an infinity in X spreads to other entries of its tile and of
//     later ones; it is reported, and Z and Y are then undefined.)
// Before the sweep the bytes of Et and Xs stage the two neighbour products.
struct SweepSmem {
  double Ct[TCN];
  double Us[TB * TE];
  union {
    struct {
      double Et[TEN];
      double Xs[TEN];
    };
    Stage64 g;
  };
  double red[ST / 64];
  int bad[ST / 64];
  int done[BANDS];  // per band: steps finished
  int prep[BANDS];  // per band: steps whose values in Xs and Ct are ready
};

// Staging of one 32-deep chunk of a delivery product, filled by direct
// global -> LDS loads (each wave instruction moves 64 lanes x 16 bytes to 1 KB
// of consecutive LDS): the left operand in blocks of four rows, each row's
// 16-byte pieces permuted by an XOR with the row's position in the block and
// every block padded by 64 bytes (an MFMA operand read of 16 rows then hits 16
// distinct bank groups), the right operand as rows b[k][col] padded to 130
// doubles. With the tile-contiguous storage a left-operand load reads 1 KB of
// contiguous memory and a right-operand load two 512-byte runs.
constexpr int KQ = 32;
constexpr int AQ = 4 * KQ + 8;  // doubles per 4-row block of the left operand (64 B pad)
struct TaskChunk {
  double a[2 * TB / 4][AQ];
  double b[KQ][2 * TB + 2];
};
struct TaskSmem {
  TaskChunk buf[2];
};

union StageSmem {
  SweepSmem s;
  TaskSmem t;
};

// X[gi][gj] widened, 0 outside the matrix; the load is unconditional (from a
// clamped address) so that it does not serialise behind a branch.
template <typename T>
__device__ __forceinline__ double load_x(const T* X, int64_t ldx, int cstep, int gi, int gj, int m,
                                         int n) {
  const bool ok = gi < m && gj < n;
  const T v = X[ok ? (int64_t)gi * ldx + gj * cstep : 0];
  return ok ? (double)v : 0.0;
}

// Operands of one delivery (uniform over the work group): out (+)= A B with
// A the (64 nr) x (64 K) source panel and B the (64 K) x (64 nc) panel, all
// tile-contiguous: A points at its first tile (S order), the next tile row
// ars doubles on and the next source tile 4096 on; B at its first tile (R
// order), the next source tile row bks on and the next tile column 4096 on;
// out at the first target tile (R order), the next tile row ors on.
struct TaskOp {
  const double* A;
  const double* B;
  double* out;
  int64_t ars, bks, ors;
  int nch, ow, nr, nc;
};

__device__ __forceinline__ TaskOp task_op(const StageArgs& a, int4 tk) {
  const int dir = tk.x & 1;
  const int ti = tk.y, tj = tk.z, s0 = tk.w & 0xffff, s1 = tk.w >> 16;
  TaskOp T;
  T.ow = (tk.x >> 1) & 1;
  T.nr = ((tk.x >> 2) & 1) + 1;
  T.nc = ((tk.x >> 3) & 1) + 1;
  T.nch = (s1 - s0) * (TB / KQ);
  T.bks = tile_off(1, 0, a.NT);
  T.ors = tile_off(1, 0, a.NT);
  if (dir == 0) {
    T.A = a.L + tile_off(ti, s0, a.MT);
    T.ars = tile_off(1, 0, a.MT);
    T.B = a.E + tile_off(s0, tj, a.NT);
    T.out = a.P + tile_off(ti, tj, a.NT);
  } else {
    T.A = a.C + tile_off(ti, s0, a.NT);
    T.ars = tile_off(1, 0, a.NT);
    T.B = a.U + tile_off(s0, tj, a.NT);
    T.out = a.R + tile_off(ti, tj, a.NT);
  }
  return T;
}

typedef __attribute__((address_space(3))) void lds_void;

// Chunk c of task T into d (source tile c / 2, its columns (rows of B)
// 32 (c % 2) ..): wave w moves the left-operand row blocks j = w + 8i (rows
// 4j .. 4j+3, i < 2 nr: 1 KB of contiguous memory in S order) and the
// right-operand rows k = w + 8i (i < 4), each a 1 KB direct global -> LDS
// load. Lane l of a left-operand load takes the 16-byte piece
// (l & 15) ^ (l >> 4) of row 4j + (l >> 4); of a right-operand load the
// columns 2l, 2l+1 (clamped to the target: never used past it).
// (i0, i1 select the part i0 <= i < i1 of the loads)
__device__ __forceinline__ void task_issue(const TaskOp& T, int c, TaskChunk& d, int w, int l, int i0 = 0,
                                           int i1 = 4) {
  const int ar = l >> 4, ap = (l & 15) ^ ar;
  const double* ac = T.A + (int64_t)(c >> 1) * 4096 + (c & 1) * 2048;
  const int col = min(2 * l, TB * T.nc - 2);
  const double* pb = T.B + (int64_t)(c >> 1) * T.bks + (c & 1) * 32 * TB + (col >> 6) * 4096 + (col & 63);
#pragma unroll
  for (int i = i0; i < i1; ++i) {
    const int j = w + 8 * i;
    if (i < 2 * T.nr) {
      const double* pa = ac + (j >> 4) * T.ars + (4 * (j & 15) + ar) * 32 + 2 * ap;
      __builtin_amdgcn_global_load_lds((const void*)pa, (lds_void*)&d.a[j][0], 16, 0, 0);
    }
    __builtin_amdgcn_global_load_lds((const void*)(pb + j * TB), (lds_void*)&d.b[j][0], 16, 0, 0);
  }
}

// The part of a (64 nr) x (64 nc) target that wave w computes, as NI x NJ
// MFMA blocks of 16 x 16 from row rb and column cb:
//   2 x 2 tiles: 64 x 32  NI = 4, NJ = 2
//   2 x 1 and 1 x 2 tiles: 32 x 32  NI = NJ = 2
//   1 x 1 tile : 32 x 16  NI = 2, NJ = 1
__device__ __forceinline__ void task_part(const TaskOp& T, int w, int& rb, int& cb) {
  if (T.nr == 2 && T.nc == 2) { rb = 64 * (w >> 2); cb = 32 * (w & 3); }
  else if (T.nr == 2) { rb = 32 * (w >> 1); cb = 32 * (w & 1); }
  else if (T.nc == 2) { rb = 32 * (w >> 2); cb = 32 * (w & 3); }
  else { rb = 32 * (w >> 2); cb = 16 * (w & 3); }
}

// Accumulators of the wave's part: the old target values (a delivery that
// adds) or zero (one that overwrites).
// Entry (row, col) of a target (rows and columns counted from its first
// tile) relative to T.out.
__device__ __forceinline__ int64_t task_at(const TaskOp& T, int row, int col) {
  return (row >> 6) * T.ors + (col >> 6) * 4096 + r_idx(row & 63, col & 63);
}

template <int NI, int NJ>
__device__ __forceinline__ void task_init(d4 (&acc)[NI][NJ], const TaskOp& T, int rb, int cb, int l) {
  if (!T.ow) {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          acc[i][j][r] = T.out[task_at(T, rb + 16 * i + 4 * r + (l >> 4), cb + 16 * j + (l & 15))];
    // the accumulators are complete before the chunk loop (so that no wait
    // for them lands inside it, where it would also wait for the next chunk)
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  } else {
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = d4{0.0, 0.0, 0.0, 0.0};
  }
}

template <int NI, int NJ>
__device__ __forceinline__ void task_store(const d4 (&acc)[NI][NJ], const TaskOp& T, int rb, int cb,
                                           int l) {
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        T.out[task_at(T, rb + 16 * i + 4 * r + (l >> 4), cb + 16 * j + (l & 15))] = acc[i][j][r];
}

// One staged chunk on MFMA: acc[i][j] += A(rows rb + 16 i ..) B(cols cb + 16 j ..).
// The operands of k-step kk + 1 are read while kk is on MFMA (two register
// sets), the reads spread between the MFMAs; mid() runs half-way (before the
// MFMAs of k-step KQ / 8).
template <int NI, int NJ, typename Mid>
__device__ __forceinline__ void task_mma(d4 (&acc)[NI][NJ], const TaskChunk& st, int rb, int cb, int l,
                                         Mid&& mid) {
  const int r0 = l & 15, rr = r0 & 3;
  double av[2][NI], bv[2][NJ];
#pragma unroll
  for (int kk = -1; kk < KQ / 4; ++kk) {
    const int nx = (kk + 1) & 1;
    if (kk + 1 < KQ / 4) {
      const int k = 4 * (kk + 1) + (l >> 4), kp = 2 * (kk + 1) + (l >> 5), e = (l >> 4) & 1;
      const int ao = KQ * rr + 2 * (kp ^ rr) + e;
#pragma unroll
      for (int i = 0; i < NI; ++i) av[nx][i] = st.a[(rb + 16 * i + r0) >> 2][ao];
#pragma unroll
      for (int j = 0; j < NJ; ++j) bv[nx][j] = st.b[k][cb + 16 * j + r0];
    }
    if (kk == KQ / 8) {
      // half-way: the rest of the next chunk's loads
      __builtin_amdgcn_sched_barrier(0);
      mid();
      __builtin_amdgcn_sched_barrier(0);
    }
    if (kk >= 0) {
      const int cur = kk & 1;
#pragma unroll
      for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[cur][i], bv[cur][j], acc[i][j], 0, 0, 0);
      if (kk + 1 < KQ / 4) {
        constexpr int NM = NI * NJ, NR = NI + NJ;  // MFMAs and reads per k-step
#pragma unroll
        for (int u = 0; u < NR; ++u) {
          __builtin_amdgcn_sched_group_barrier(0x008, NM / NR > 0 ? NM / NR : 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      }
    }
  }
}

// A run of n deliveries of one target shape (NI x NJ blocks per wave),
// streamed through one double-buffered pipeline: the next chunk of a
// delivery is loaded while the current one is on MFMA. At a delivery's end
// its result is stored first, and only then are the next delivery's first
// chunk and old target values loaded: stores queued behind loads wait for
// the memory pipeline, which costs more than the one exposed load latency.
// Every wave has a part of every target (task_part).
template <int NI, int NJ>
__device__ void run_stream(const StageArgs& a, const int4* tk, int n, TaskSmem& sm) {
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
  d4 acc[NI][NJ];
  TaskOp T = task_op(a, tk[0]);
  int rb, cb;
  task_part(T, w, rb, cb);
  task_issue(T, 0, sm.buf[0], w, l);
  task_init<NI, NJ>(acc, T, rb, cb, l);
  int idx = 0, c = 0, p = 0;
  for (;;) {
    const bool last = c + 1 == T.nch;
    // the next chunk's loads go out in two halves, the second one half-way
    // through this chunk's MFMAs (one batch of them stalls this wave's issue
    // until the memory pipeline takes it)
    if (!last) task_issue(T, c + 1, sm.buf[p ^ 1], w, l, 0, 2);
    // chunk c has landed (issued after it: the first half of the next, 4 loads)
    if (!last) __builtin_amdgcn_s_waitcnt(0x0f74);  // vmcnt(4)
    else __builtin_amdgcn_s_waitcnt(0x0f70);        // vmcnt(0)
    // a bare barrier: the wait above already covers this wave's part of
    // chunk c, and a fenced barrier would also wait for the next chunk
    asm volatile("s_barrier" ::: "memory");
    task_mma<NI, NJ>(acc, sm.buf[p], rb, cb, l, [&]() {
      if (!last) task_issue(T, c + 1, sm.buf[p ^ 1], w, l, 2, 4);
    });
    // buffer p is refilled next: every wave's reads of it are complete
    // before the barrier, while the next chunk stays in flight
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    p ^= 1;
    if (last) {
      task_store<NI, NJ>(acc, T, rb, cb, l);
      if (++idx == n) break;
      T = task_op(a, tk[idx]);
      c = 0;
      task_issue(T, 0, sm.buf[p], w, l);
      task_init<NI, NJ>(acc, T, rb, cb, l);
    } else {
      ++c;
    }
  }
}

// One bin of a launch's deliveries, bin = {first task, n22 | n21 << 16,
// n12 | n11 << 16, 0}: the counts of 2 x 2, 2 x 1, 1 x 2 and 1 x 1 targets,
// the tasks grouped in that order; each group is one stream.
__device__ void run_bin(const StageArgs& a, int4 bin, TaskSmem& sm) {
  const int4* tk = a.tasks + bin.x;
  const int n4 = bin.y & 0xffff, n21 = bin.y >> 16, n12 = bin.z & 0xffff, n11 = bin.z >> 16;
  bool busy = false;  // a group before this one used the staging buffers
  if (n4) { run_stream<4, 2>(a, tk, n4, sm); busy = true; }
  tk += n4;
  if (n21) { if (busy) __syncthreads(); run_stream<2, 2>(a, tk, n21, sm); busy = true; }
  tk += n21;
  if (n12) { if (busy) __syncthreads(); run_stream<2, 2>(a, tk, n12, sm); busy = true; }
  tk += n12;
  if (n11) { if (busy) __syncthreads(); run_stream<2, 1>(a, tk, n11, sm); }
}

typedef __attribute__((address_space(3))) double lds_double;

// v_mfma_f64_4x4x4: four independent 4 x 4 products, one per bank of four
// lanes in every row of 16. With lane = 16 r + 4 b + c, bank b:
//   A lane holds A[c][r], B lane B[r][c], D lane D[r][c].
// So a value in D's layout is the transpose of what it is as operand A, and
// itself as operand B.
__device__ __forceinline__ double mfma4(double a, double b, double c) {
  return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
}

// Bounded wait until a band's counter reaches v; a wait that runs out raises
// the time-out flag instead of hanging. A counter is written after the values
// it stands for by the same wave, and LDS serves a wave in order.
__device__ __forceinline__ int load_count(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// seen: the last value read; the counter is read again only if that is short
__device__ __forceinline__ void wait_count(const int* p, int v, int& seen, int& bad) {
  int spins = 0;
  while (__builtin_amdgcn_readfirstlane(seen) < v) {
    seen = load_count(p);
    if (++spins > (1 << 22)) {
      bad |= FLAG_TIMEOUT;
      break;
    }
  }
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void store_count(int* p, int v) {
  asm volatile("" ::: "memory");
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// y += w * (e of lane N of the lane's row of 16), a DPP broadcast inside the
// multiply-add.
#define G2D_PUSH(N_, y_, e_, w_) \
  "v_fmac_f64_dpp %[" #y_ "], %[" #e_ "], %[" #w_ "] row_newbcast:" #N_ " row_mask:0xf bank_mask:0xf\n\t"
// e = rint(y) - y. A DPP operand may be read two wait states after it was
// written: two of the next weights are formed in between.
#define G2D_ERR(e_, y_) "v_rndne_f64 %[" #e_ "], %[" #y_ "]\n\tv_add_f64 %[" #e_ "], %[" #e_ "], -%[" #y_ "]\n\t"
#define G2D_WEIGHT(w_, l_, u_, s_) "v_fma_f64 %[" #w_ "], %[" #l_ "], %[" #u_ "], %[" #s_ "]\n\t"

// The seven entry anti-diagonals of a 4 x 4 block, a lane per entry (i, j) = (lane / 4 % 4,
// lane % 4): on entry y holds everything from outside the block, on return the
// corrected values; e the errors. Entry n = 4 i' + j' reaches the others with the
// weight L[i][i'] U[j'][j] (self[n] takes the 1 at the entry itself away). One
// block of assembly, so that each weight stands where the chain has to wait.
__device__ __forceinline__ void block_chain(double& y, double& e, const double (&l)[BS], const double (&u)[BS],
                                            const double (&self)[15]) {
  double w0 = fma(l[0], u[0], self[0]), w1, w2, w3, w4, w5, w6;
  asm volatile(
      G2D_ERR(e, y) G2D_WEIGHT(w1, l0, u1, s1) G2D_WEIGHT(w2, l1, u0, s4)
      G2D_PUSH(0, y, e, w0)
      G2D_ERR(e, y) G2D_WEIGHT(w3, l0, u2, s2) G2D_WEIGHT(w4, l1, u1, s5)
      G2D_PUSH(1, y, e, w1) G2D_WEIGHT(w5, l2, u0, s8) G2D_PUSH(4, y, e, w2)
      G2D_ERR(e, y) G2D_WEIGHT(w0, l0, u3, s3) G2D_WEIGHT(w1, l1, u2, s6)
      G2D_PUSH(2, y, e, w3) G2D_WEIGHT(w2, l2, u1, s9) G2D_PUSH(5, y, e, w4) G2D_WEIGHT(w6, l3, u0, s12)
      G2D_PUSH(8, y, e, w5)
      G2D_ERR(e, y) G2D_WEIGHT(w3, l1, u3, s7) G2D_WEIGHT(w4, l2, u2, s10)
      G2D_PUSH(3, y, e, w0) G2D_WEIGHT(w5, l3, u1, s13) G2D_PUSH(6, y, e, w1)
      G2D_PUSH(9, y, e, w2) G2D_PUSH(12, y, e, w6)
      G2D_ERR(e, y) G2D_WEIGHT(w0, l2, u3, s11) G2D_WEIGHT(w1, l3, u2, s14)
      G2D_PUSH(7, y, e, w3) G2D_PUSH(10, y, e, w4) G2D_PUSH(13, y, e, w5)
      G2D_ERR(e, y) "s_nop 1\n\t"
      G2D_PUSH(11, y, e, w0) G2D_PUSH(14, y, e, w1)
      G2D_ERR(e, y)
      : [y] "+&v"(y), [e] "=&v"(e), [w0] "+&v"(w0), [w1] "=&v"(w1), [w2] "=&v"(w2), [w3] "=&v"(w3),
        [w4] "=&v"(w4), [w5] "=&v"(w5), [w6] "=&v"(w6)
      : [l0] "v"(l[0]), [l1] "v"(l[1]), [l2] "v"(l[2]), [l3] "v"(l[3]), [u0] "v"(u[0]), [u1] "v"(u[1]),
        [u2] "v"(u[2]), [u3] "v"(u[3]), [s1] "v"(self[1]), [s2] "v"(self[2]), [s3] "v"(self[3]),
        [s4] "v"(self[4]), [s5] "v"(self[5]), [s6] "v"(self[6]), [s7] "v"(self[7]), [s8] "v"(self[8]),
        [s9] "v"(self[9]), [s10] "v"(self[10]), [s11] "v"(self[11]), [s12] "v"(self[12]), [s13] "v"(self[13]),
        [s14] "v"(self[14]));
}

// What bounds a tile sweep is the chain of entry anti-diagonals, one after
// another: with all 64 lanes rounding 2 x 2 blocks of a 16 x 16 sub-tile in each
// of 15 steps it took about 8.9k cycles a sub-tile and 62k a tile (26 us; every
// step waited for an LDS exchange of errors and C and issued 49 instructions).
// Blocks of 4 x 4 in rows of 16 lanes exchange errors by DPP broadcasts and
// everything between blocks goes through the matrix unit: 232 cycles for a
// block's seven anti-diagonals, about 800 for a whole step of a wave that runs
// by itself. fp64 vector and matrix instructions share one pipe, so a band's
// older feedback, prepared on another SIMD, still delays the chains there. Whole
// problems went from 182 to 130 us (200 x 120), from 829 to 696 us (512 x 384,
// factorisation included), 4096 x 4096 rounds in 5.8 instead of 6.25 ms.
// Algorithm 3 on the 16 rows of band W. In step s, row-of-16 g of the wave
// rounds the 4 x 4 block (g, J = s - g) of the band, a lane per entry (lane =
// 16 g + 4 i + j), so the wave moves over the band along its block
// anti-diagonals in 19 steps. A step has two parts:
//   - the block's seven entry anti-diagonals. Each finished entry's error
//     reaches every later entry of its block as one multiply-add with a
//     broadcast operand: L[i][i'] U[j'][j] e, the weights formed beforehand.
//   - what the next step waits for, with matrix instructions: C = L E + D of
//     the block just finished (kept transposed: operand A as it is), its right
//     feedback C U on the next block, and the down feedback of the band's block
//     above the next one (as D U, and added to D). The two layouts meet in LDS.
// The feedback of the step before it is added on the way; all older feedback
// is prepared by the band's second wave (prepare_band) three steps ahead. A bank
// whose block column is before the tile's first or past the last holds zeros
// throughout.
// Feedback is summed by itself and added to an entry's value in one addition: a
// product accumulated onto the value would round at the value's magnitude in
// every term. Error of Y against long double, 200 x 120: 1.6e-16 (3.7e-16 with
// the products accumulated onto X), in the same time (126 us, 125).
template <int W>
__device__ __forceinline__ void sweep_band(const double* Ltile, SweepSmem& sm, int l, int& bad) {
  const int r = l >> 4, b = (l >> 2) & 3, c = l & 3;  // matrix layout: bank b, entry (r, c)
  // L[.][.] of the lane's block row against its own block and the two above
  const int lr = BS * (BANDB * W + b) + c;
  const double v0 = Ltile[s_idx(lr, BS * (BANDB * W + b) + r)];
  const double v1 = Ltile[s_idx(lr, BS * (BANDB * W + max(b - 1, 0)) + r)];
  const double v2 = Ltile[s_idx(lr, BS * (BANDB * W + max(b - 2, 0)) + r)];
  // chain layout: block row r, entry (b, c)
  const int cr = BS * (BANDB * W + r);
  double lw[BS], self[15];
#pragma unroll
  for (int k = 0; k < BS; ++k) lw[k] = Ltile[s_idx(cr + b, cr + k)];
  const double la0 = r < c ? v0 : r == c ? 1.0 : 0.0, la1 = b > 0 ? v1 : 0.0, la2 = b > 1 ? v2 : 0.0;
#pragma unroll
  for (int k = 0; k < BS; ++k) lw[k] = k < b ? lw[k] : k == b ? 1.0 : 0.0;
#pragma unroll
  for (int k = 0; k < 15; ++k) self[k] = (l & 15) == k ? -1.0 : 0.0;

  // LDS addresses of step 0; one block column further per step
  const int mrow = BS * (BANDB * W + b);
  lds_double* pu = (lds_double*)(sm.Us + (r - BS * b) * TE + c - BS * b);  // block (J, J) of U
  lds_double* pw = (lds_double*)(sm.Us - BS * r * TE + c - BS * r);        // the same, chain layout
  lds_double* pt = (lds_double*)(sm.Ct + PAD + (mrow + c) * TC + r - BS * b);  // Ct, transposed
  // Et, matrix layout, two block rows up (their weights are zero where the
  // band has none); Xs is at a constant distance
  lds_double* pe = (lds_double*)(sm.Et + PAD + (mrow - 2 * BS + r) * TE + c - BS * b);
  lds_double* po = (lds_double*)(sm.Et + PAD + (cr + b) * TE + c - BS * r);    // Et, chain layout
  constexpr int EX = TEN;  // from Et to Xs

  int seen = 0;
  wait_count(&sm.prep[W], 1, seen, bad);
  double dt = pt[0], ct = 0.0, u2 = 0.0;
  pe[EX + 2 * BS * TE] += mfma4(dt, pu[0], 0.0);
  asm volatile("" ::: "memory");
  double y = po[EX], err;
  double uw[BS];
#pragma unroll
  for (int k = 0; k < BS; ++k) uw[k] = pw[k * TE];
#pragma unroll 1
  for (int s = 0; s < STEPS; ++s) {
    // (opaque addresses: constant offsets from them fit the LDS instructions)
    asm volatile("" : "+v"(pu), "+v"(pw), "+v"(pt), "+v"(pe), "+v"(po));
    // operands of the next step, read while this one's chain runs; if its
    // values were not ready yet they are read again behind it
    seen = load_count(&sm.prep[W]);
    asm volatile("" ::: "memory");
    double xn = pe[EX + 2 * BS * TE + BS], dn = pt[BS];
    const double e2 = pe[BS], u1 = pu[BS], un = pu[BS * TE + BS], u2n = pu[2 * BS];
    block_chain(y, err, lw, uw, self);
    po[0] = err;
    asm volatile("" ::: "memory");
    const double em = pe[2 * BS * TE], e1 = pe[BS * TE + BS];
    po[EX] = y;
#pragma unroll
    for (int k = 0; k < BS; ++k) uw[k] = pw[BS * TE + BS + k * TE];
    const double xa = mfma4(ct, u2, 0.0);
    double da = mfma4(e2, la2, dn);
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(seen) < min(s + 2, STEPS), 0)) {
      // (counter before values: the values are valid if the counter was)
      int spins = 0;
      do {
        seen = load_count(&sm.prep[W]);
        asm volatile("" ::: "memory");
        xn = pe[EX + 2 * BS * TE + BS];
        dn = pt[BS];
        if (++spins > (1 << 22)) {
          bad |= FLAG_TIMEOUT;
          break;
        }
      } while (__builtin_amdgcn_readfirstlane(seen) < min(s + 2, STEPS));
      da = mfma4(e2, la2, dn);
    }
    ct = mfma4(em, la0, dt);
    dt = mfma4(e1, la1, da);
    double ym = mfma4(ct, u1, xa);
    ym = xn + mfma4(dt, un, ym);
    pt[0] = ct;
    if (s + 1 < STEPS) pe[EX + 2 * BS * TE + BS] = ym;  // (a column further is the next row's first)
    asm volatile("" ::: "memory");
    y = po[EX + BS];
    store_count(&sm.done[W], s + 1);
    u2 = u2n;
    pu += BS * TE + BS;
    pw += BS * TE + BS;
    pt += BS;
    pe += BS;
    po += BS;
  }
}

// The second wave of band W: three steps ahead of the first it completes the
// values that step k starts from. acc[d] holds the right feedback that the
// blocks finished so far (steps <= k - 3) have on the blocks of step k + d; the
// down feedback comes from the band's block three above and from all blocks of
// the bands above.
template <int W>
__device__ __forceinline__ void prepare_band(const double* Ltile, SweepSmem& sm, int l, int& bad) {
  const int r = l >> 4, b = (l >> 2) & 3, c = l & 3;
  const int mrow = BS * (BANDB * W + b), lr = mrow + c;
  constexpr int NQ = BANDB * W;           // blocks above the band
  constexpr int NO = W > 1 ? NQ - BANDB : 0;  // of which not in the band next above
  double lb[NQ > 0 ? NQ : 1];
#pragma unroll
  for (int q = 0; q < NQ; ++q) lb[q] = Ltile[s_idx(lr, BS * q + r)];
  const double v3 = Ltile[s_idx(lr, max(mrow - 3 * BS, 0) + r)];
  const double la3 = b > 2 ? v3 : 0.0;

  // LDS addresses of step 0
  lds_double* pu = (lds_double*)(sm.Us + (r - BS * b - 3 * BS) * TE + c - BS * b);  // block (J - 3, J) of U
  lds_double* pm = (lds_double*)(sm.Xs + PAD + (mrow + r) * TE + c - BS * b);
  lds_double* pt = (lds_double*)(sm.Ct + PAD + (mrow + c) * TC + r - BS * b);
  lds_double* pe = (lds_double*)(sm.Et + PAD + r * TE + c - BS * b);
  lds_double* p3 = (lds_double*)(sm.Et + PAD + (mrow - 3 * BS + r) * TE + c - BS * b);

  constexpr int ND = NB - 3;
  double acc[ND + 1], uv[ND], ev[NQ > 0 ? NQ : 1];
#pragma unroll
  for (int d = 0; d <= ND; ++d) acc[d] = 0.0;
  int seen = 0, above = 0;  // steps known to be finished: this band, the band above
  int* const up = &sm.done[W > 0 ? W - 1 : 0];
  if (W > 0) wait_count(up, BANDB, above, bad);
  // A step's values, but for its right feedback, from the down feedback of the
  // bands above; those of the blocks further above are there (the band next
  // above waited for them before its own last steps).
  double x, d0, d1;
  auto begin = [&](int at) {
    x = pm[at];
    d0 = pt[at];
    d1 = 0.0;
#pragma unroll
    for (int q = 0; q < NO; ++q) ev[q] = pe[BS * q * TE + at];
  };
  auto far = [&]() {
#pragma unroll
    for (int q = 0; q < NO; ++q) (q & 1 ? d1 : d0) = mfma4(ev[q], lb[q], q & 1 ? d1 : d0);
  };
  auto near = [&]() {
#pragma unroll
    for (int q = NO; q < NQ; ++q) (q & 1 ? d1 : d0) = mfma4(ev[q], lb[q], q & 1 ? d1 : d0);
  };
  // steps 0, 1, 2: no block of the band is finished early enough
#pragma unroll 1
  for (int k = 0; k < 3; ++k) {
    begin(0);
    if (W > 0) wait_count(up, k + BANDB, above, bad);
#pragma unroll
    for (int q = NO; q < NQ; ++q) ev[q] = pe[BS * q * TE];
    far();
    near();
    if (W > 0) *pt = d0 + d1;
    store_count(&sm.prep[W], k + 1);
    pu += BS * TE + BS;
    pm += BS;
    pt += BS;
    pe += BS;
    p3 += BS;
  }
  begin(0);
  uv[0] = pu[0];
  far();
#pragma unroll 1
  for (int k = 3; k < STEPS; ++k) {
    asm volatile("" : "+v"(pu), "+v"(pm), "+v"(pt), "+v"(pe), "+v"(p3));
    // counters before values: the values are valid if the counters were
    double ct, e3;
    for (int spins = 0;;) {
      seen = load_count(&sm.done[W]);
      if (W > 0) above = load_count(up);
      asm volatile("" ::: "memory");
      ct = pt[-3 * BS];
      e3 = *p3;
#pragma unroll
      for (int q = NO; q < NQ; ++q) ev[q] = pe[BS * q * TE];
      const bool there = __builtin_amdgcn_readfirstlane(seen) >= k - 2 &&
                         (W == 0 || __builtin_amdgcn_readfirstlane(above) >= min(k + BANDB, STEPS));
      if (__builtin_expect(there, 1)) break;
      if (++spins > (1 << 22)) {
        bad |= FLAG_TIMEOUT;
        break;
      }
    }
#pragma unroll
    for (int d = 1; d < ND; ++d) uv[d] = pu[BS * d];
    __builtin_amdgcn_sched_barrier(0);
    acc[0] = mfma4(ct, uv[0], acc[1]);
    d1 = mfma4(e3, la3, d1);
    near();
    *pm = x + acc[0];
    *pt = d0 + d1;
    store_count(&sm.prep[W], k + 1);
    // the next step's operands
    begin(BS);
    uv[0] = pu[BS * TE + BS];
    __builtin_amdgcn_sched_barrier(0);
    // the feedback on the steps further ahead; blocks past the tile's last
    // column are left out
#pragma unroll
    for (int c0 = 1; c0 < ND; c0 += 4) {
      if (k + c0 < STEPS) {
#pragma unroll
        for (int d = c0; d < c0 + 4 && d < ND; ++d) acc[d] = mfma4(ct, uv[d], acc[d + 1]);
      }
    }
    far();
    pu += BS * TE + BS;
    pm += BS;
    pt += BS;
    pe += BS;
    p3 += BS;
  }
}

// Rows r0 .. r0 + n - 1 of a finished tile by one wave, a lane per column: Z,
// Y, E, C and the lane's part of the objective.
template <typename T>
__device__ __forceinline__ void sweep_output(const StageArgs& a, const SweepSmem& sm, int I, int J, int r0,
                                             int n, double du, bool interior, double& part, int& bad) {
  const int l = threadIdx.x & 63;
  const int64_t gj = (int64_t)J * TB + l;
  double* const E = a.E + tile_off(I, J, a.NT);
  double* const C = a.C + tile_off(I, J, a.NT);
  const bool in = gj < a.n;
#pragma unroll 2
  for (int i = 0; i < n; ++i) {
    const int rr = r0 + i;
    const int64_t gi = (int64_t)I * TB + rr;
    const int at = PAD + rr * TE + l;
    const double y = sm.Xs[at], e = sm.Et[at];
    E[r_idx(rr, l)] = e;
    C[s_idx(rr, l)] = sm.Ct[PAD + rr * TC + l];
    if (interior || (in && gi < a.m)) {
      // (a NaN fails the range test, too)
      if (!(y >= -2147483648.5 && y < 2147483647.5)) bad |= isfinite(y) ? FLAG_OVERFLOW : FLAG_NONFINITE;
      const double z = fmin(fmax(rint(y), -2147483648.0), 2147483647.0);
      a.Z[gi * a.ldz + gj * a.cstep] = (int32_t)z;
      if (a.Y) ((T*)a.Y)[gi * a.ldy + gj * a.cstep] = (T)y;
      part = fma(e * e, a.dL[gi] * du, part);
    }
  }
}

// 64 x 64 blocks by the 512 threads of a work group: element e = t + 512 s.
__device__ __forceinline__ void sweep_load(const double* p, double (&v)[8]) {
#pragma unroll
  for (int s = 0; s < 8; ++s) v[s] = p[threadIdx.x + ST * s];
}
// operands of a neighbour product: a (in S order) and b (in R order), both
// k-major in LDS
__device__ __forceinline__ void sweep_stage(Stage64& g, const double (&a)[8], const double (&b)[8]) {
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int e = threadIdx.x + ST * s;
    g.a[((e >> 11) << 5) + (e & 31)][(e >> 5) & 63] = a[s];
    g.b[e >> 6][e & 63] = b[s];
  }
}
// acc[u] += rows 32 (w / 4) + 16 u .., columns 16 (w % 4) .. of the staged product
__device__ __forceinline__ void sweep_product(d4 (&acc)[2], const Stage64& g) {
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int rb = 32 * (w >> 2) + (l & 15), cb = 16 * (w & 3) + (l & 15);
#pragma unroll
  for (int kk = 0; kk < TB / 4; ++kk) {
    const int k = 4 * kk + (l >> 4);
    const double a0 = g.a[k][rb], a1 = g.a[k][rb + 16], b0 = g.b[k][cb];
    acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a0, b0, acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a1, b0, acc[1], 0, 0, 0);
  }
}

// Sweep of one tile. The deferred feedback (P, R) and the two neighbour products
// (L[I][I-1] E[I-1][J] and C[I][J-1] U[J-1][J], each a sum of its own) are added
// in the accumulator layout of the products, the right feedback then to X, and go
// to LDS, where the bands' sweeps start from them.
template <typename T>
__device__ void run_sweep(const StageArgs& a, int I, int J, SweepSmem& sm) {
  const int t = threadIdx.x, w = t >> 6, l = t & 63;
  const int gi0 = I * TB, gj0 = J * TB;
  const T* X = (const T*)a.X;

  // every global load of the prologue is issued before any is used
  double uv[8], ga[8], gb[8], gc[8], gd[8];
  if (I >= 1) {
    sweep_load(a.L + tile_off(I, I - 1, a.MT), ga);
    sweep_load(a.E + tile_off(I - 1, J, a.NT), gb);
  }
  if (J >= 1) {
    sweep_load(a.C + tile_off(I, J - 1, a.NT), gc);
    sweep_load(a.U + tile_off(J - 1, J, a.NT), gd);
  }
  sweep_load(a.U + tile_off(J, J, a.NT), uv);
  d4 accR[2], accD[2];
  double xv[2][4], rv[2][4], pv[2][4];
  const double* const Rt = a.R + tile_off(I, J, a.NT);
  const double* const Pt = a.P + tile_off(I, J, a.NT);
  const int ar = 32 * (w >> 2) + (l >> 4), ac = 16 * (w & 3) + (l & 15);  // + 16 u + 4 q rows
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int rr = ar + 16 * u + 4 * q;
      xv[u][q] = load_x<T>(X, a.ldx, a.cstep, gi0 + rr, gj0 + ac, a.m, a.n);
      rv[u][q] = J >= 2 ? Rt[r_idx(rr, ac)] : 0.0;
      pv[u][q] = I >= 2 ? Pt[r_idx(rr, ac)] : 0.0;
      accR[u][q] = accD[u][q] = 0.0;
    }
  const double du = a.dU[gj0 + l];

  // U_JJ, unit upper, and its zero columns
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const int e = t + ST * s, r = e >> 6, x = e & 63;
    sm.Us[r * TE + x] = x > r ? uv[s] : x == r ? 1.0 : 0.0;
  }
  for (int e = t; e < TB * PAD; e += ST) sm.Us[(e / PAD) * TE + TB + e % PAD] = 0.0;
  if (t < BANDS) sm.done[t] = sm.prep[t] = 0;
  if (I >= 1) {
    sweep_stage(sm.g, ga, gb);
    __syncthreads();
    sweep_product(accD, sm.g);
    __syncthreads();
  }
  if (J >= 1) {
    sweep_stage(sm.g, gc, gd);
    __syncthreads();
    sweep_product(accR, sm.g);
    __syncthreads();
  }
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      sm.Xs[PAD + (ar + 16 * u + 4 * q) * TE + ac] = xv[u][q] + (rv[u][q] + accR[u][q]);
      sm.Ct[PAD + (ar + 16 * u + 4 * q) * TC + ac] = pv[u][q] + accD[u][q];
    }
  // the zero columns; no errors yet (a product with a zero weight must not meet
  // a NaN in memory that nobody has written)
  for (int e = t; e < (TB + 1) * PAD; e += ST) sm.Xs[(e / PAD) * TE + e % PAD] = 0.0;
  for (int e = t; e < PAD + TB * (TC - TB); e += ST)
    sm.Ct[e < PAD ? e : PAD + TB + (e - PAD) / (TC - TB) * TC + (e - PAD) % (TC - TB)] = 0.0;
  for (int e = t; e < TEN / 2; e += ST) *reinterpret_cast<double2*>(&sm.Et[2 * e]) = double2{0.0, 0.0};
  __syncthreads();

  double part = 0.0;
  int bad = 0;
  const double* const Lt = a.L + tile_off(I, I, a.MT);
  // (the second wave of a band runs on the SIMD of a band two further down,
  // which has half of its steps at another time)
  const int band = (w < BANDS ? w : w + 2) & (BANDS - 1);
  if (w < BANDS) {
    __builtin_amdgcn_s_setprio(2);
    if (band == 0) sweep_band<0>(Lt, sm, l, bad);
    else if (band == 1) sweep_band<1>(Lt, sm, l, bad);
    else if (band == 2) sweep_band<2>(Lt, sm, l, bad);
    else sweep_band<3>(Lt, sm, l, bad);
    __builtin_amdgcn_s_setprio(0);
  } else {
    if (band == 0) prepare_band<0>(Lt, sm, l, bad);
    else if (band == 1) prepare_band<1>(Lt, sm, l, bad);
    else if (band == 2) prepare_band<2>(Lt, sm, l, bad);
    else prepare_band<3>(Lt, sm, l, bad);
  }
  // the bands' outputs: half a band by each of its two waves, the last band's
  // by all
  const bool interior = gi0 + TB <= a.m && gj0 + TB <= a.n;
  constexpr int BR = BS * BANDB;
  if (band < BANDS - 1) {
    int seen = 0;
    wait_count(&sm.done[band], STEPS, seen, bad);
    sweep_output<T>(a, sm, I, J, BR * band + (w < BANDS ? 0 : BR / 2), BR / 2, du, interior, part, bad);
  }
  __syncthreads();
  sweep_output<T>(a, sm, I, J, BR * (BANDS - 1) + BR / 8 * w, BR / 8, du, interior, part, bad);

  bad = __any(bad & FLAG_NONFINITE) ? bad | FLAG_NONFINITE : bad;
  bad = __any(bad & FLAG_OVERFLOW) ? bad | FLAG_OVERFLOW : bad;
  bad = __any(bad & FLAG_TIMEOUT) ? bad | FLAG_TIMEOUT : bad;
  auto wave_sum = [](double v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
  };
  auto group_sum = [&]() {
    return ((sm.red[0] + sm.red[1]) + (sm.red[2] + sm.red[3])) + ((sm.red[4] + sm.red[5]) + (sm.red[6] + sm.red[7]));
  };
  part = wave_sum(part);
  if (l == 0) {
    sm.red[w] = part;
    sm.bad[w] = bad;
  }
  __syncthreads();
  const double own = group_sum();
  if (t == 0) {
    int any = 0;
#pragma unroll
    for (int i = 0; i < ST / 64; ++i) any |= sm.bad[i];
    // the first launch of a round has one tile, which sets the error word (a
    // batch shares one word, cleared beforehand)
    if (a.set_flags) a.flags[0] = any;
    else if (any) raise_flag(a.flags, any);
    a.objp[I * a.NT + J] = own;
  }
  // the last launch has one tile, too: every other tile's part is in memory
  if (a.obj && I == a.MT - 1 && J == a.NT - 1) {
    const int count = a.MT * a.NT - 1;
    double s = 0.0;
    for (int i = t; i < count; i += ST) s += a.objp[i];
    s = wave_sum(s);
    __syncthreads();
    if (l == 0) sm.red[w] = s;
    __syncthreads();
    if (t == 0) a.obj[0] = group_sum() + own;
  }
}

template <typename T>
__global__ __launch_bounds__(ST) void k_stage(StageArgs a) {
  __shared__ StageSmem sm;
  const int b = blockIdx.x;
  if (b < a.nsweep) {
    const int I = a.ilo + b;
    run_sweep<T>(a, I, a.stage - I, sm.s);
  } else {
    run_bin(a, a.bins[b - a.nsweep], sm.t);
  }
}

// ---------------------------------------------------------------------------
// Batched rounding: independent problems (each with its own factors, X, Z, Y
// and workspace region) share the stage launches. Launch k holds the stage-k
// work groups of every problem that has a stage k: problem p owns the blocks
// off[p] .. off[p+1]-1 and runs them exactly as k_stage would, so the merged
// launch has the work of all problems in flight at once (small problems
// occupy a few compute units each). Problem p's record in a device table
// holds what differs between calls; the rest of its StageArgs is its
// handle's, kept on the device with the handle.
constexpr int BATCH_MAX = 512;  // problems per launch (block offsets travel as kernel arguments)
struct BatchProb {
  const StageArgs* base;  // the handle's fixed part (shape, factors, plan)
  const void* X;
  int32_t* Z;
  void* Y;
  int64_t ldx, ldz, ldy, cstep;
  void* ws;  // the problem's workspace region (layout of carve_workspace)
};
struct BatchLaunch {
  const BatchProb* desc;
  int* flags;  // the batch's error word
  double* obj; // the problems' objectives (nullable)
  int count, stage;
  int off[BATCH_MAX + 1];
};

// Tables that no work group of the launch writes, through the scalar cache: as
// ordinary loads, which the kernel's stores might alias, they would put the problem's
// arguments into 50 vector registers of every lane, and two would spill.
template <typename S>
__device__ __forceinline__ S scalar_load(const S* p) {
  typedef const __attribute__((address_space(4))) uint64_t* words;
  static_assert(sizeof(S) % sizeof(uint64_t) == 0, "loaded in 8-byte words");
  const words q = (words)(uintptr_t)p;
  uint64_t w[sizeof(S) / sizeof(uint64_t)];
#pragma unroll
  for (size_t i = 0; i < sizeof(S) / sizeof(uint64_t); ++i) w[i] = q[i];
  S s;
  __builtin_memcpy(&s, w, sizeof(S));
  return s;
}

__device__ __forceinline__ StageArgs batch_args(const BatchProb* prob, int* flags) {
  const BatchProb q = scalar_load(prob);
  StageArgs a = scalar_load(q.base);
  a.X = q.X;
  a.ldx = q.ldx;
  a.Z = q.Z;
  a.ldz = q.ldz;
  a.Y = q.Y;
  a.ldy = q.ldy;
  a.cstep = (int)q.cstep;
  const Workspace w = carve_workspace(q.ws, a.mp, a.np, a.MT, a.NT);
  a.objp = w.objp;
  a.P = w.P;
  a.R = w.R;
  a.E = w.E;
  a.C = w.C;
  a.flags = flags;
  return a;
}

template <typename T>
__global__ __launch_bounds__(ST) void k_stage_batch(BatchLaunch bl) {
  __shared__ StageSmem sm;
  const int b = blockIdx.x;
  // the last p with off[p] <= b (problems without a stage k own no block)
  int lo = 0, hi = bl.count - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (bl.off[mid] <= b) lo = mid;
    else hi = mid - 1;
  }
  StageArgs a = batch_args(bl.desc + lo, bl.flags);
  a.obj = bl.obj ? bl.obj + lo : nullptr;
  const int k = bl.stage, lb = b - bl.off[lo];
  const int4 st = scalar_load(a.stab + k);
  a.stage = k;
  int ihi;
  stage_rows(a.MT, a.NT, k, a.ilo, ihi);
  a.nsweep = ihi - a.ilo + 1;
  a.tasks = a.tasks ? a.tasks + st.x : nullptr;
  a.bins = a.bins ? a.bins + st.y : nullptr;
  if (lb < a.nsweep) {
    const int I = a.ilo + lb;
    run_sweep<T>(a, I, k - I, sm.s);
  } else {
    run_bin(a, a.bins[lb - a.nsweep], sm.t);
  }
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

static size_t align256(size_t b) { return (b + 255) / 256 * 256; }

size_t workspace_bytes(const Factors& f) {
  const size_t tile = (size_t)f.mp * f.np * sizeof(double);
  return 256 + align256((size_t)f.MT * f.NT * sizeof(double)) + 4 * tile;
}

Workspace workspace_carve(const Factors& f, void* base) {
  return carve_workspace(base, f.mp, f.np, f.MT, f.NT);
}

// Delivery plan of the deferred feedback. Targets are grouped in 2 x 2
// super-tiles (fewer at an odd edge); for super-tile rows {2a, 2a+1} and
// columns {2b, 2b+1} the down direction gets
//   - source tile rows 0 .. 2a-4 in batches of g, as products onto the whole
//     super-tile (up to 128 x 128), each in a launch after its sources are
//     swept and at least two launches before the super-tile's first sweep;
//   - source rows 2a-3 .. 2a-2 onto rows 2a, 2a+1 of one tile column c at a
//     time, in launch 2a + c - 1 (the last before tile (2a, c) is swept);
//   - source row 2a-1 onto tile (2a+1, c), in launch 2a + c;
// (source row 2a-1 of tile (2a, c) and 2a of tile (2a+1, c) are the sweeping
// workgroup's own neighbour products). The right direction is the same with
// rows and columns exchanged. Every target gets each source once, at most one
// delivery per launch, the first one (in launch order) overwriting.
//
// The far batches have a window of launches; they are placed earliest-
// deadline-first into the room that each launch leaves beside its tile
// sweeps (a launch lasts at least one tile sweep, so deliveries that fit in
// that time on the idle compute units are free), and otherwise at their
// deadline. Batches of one super-tile and direction get distinct launches.
// Task word: x = dir | overwrite << 1 | (rows - 1) << 2 | (cols - 1) << 3
// (rows, cols in tiles), y = first target tile row, z = first target tile
// column, w = first source | (one past the last source) << 16.
// (creating a handle waits for this: stable counting sorts instead of comparisons)

// Stable order of the items by key (0 <= key < n), and each key's first place.
static void counting_order(const std::vector<int>& key, int n, std::vector<int>& order, std::vector<int>& at) {
  at.assign(n + 1, 0);
  for (int k : key) ++at[k + 1];
  for (int k = 0; k < n; ++k) at[k + 1] += at[k];
  order.resize(key.size());
  std::vector<int> next(at);
  for (size_t i = 0; i < key.size(); ++i) order[next[key[i]]++] = (int)i;
}

void schedule_tasks(int MT, int NTt, int g, std::vector<int4>& all, std::vector<int>& off) {
  const int S = MT + NTt - 1;
  g = std::max(1, std::min(g, std::max(MT, NTt)));  // (wider ones are the same)
  std::vector<int4> found;
  std::vector<int> key;  // of the task: work, launch
  std::vector<double> load(S, 0.0);
  auto work = [](int nr, int nc, int k) { return nr * nc * k; };  // in 64^3 units
  const int wmax = 4 * std::max(g, 2);
  auto emit = [&](int launch, int dir, int ti, int tj, int nr, int nc, int s0, int s1) {
    const int w = work(nr, nc, s1 - s0);
    found.push_back(make_int4(dir | ((nr - 1) << 2) | ((nc - 1) << 3), ti, tj, s0 | (s1 << 16)));
    key.push_back(launch * wmax + (wmax - w));
    load[launch] += w;
  };
  struct Batch {
    int release, deadline, slot, dir, r0, c0, nr, nc, s0, s1;
  };
  std::vector<Batch> batches;
  int nslot = 0;
  for (int a = 0; 2 * a < MT; ++a) {
    for (int b = 0; 2 * b < NTt; ++b) {
      const int r0 = 2 * a, c0 = 2 * b;
      const int nr = std::min(2, MT - r0), nc = std::min(2, NTt - c0);
      for (int dir = 0; dir < 2; ++dir, ++nslot) {
        // along: the target index that sources run along (rows for down)
        const int t0 = dir == 0 ? r0 : c0, nt = dir == 0 ? nr : nc;
        const int o0 = dir == 0 ? c0 : r0, no = dir == 0 ? nc : nr;  // the other index
        // far sources 0 .. t0-4, batched; batch beta of nb may go no later
        // than latest - (nb - 1 - beta), which keeps distinct launches
        // feasible (its sources are swept one launch after the previous
        // batch's at the latest)
        const int far = t0 - 4;
        const int latest = r0 + c0 - 2;  // two launches before the first sweep
        const int nbatch = far >= 0 ? far / g + 1 : 0;
        for (int beta = 0; beta < nbatch; ++beta) {
          const int s0 = beta * g, sl = std::min(far, s0 + g - 1);
          batches.push_back(Batch{sl + o0 + no, latest - (nbatch - 1 - beta), nslot, dir, r0, c0, nr, nc, s0,
                                  sl + 1});
        }
        // near sources t0-3 .. t0-2 onto both targets along, one other index at a time
        if (t0 - 2 >= 0) {
          const int s0 = std::max(0, t0 - 3);
          for (int o = o0; o < o0 + no; ++o) {
            const int launch = t0 + o - 1;
            if (dir == 0) emit(launch, 0, r0, o, nt, 1, s0, t0 - 1);
            else emit(launch, 1, o, c0, 1, nt, s0, t0 - 1);
          }
        }
        // source t0-1 onto the second target along only
        if (nt == 2 && t0 - 1 >= 0) {
          for (int o = o0; o < o0 + no; ++o) {
            const int launch = t0 + o;
            if (dir == 0) emit(launch, 0, r0 + 1, o, 1, 1, t0 - 1, t0);
            else emit(launch, 1, o, c0 + 1, 1, 1, t0 - 1, t0);
          }
        }
      }
    }
  }
  // room per launch beside its sweeps: the idle compute units for the
  // duration of one tile sweep, in 64^3-product units (only the ratio between
  // launches and the total matter for the placement). Measured rounds in ms at
  // 12 / 16 / 20 units: 4096 x 4096 5.59 / 5.39 / 6.25, 4096 x 11008 20.3 / 19.7 /
  // 18.9, 8192 x 8192 30.0 / 29.3 / 28.8: with more than 64 tiles on a side the
  // middle launches are bound by the deliveries that are due there, and the
  // early ones take more of them.
  const double per_unit = std::max(MT, NTt) > 64 ? 20.0 : 16.0;
  // A super-tile and direction has its batches in the order of their deadlines, and
  // one per launch: only its first one left waits for room. come[k]: the slots whose
  // next batch can go from launch k on (a list through slot_next).
  std::vector<int> come(S + 1, -1), slot_next(nslot);
  auto arrive = [&](int i, int k) {
    slot_next[batches[i].slot] = come[std::min(k, S)];
    come[std::min(k, S)] = i;
  };
  for (int i = 0; i < (int)batches.size(); ++i)
    if (i == 0 || batches[i].slot != batches[i - 1].slot) arrive(i, batches[i].release);
  // earliest deadline first, then the batch found first
  std::priority_queue<int64_t, std::vector<int64_t>, std::greater<int64_t>> avail;
  for (int k = 0; k < S; ++k) {
    for (int i = come[k]; i >= 0; i = slot_next[batches[i].slot])
      avail.push((int64_t)batches[i].deadline << 32 | i);
    const int nsweep = std::min(k, MT - 1) - std::max(0, k - NTt + 1) + 1;
    const double room = per_unit * std::max(0, 256 - nsweep);
    while (!avail.empty()) {
      const int64_t top = avail.top();
      const bool due = (top >> 32) <= k;
      if (!due && load[k] >= room) break;
      avail.pop();
      const int i = (int)(uint32_t)top;
      const Batch& bt = batches[i];
      emit(k, bt.dir, bt.r0, bt.c0, bt.nr, bt.nc, bt.s0, bt.s1);
      if (i + 1 < (int)batches.size() && batches[i + 1].slot == bt.slot)
        arrive(i + 1, std::max(k + 1, batches[i + 1].release));
    }
  }
  // overwrite flag: the first delivery in launch order into each target
  std::vector<char> seen((size_t)2 * MT * NTt, 0);
  // launch by launch, biggest products first, so the short ones fill in behind them
  std::vector<int> order, at;
  counting_order(key, S * wmax, order, at);
  all.resize(found.size());
  for (size_t i = 0; i < order.size(); ++i) {
    int4& tk = all[i] = found[order[i]];
    const int dir = tk.x & 1;
    char& f = seen[2 * ((size_t)tk.y * NTt + tk.z) + dir];
    if (!f) tk.x |= 2;
    const int nr = ((tk.x >> 2) & 1) + 1, nc = ((tk.x >> 3) & 1) + 1;
    for (int r = 0; r < nr; ++r)
      for (int c = 0; c < nc; ++c) seen[2 * ((size_t)(tk.y + r) * NTt + tk.z + c) + dir] = 1;
  }
  off.resize(S + 1);
  for (int k = 0; k <= S; ++k) off[k] = at[k * wmax];
}

// Bins of a stage: one per compute unit, filled longest-processing-time
// first with an estimated cost per task (microseconds per 32-deep chunk by
// target size, plus a start cost that is larger when the old target values
// are read), so that the bins finish close together; a work group per
// non-empty bin, after the sweeps. The first units - nsweep bins start
// beside the sweeps; the others only when a sweep is done, so they start
// loaded with its duration (and stay empty when the work fits beside the
// sweeps).
// (The costs of the products are a least-squares fit of bin durations at 4096 and 8192
// that was made with four waves a delivery; with eight a chunk onto 2 x 2 tiles has
// about 3.4 of matrix work. The sweep's was lowered from 45 with the 4 x 4 blocks,
// whose tiles take about 23. What they are for is the ratio between bins: the
// launches they add up to are within 10 % of the measured rounds.)
constexpr double kSweepCost = 35.0;   // one tile sweep
constexpr double kChunk4 = 5.1;       // 32-deep chunk onto 2 x 2 tiles
constexpr double kChunk2 = 2.4;       // onto 2 x 1 or 1 x 2 tiles
constexpr double kChunk1 = 1.2;       // onto one tile
constexpr double kStartOw = 1.0;      // a delivery that overwrites
constexpr double kStartAdd = 6.0;     // a delivery that adds to the old values
gptq2d_status pack_bins(int MT, int NTt, int units, std::vector<int4>& all,
                        const std::vector<int>& off, std::vector<int4>& bins, std::vector<int>& boff) {
  const int S = MT + NTt - 1;
  bins.clear();
  boff.assign(S + 1, 0);
  std::vector<int4> out;
  out.reserve(all.size());
  auto shape = [](const int4& x) { return 3 - ((x.x >> 2) & 1) * 2 - ((x.x >> 3) & 1); };  // 2 x 2, 2 x 1, 1 x 2, 1 x 1
  auto depth = [](const int4& x) { return (x.w >> 16) - (x.w & 0xffff); };
  auto cost = [](int sh, int K, int ow) {
    const double chunk = sh == 0 ? kChunk4 : sh == 3 ? kChunk1 : kChunk2;
    return (ow ? kStartOw : kStartAdd) + chunk * (TB / KQ) * K;
  };
  // the kinds of tasks (depth, shape, overwrite) by falling cost, equal costs together
  int kmax = 0;
  for (const int4& x : all) kmax = std::max(kmax, depth(x));
  auto kind = [&](const int4& x) { return (depth(x) * 4 + shape(x)) * 2 + ((x.x >> 1) & 1); };
  const int kinds = 8 * (kmax + 1);
  std::vector<double> kcost(kinds);
  std::vector<int> by(kinds), rank(kinds);
  for (int q = 0; q < kinds; ++q) {
    kcost[q] = cost((q >> 1) & 3, q >> 3, q & 1);
    by[q] = q;
  }
  std::sort(by.begin(), by.end(), [&](int x, int y) { return kcost[x] > kcost[y]; });
  for (int x = 0; x < kinds; ++x) rank[by[x]] = x > 0 && kcost[by[x]] == kcost[by[x - 1]] ? rank[by[x - 1]] : x;
  const int nb = std::max(1, units);
  std::vector<int> key, order, at, home;
  typedef std::pair<double, int> Load;
  std::vector<Load> heap;
  for (int k = 0; k < S; ++k) {
    boff[k] = (int)bins.size();
    const int n = off[k + 1] - off[k];
    if (n == 0) continue;
    const int4* tk = all.data() + off[k];
    const int nsweep = std::min(k, MT - 1) - std::max(0, k - NTt + 1) + 1;
    const int nfree = std::max(0, units - nsweep);
    key.resize(n);
    home.resize(n);
    for (int i = 0; i < n; ++i) key[i] = rank[kind(tk[i])];
    counting_order(key, kinds, order, at);
    if (n <= nfree) {  // an empty bin for each
      for (int i = 0; i < n; ++i) home[order[i]] = i;
    } else {
      // least-loaded bin first (ties: lowest index)
      heap.clear();
      for (int b = 0; b < nb; ++b) heap.emplace_back(b < nfree ? 0.0 : kSweepCost, b);  // (in heap order)
      for (int i : order) {
        home[i] = heap[0].second;
        const Load top(heap[0].first + kcost[kind(tk[i])], heap[0].second);
        int p = 0;
        for (int c = 1; c < nb; c = 2 * p + 1) {
          if (c + 1 < nb && heap[c + 1] < heap[c]) ++c;
          if (top < heap[c]) break;
          heap[p] = heap[c];
          p = c;
        }
        heap[p] = top;
      }
    }
    // bin by bin, grouped by target shape, in the order they were taken
    key.clear();
    for (int i : order) key.push_back(home[i] * 4 + shape(tk[i]));
    std::vector<int>& taken = home;
    taken.swap(order);
    counting_order(key, 4 * nb, order, at);
    const int base = (int)out.size();
    for (int x : order) out.push_back(tk[taken[x]]);
    for (int b = 0; b < nb; ++b) {
      const int* c = &at[4 * b];
      if (c[4] == c[0]) continue;
      if (c[4] - c[0] > 0xffff) {
        set_error("delivery plan: too many products in one bin");
        return GPTQ2D_ERR_INVALID_ARG;
      }
      bins.push_back(make_int4((int)out.size() - base - n + c[0], (c[1] - c[0]) | ((c[2] - c[1]) << 16),
                               (c[3] - c[2]) | ((c[4] - c[3]) << 16), 0));
    }
  }
  boff[S] = (int)bins.size();
  all.swap(out);
  return GPTQ2D_OK;
}

// Both plans in one allocation and one upload (each costs the creation of a handle
// 10 to 20 us), and one plan where they are the same.
gptq2d_status build_schedules(Factors& f, int g, int gbatch) {
  int units = 0;
  if (hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, f.device) != hipSuccess ||
      units <= 0)
    units = 256;
  const int S = f.MT + f.NT - 1;
  std::vector<int4> all[2], bins[2];
  schedule_tasks(f.MT, f.NT, std::max(g, 1), all[0], f.sched.offset);
  if (gbatch != g) schedule_tasks(f.MT, f.NT, std::max(gbatch, 1), all[1], f.bsched.offset);
  const bool same = gbatch == g || (f.sched.offset == f.bsched.offset &&
                                    !memcmp(all[0].data(), all[1].data(), all[0].size() * sizeof(int4)));
  const int plans = same ? 1 : 2;
  Schedule* const sc[2] = {&f.sched, &f.bsched};
  size_t at[2] = {0, 0}, total = 0;  // in int4s: tasks, bins, stage table, stage arguments
  for (int p = 0; p < plans; ++p) {
    const gptq2d_status st = pack_bins(f.MT, f.NT, units, all[p], sc[p]->offset, bins[p], sc[p]->bin_offset);
    if (st != GPTQ2D_OK) return st;
    at[p] = total;
    total += all[p].size() + bins[p].size() + S + (sizeof(StageArgs) + sizeof(int4) - 1) / sizeof(int4);
  }
  void* block = nullptr;
  hipError_t e = hipMalloc(&block, total * sizeof(int4));
  if (e != hipSuccess) return hip_fail(e, "schedule allocation");
  f.allocations.push_back(block);
  std::vector<int4> image(total);
  for (int p = 0; p < plans; ++p) {
    Schedule& q = *sc[p];
    int4* const dev = (int4*)block + at[p];
    const size_t nt = all[p].size(), nbins = bins[p].size();
    q.stages = S;
    q.d_tasks = nt ? dev : nullptr;
    q.d_bins = nt ? dev + nt : nullptr;
    q.d_stage = dev + nt + nbins;
    q.d_base = dev + nt + nbins + S;
    int4* const h = image.data() + at[p];
    std::copy(all[p].begin(), all[p].end(), h);
    std::copy(bins[p].begin(), bins[p].end(), h + nt);
    for (int k = 0; k < S; ++k)
      h[nt + nbins + k] = int4{q.offset[k], q.bin_offset[k], q.bin_offset[k + 1] - q.bin_offset[k], 0};
    // the fixed stage arguments of the handle (batched rounding)
    StageArgs b{};
    b.m = f.m;
    b.n = f.n;
    b.mp = f.mp;
    b.np = f.np;
    b.MT = f.MT;
    b.NT = f.NT;
    b.L = f.L;
    b.U = f.U;
    b.dL = f.dL;
    b.dU = f.dU;
    b.tasks = q.d_tasks;
    b.bins = q.d_bins;
    b.stab = q.d_stage;
    memcpy(h + nt + nbins + S, &b, sizeof(b));
  }
  e = hipMemcpy(block, image.data(), total * sizeof(int4), hipMemcpyHostToDevice);
  if (e != hipSuccess) return hip_fail(e, "schedule upload");
  if (same) f.bsched = f.sched;
  return GPTQ2D_OK;
}

template <typename T>
static StageArgs stage_args(const Factors& f, const void* X, int64_t ldx, int32_t* Z, int64_t ldz,
                            void* Y, int64_t ldy, const Workspace& ws) {
  StageArgs a{};
  a.m = f.m;
  a.n = f.n;
  a.mp = f.mp;
  a.np = f.np;
  a.MT = f.MT;
  a.NT = f.NT;
  a.L = f.L;
  a.U = f.U;
  a.dL = f.dL;
  a.dU = f.dU;
  if (f.rev) {  // the index-reversed problem: X[m-1-i][n-1-j] etc.
    const int64_t last_x = (int64_t)(f.m - 1) * ldx + (f.n - 1);
    const int64_t last_z = (int64_t)(f.m - 1) * ldz + (f.n - 1);
    const int64_t last_y = (int64_t)(f.m - 1) * ldy + (f.n - 1);
    a.X = (const T*)X + last_x;
    a.ldx = -ldx;
    a.Z = Z + last_z;
    a.ldz = -ldz;
    a.Y = Y ? (void*)((T*)Y + last_y) : nullptr;
    a.ldy = -ldy;
    a.cstep = -1;
  } else {
    a.X = X;
    a.ldx = ldx;
    a.Z = Z;
    a.ldz = ldz;
    a.Y = Y;
    a.ldy = ldy;
    a.cstep = 1;
  }
  a.P = ws.P;
  a.R = ws.R;
  a.E = ws.E;
  a.C = ws.C;
  a.objp = ws.objp;
  a.flags = ws.flags;
  return a;
}

// work groups of stage k of a problem of a batch: the tile sweeps beside the
// delivery bins
static int stage_blocks(const Factors& f, int k) {
  int ilo, ihi;
  stage_rows(f.MT, f.NT, k, ilo, ihi);
  return (ihi - ilo + 1) + (f.bsched.bin_offset[k + 1] - f.bsched.bin_offset[k]);
}

template <typename T>
static gptq2d_status round_typed(const Factors& f, const void* X, int64_t ldx, int32_t* Z,
                                 int64_t ldz, void* Y, int64_t ldy, double* objective,
                                 const Workspace& ws, hipStream_t s, bool allow_timing) {
  StageArgs a = stage_args<T>(f, X, ldx, Z, ldz, Y, ldy, ws);
  a.obj = objective;
  const Schedule& S = f.sched;
  for (int k = 0; k < S.stages; ++k) {
    int ilo, ihi;
    stage_rows(f.MT, f.NT, k, ilo, ihi);
    a.stage = k;
    a.ilo = ilo;
    a.nsweep = ihi - ilo + 1;
    a.set_flags = k == 0;
    const int ntasks = S.bin_offset[k + 1] - S.bin_offset[k];  // work groups beside the sweeps
    a.tasks = S.d_tasks ? S.d_tasks + S.offset[k] : nullptr;
    a.bins = S.d_bins ? S.d_bins + S.bin_offset[k] : nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (f.stage_timing && allow_timing) {
      while (f.stage_ev.size() < f.stage_ev_used + 2) {
        hipEvent_t ev;
        hipError_t e = hipEventCreate(&ev);
        if (e != hipSuccess) return hip_fail(e, "hipEventCreate");
        f.stage_ev.push_back(ev);
      }
      e0 = f.stage_ev[f.stage_ev_used];
      e1 = f.stage_ev[f.stage_ev_used + 1];
      f.stage_ev_used += 2;
    }
    // with timing on, the two events take the start and end time stamps of
    // the dispatch itself (no marker packets between the launches)
    hipExtLaunchKernelGGL(k_stage<T>, dim3(a.nsweep + ntasks), dim3(ST), 0, s, e0, e1, 0, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "sweep launch");
  return GPTQ2D_OK;
}

gptq2d_status launch_round(const Factors& f, gptq2d_dtype dt, const void* X, int64_t ldx,
                           int32_t* Z, int64_t ldz, void* Y, int64_t ldy, double* objective,
                           const Workspace& ws, hipStream_t s, bool allow_timing) {
  if (dt == GPTQ2D_F32) return round_typed<float>(f, X, ldx, Z, ldz, Y, ldy, objective, ws, s, allow_timing);
  return round_typed<double>(f, X, ldx, Z, ldz, Y, ldy, objective, ws, s, allow_timing);
}

// Workspace of a batch: the batch's error flags (256 bytes), the problems'
// StageArgs table, then one gptq2d_round workspace region per problem.
static size_t batch_table_bytes(int count) { return align256((size_t)count * sizeof(BatchProb)); }

size_t batched_workspace_bytes(int count, const Factors* const* f) {
  size_t b = 256 + batch_table_bytes(count);
  for (int p = 0; p < count; ++p) b += align256(workspace_bytes(*f[p]));
  return b;
}

template <typename T>
static gptq2d_status round_batched_typed(int count, const Factors* const* f, const void* const* X,
                                         const int64_t* ldx, int32_t* const* Z, const int64_t* ldz,
                                         void* const* Y, const int64_t* ldy, double* objective,
                                         void* workspace, hipStream_t s) {
  static_assert(sizeof(BatchProb) % sizeof(uint64_t) == 0, "the table is uploaded in 8-byte words");
  char* base = (char*)workspace;
  int* flags = (int*)base;
  BatchProb* desc = (BatchProb*)(base + 256);
  char* region = base + 256 + batch_table_bytes(count);
  // the table behind a cleared error word, in one upload
  std::vector<char> head(256 + (size_t)count * sizeof(BatchProb), 0);
  BatchProb* const h = reinterpret_cast<BatchProb*>(head.data() + 256);
  for (int p = 0; p < count; ++p) {
    const Workspace ws = workspace_carve(*f[p], region);
    // X, Z, Y as the problem's sweep addresses them (mirrored in reverse order)
    const StageArgs a = stage_args<T>(*f[p], X[p], ldx[p], Z[p], ldz[p], Y ? Y[p] : nullptr, Y ? ldy[p] : 0, ws);
    h[p] = BatchProb{(const StageArgs*)f[p]->bsched.d_base, a.X, a.Z, a.Y, a.ldx, a.ldz, a.ldy, a.cstep, region};
    region += align256(workspace_bytes(*f[p]));
  }
  const gptq2d_status st = enqueue_upload(base, head.data(), head.size(), s);
  if (st != GPTQ2D_OK) return st;
  for (int g0 = 0; g0 < count; g0 += BATCH_MAX) {
    const int cnt = std::min(BATCH_MAX, count - g0);
    int smax = 0;
    for (int q = 0; q < cnt; ++q) smax = std::max(smax, f[g0 + q]->bsched.stages);
    BatchLaunch bl;
    bl.desc = desc + g0;
    bl.flags = flags;
    bl.obj = objective ? objective + g0 : nullptr;
    bl.count = cnt;
    for (int k = 0; k < smax; ++k) {
      int tot = 0;
      for (int q = 0; q < cnt; ++q) {
        bl.off[q] = tot;
        if (k < f[g0 + q]->bsched.stages) tot += stage_blocks(*f[g0 + q], k);
      }
      bl.off[cnt] = tot;
      bl.stage = k;
      hipLaunchKernelGGL(k_stage_batch<T>, dim3(tot), dim3(ST), 0, s, bl);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "batched sweep launch");
  return GPTQ2D_OK;
}

gptq2d_status launch_round_batched(int count, const Factors* const* f, gptq2d_dtype dt,
                                   const void* const* X, const int64_t* ldx, int32_t* const* Z,
                                   const int64_t* ldz, void* const* Y, const int64_t* ldy,
                                   double* objective, void* workspace, hipStream_t s) {
  if (dt == GPTQ2D_F32)
    return round_batched_typed<float>(count, f, X, ldx, Z, ldz, Y, ldy, objective, workspace, s);
  return round_batched_typed<double>(count, f, X, ldx, Z, ldz, Y, ldy, objective, workspace, s);
}

}  // namespace g2d
