// Per-column Krylov growth and projection (hot path of the multiple Arnoldi
// method: one Krylov subspace per column j of G = (zS - H)^-1, Eq. 1).
//
// One workgroup of eight waves owns up to two columns j = (J, alpha) of one
// atom at a time: the columns of an atom share its cluster C(J), so every
// block of H_C is read once for both.  Per column:
//   growth, nu steps:
//     w = H_C q_k                         SpMV on the matrix cores
//     w -= alpha q_k + beta_{k-1} q_{k-1}  (alpha = q_k^T w from the SpMV's epilogue)
//     c = Q^T w;  w -= Q c                 one Gram-Schmidt pass over the basis
//     h[:,k] = c + alpha e_k + beta_{k-1} e_{k-1}
//     q_{k+1} = w / |w|                    (breakdown: |w| <= tol |H q_k|)
//   projection of S, once: s = Q^T (S_C Q), S_C Q as a multi-vector product.
// The local subtraction removes what cancels most (H is symmetric, so h is
// tridiagonal up to rounding), so the one full pass leaves w orthogonal to a
// few ulps; when it still removes more than half of |w|^2 (an almost invariant
// space) two more passes run, and the last one's |w|^2 - |c|^2 is the norm.  The basis is
// Euclidean-orthonormal; it spans the same Krylov space K_nu(H_C; e_l) as the
// S-orthonormal basis of the method's reading, so the projected pencil (h, s)
// has the same Ritz pairs.
//
// SpMV.  v_mfma_f64_4x4x4_4b multiplies four independent 4x4 blocks by four
// vectors of length four: a wave takes a tile of four cluster atoms, one block
// of each per instruction, the vectors being the columns (two of the four).
// Cluster atoms are ordered by their number of blocks (rank, ties by atom
// id), so the four of a tile end together.  A tile's first blocks sit in LDS
// (as many as fit), the others stream from L2 while the cached ones are used.
//
// Basis.  It stays in registers: half of a column's lanes hold its even
// vectors and half the odd ones (bit 4 of the lane), each lane the rows p +
// LROWS m of its row-lane p.  Dot products then need five reduction levels for
// sixteen values at a time, and a row's sum over the basis one exchange.
// Reductions run in a fixed order that depends on the cluster and on nu only,
// so a column's bits depend neither on the launch nor on its partner column.
//
// What bounds it: latency along a step's serial chain (SpMV, local subtraction,
// dots, subtraction, three barriers between them), with two waves on each SIMD,
// as many as the basis registers leave room for: a wave waits for memory or a
// barrier in 45% of its cycles, for an issue slot in 21%, and issues in 34%; a
// SIMD's vector pipe is active 42% of the time, its matrix pipe 15% (nu = 30, all
// 15,568 columns of 3,892 atoms).  A step of two
// columns in clusters of about 156 atoms takes about 14,000 cycles: SpMV 5,600
// (a third of it from the cache), local subtraction 1,500, dots 1,300, totals,
// subtraction and store 4,100; the projection adds about 5,000 per step.
// Measured (MI355X, nu = 30, all 15,568 columns of 3,892 atoms in one launch):
// 7.3 ms; one column per 768-thread workgroup with vector FMA and two full
// orthogonalization passes took 13.5 ms.  The 29,000-atom void cell at nu =
// 20, clusters up to 164 atoms: 32 against 61 ms; nu = 48 at 3,892 atoms and
// r = 4.5: 13 against 23 ms.
//
// Scheduling: persistent workgroups pull columns from KRYLOV_QUEUES device
// queues, each a spatially compact range of atoms; workgroup w starts on
// queue w % KRYLOV_QUEUES (workgroups are dealt to the XCDs round-robin, so a
// queue's clusters share that XCD's L2) and steals from the others when its
// own is empty.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "mag_internal.h"
#include "wave.h"

namespace mag {

constexpr int ENT_MAX = CLUSTER_MAX * 24;  // local blocks of a cluster
constexpr int KTPB = 512;                  // threads per workgroup
constexpr int KW = KTPB / 64;              // waves
constexpr int TILE_MAX = CLUSTER_MAX / 4;
constexpr int HASH = 512;                  // slots of the cluster's atom lookup
constexpr int PAIR_CACHE = 1024;           // LDS bytes of one cached pair of tile blocks (H only)
// A wave's work is a list of units, four blocks of each atom of a tile.  A lane
// reads two neighbouring columns of one row of a block (16 bytes), the lanes of
// the instruction's four contraction indices y the columns 0-1 and 2-3 of two
// blocks; one instruction contracts the first columns, a second one the others,
// so two instructions and one 16-byte read of each operand cover two blocks.
// A unit has two table entries per atom and half of the lanes (y / 2): the byte
// offsets of its two column atoms' operands (16 bits each), and the places of
// the two blocks in the global array, in units of 16 bytes
constexpr int TAB_UNIT = 96, TAB_B = 32;   // bytes of both, offset of the second
// streamed units read ahead, eight registers each next to the basis (an even
// number, as the operands alternate between two places): with four instead of
// two the smaller shapes gain nothing and the larger spill (3,892 atoms, nu = 30:
// r = 5, 120 registers of basis, 5.36 against 5.04 ms; r = 6, 150, 10.6 against 7.3)
constexpr int RING = 2;
constexpr int PAD_UNITS = 2;               // dummy units after a wave's last

// LDS bytes of an operand buffer and of the product
// (two planes, of orbitals 0-1 and 2-3; an atom has two columns of an orbital
// pair there, 32 bytes)
constexpr int x_plane(int rows) { return (rows / 4 + 1) * 32 + 64; }
constexpr size_t x_bytes(int rows) { return (size_t)2 * x_plane(rows); }
constexpr size_t w_bytes(int rows) { return (size_t)rows * 16; }
// basis vectors of each column per pass of the S projection
constexpr int PROJ_CB = 4;
// (kept like the operands: per atom two orbital pairs, 16 bytes per vector, and
// a pad against bank conflicts, narrower where the LDS is full)
constexpr int proj_atom(int rows, int ncol) {
  return 2 * ncol * PROJ_CB * 16 + (rows > 640 ? 32 : 64);
}
constexpr size_t proj_bytes(int rows, int ncol, int nset) {
  return (size_t)(2 * (rows / 4) + 1) * proj_atom(rows, ncol) + (size_t)PROJ_CB * KW * 32 * nset * 8;
}
constexpr int tiles_per_wave(int rows) { return (rows / 16 + KW - 1) / KW; }
// units of a cluster at most: eight a tile, and by the tiles' longest rows L
// (which fall with the tile, so that 4 L is at most the entries of the tile
// before) (ENT_MAX / 4 + BLOCKS_MAX + 3 tiles) / 4
constexpr int units_max(int rows) {
  const int t = rows / 16, a = t * (BLOCKS_MAX / 4), b = (ENT_MAX / 4 + BLOCKS_MAX + 3 * t) / 4;
  return a < b ? a : b;
}
constexpr size_t tab_bytes(int rows) {
  return (size_t)(units_max(rows) + KW * PAD_UNITS) * TAB_UNIT;
}
// dynamic LDS a workgroup needs whatever the cluster: the largest block table
// and the larger of the growth's and the projection's buffers
constexpr size_t pool_bytes(int rows, int ncol, int nset) {
  const size_t grow = 2 * x_bytes(rows) + w_bytes(rows) + 2 * PAIR_CACHE;
  const size_t proj = proj_bytes(rows, ncol, nset);
  return tab_bytes(rows) + (grow > proj ? grow : proj);
}
constexpr size_t LDS_CU = 160 * 1024, LDS_STATIC = 9 * 1024;  // of a CU, of the kernel's own

// lane -> value index of red16 and red8 below (bit 0 of the lane is free)
__device__ __forceinline__ int red16_index(int lane) {
  return ((lane >> 5) & 1) * 8 + ((lane >> 1) & 1) * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 3) & 1);
}
// 16 values per lane -> this lane's value (red16_index) summed over the lanes
// that share bit 4 with it
__device__ __forceinline__ double red16(double* v, bool b1) {
#pragma unroll
  for (int t = 0; t < 8; ++t) v[t] = swap32_add(v[t], v[t + 8]);
  const double u0 = rs_mirror(v[0], v[1]), u1 = rs_mirror(v[2], v[3]);
  const double u2 = rs_mirror(v[4], v[5]), u3 = rs_mirror(v[6], v[7]);
  const double x0 = rs_half_mirror(u0, u1), x1 = rs_half_mirror(u2, u3);
  const double keep = b1 ? x1 : x0, send = b1 ? x0 : x1;
  double r = keep + dpp_f64<DPP_QUAD_XOR2>(send);
  r += dpp_f64<DPP_QUAD_XOR1>(r);
  return r;
}

// 8 values per lane -> value 4 b5 + 2 b2 + b3 (b_n: bit n of the lane id)
__device__ __forceinline__ int red8_index(int lane) {
  return ((lane >> 5) & 1) * 4 + ((lane >> 2) & 1) * 2 + ((lane >> 3) & 1);
}
__device__ __forceinline__ double red8(double* v) {
#pragma unroll
  for (int t = 0; t < 4; ++t) v[t] = swap32_add(v[t], v[t + 4]);
  double r = rs_half_mirror(rs_mirror(v[0], v[1]), rs_mirror(v[2], v[3]));
  r += dpp_f64<DPP_QUAD_XOR2>(r);
  r += dpp_f64<DPP_QUAD_XOR1>(r);
  return r;
}

// value of lane N of each row of 16, in every lane of the row
template <int N>
__device__ __forceinline__ double row_bcast(double x) {
  return dpp_f64<0x150 + N>(x);
}

__device__ __forceinline__ double lane_value(double v, int src) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), src),
                          __builtin_amdgcn_readlane(__double2loint(v), src));
}

constexpr int DPP_ROW_ROR4 = 0x124;
constexpr int DPP_ROW_ROR8 = 0x128;

// compile-time loop over t (the index reaches templates and register arrays)
template <int I, int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(static_cast<F&&>(f));
  }
}

// q[.][2 T + (tn & 1)] = w in the lanes of `own` if tn / 2 == T (tn uniform).  The
// branches are inside the asm block: as C++ branches, one per basis column, the
// compiler merges their stores, and the basis then lives in scratch memory.
#define MAG_PUT_HEAD               \
  "s_lshr_b32 %[sv], %[tn], 1\n\t" \
  "s_cmp_lg_u32 %[sv], %[t]\n\t"   \
  "s_cbranch_scc1 .Lput%=\n\t"     \
  "s_mov_b64 %[sx], exec\n\t"      \
  "s_and_b64 exec, exec, %[own]\n\t" \
  "s_bitcmp1_b32 %[tn], 0\n\t"     \
  "s_cbranch_scc1 .Lodd%=\n\t"
#define MAG_PUT_MID "s_branch .Lend%=\n.Lodd%=:\n\t"
#define MAG_PUT_TAIL          \
  ".Lend%=:\n\ts_mov_b64 exec, %[sx]\n" \
  ".Lput%=:"
template <int T>
__device__ __forceinline__ void put2(double& a0, double& a1, double& b0, double& b1, double w0,
                                     double w1, int tn, uint64_t own) {
  uint64_t sx;
  uint32_t sv;
  __asm__ volatile(MAG_PUT_HEAD "v_mov_b64 %[a0], %[w0]\n\tv_mov_b64 %[a1], %[w1]\n\t" MAG_PUT_MID
                   "v_mov_b64 %[b0], %[w0]\n\tv_mov_b64 %[b1], %[w1]\n" MAG_PUT_TAIL
                   : [a0] "+v"(a0), [a1] "+v"(a1), [b0] "+v"(b0), [b1] "+v"(b1), [sx] "=&s"(sx),
                     [sv] "=&s"(sv)
                   : [w0] "v"(w0), [w1] "v"(w1), [tn] "s"(tn), [t] "n"(T), [own] "s"(own)
                   : "scc");
}
template <int T>
__device__ __forceinline__ void put3(double& a0, double& a1, double& a2, double& b0, double& b1,
                                     double& b2, double w0, double w1, double w2, int tn,
                                     uint64_t own) {
  uint64_t sx;
  uint32_t sv;
  __asm__ volatile(MAG_PUT_HEAD
                   "v_mov_b64 %[a0], %[w0]\n\tv_mov_b64 %[a1], %[w1]\n\t"
                   "v_mov_b64 %[a2], %[w2]\n\t" MAG_PUT_MID
                   "v_mov_b64 %[b0], %[w0]\n\tv_mov_b64 %[b1], %[w1]\n\t"
                   "v_mov_b64 %[b2], %[w2]\n" MAG_PUT_TAIL
                   : [a0] "+v"(a0), [a1] "+v"(a1), [a2] "+v"(a2), [b0] "+v"(b0), [b1] "+v"(b1),
                     [b2] "+v"(b2), [sx] "=&s"(sx), [sv] "=&s"(sv)
                   : [w0] "v"(w0), [w1] "v"(w1), [w2] "v"(w2), [tn] "s"(tn), [t] "n"(T),
                     [own] "s"(own)
                   : "scc");
}
#undef MAG_PUT_HEAD
#undef MAG_PUT_MID
#undef MAG_PUT_TAIL

// a value that is the same in every lane, in a scalar register: conditions on
// it become scalar branches.  (They have to: where a lane-masked region ends
// together with one that encloses it, the compiler has been seen to reload a
// spilled basis register under the inner mask.)  Scalar branches around the
// places where a vector enters the basis make it spill the basis instead (nu =
// 30, 160 atoms: 195 registers against 35), so there what a column does follows
// from selects.
__device__ __forceinline__ int uni(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ int64_t uni(int64_t v) {
  return ((int64_t)uni((int)(v >> 32)) << 32) | (uint32_t)uni((int)v);
}

// hides a lane constant's origin, so that what is computed from it stays where
// it is used (hoisted out of the loops it would be kept in scratch memory)
__device__ __forceinline__ int opaque(int v) {
  __asm__ volatile("" : "+v"(v));
  return v;
}
// loads with the memory named: a value that comes from LDS on one path and
// from global memory on another would otherwise be read by flat loads, which
// wait for both
__device__ __forceinline__ double ld_lds(const char* p) {
  return *(const __attribute__((address_space(3))) double*)p;
}
__device__ __forceinline__ double2 ld_lds2(const char* p) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 v = *(const __attribute__((address_space(3))) v2*)p;
  return make_double2(v.x, v.y);
}
__device__ __forceinline__ double2 ld_glb2(const char* p) {
  typedef double v2 __attribute__((ext_vector_type(2)));
  const v2 v = *(const __attribute__((address_space(1))) v2*)p;
  return make_double2(v.x, v.y);
}

// what a step tells the whole workgroup about a column
enum : int { ST_DONE = 0, ST_GO = 1, ST_AGAIN = 2 };

template <int NU, int NCOL, int RPL, bool ADJ>
__global__ __launch_bounds__(KTPB) void krylov_kernel(KrylovArgs a) {
  constexpr int WPC = KW / NCOL;        // waves of a column
  constexpr int LROWS = 32 * WPC;       // row-lanes of a column
  constexpr int ROWS = LROWS * RPL;     // cluster rows held
  constexpr int NB = NU / 2;            // basis vectors of a lane
  constexpr int NSET = NB / 16 + 1;     // sets of sixteen reduced values (slot 15: the norm)
  constexpr int XB = (int)x_bytes(ROWS);
  constexpr int PL = x_plane(ROWS);
  constexpr int CB = PROJ_CB;
  constexpr int PA = proj_atom(ROWS, NCOL);   // bytes of an atom's vectors
  constexpr int PQ = NCOL * CB * 16;    // ... of one orbital pair
  constexpr int TPW = tiles_per_wave(ROWS);
  static_assert(NU % 2 == 0, "even and odd vectors");
  static_assert(pool_bytes(ROWS, NCOL, NSET) + LDS_STATIC <= LDS_CU, "LDS of a CU");
  __shared__ int32_t s_atoms[CLUSTER_MAX];
  __shared__ int32_t s_brow[CLUSTER_MAX];   // first global block of each cluster atom's row
  __shared__ __attribute__((aligned(16))) uint16_t s_key[CLUSTER_MAX];
  __shared__ uint8_t s_pos[CLUSTER_MAX];    // rank of each cluster atom
  __shared__ uint8_t s_orig[CLUSTER_MAX];   // cluster atom of each rank
  // blocks of each rank's row inside the cluster
  __shared__ __attribute__((aligned(16))) uint8_t s_len[CLUSTER_MAX];
  __shared__ uint8_t s_blen[CLUSTER_MAX];   // blocks of each cluster atom's global row
  __shared__ int16_t s_patb[CLUSTER_MAX];   // position of the rank's atom in J's block row, or -1
  __shared__ ushort2 s_tile[TILE_MAX];      // first unit in the table, pairs of blocks
  __shared__ double s_red[NCOL][WPC][2][16 * NSET];
  __shared__ double s_part[2][2][KW];       // (q^T w, |w|^2) x column x wave
  __shared__ int s_ubase[KW];               // first unit of each wave
  __shared__ int s_ctl[2];
  __shared__ int s_misc[8];
  // (16-byte reads: off that boundary they are many times slower)
  extern __shared__ __attribute__((aligned(128))) double s_pool[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int cap = a.cap;
  int q = a.queue ? (int)(blockIdx.x % (unsigned)a.nqueue) : 0;
  int tried = 0;
  // a queue hands out the NORB columns of an atom together while more than
  // that remains for every workgroup of the queue, then pairs, then single
  // columns
  const int64_t wgq = a.queue ? (int64_t)(gridDim.x / a.nqueue + 1) : 0;
  // basis lanes
  const int col = NCOL == 2 ? wave / WPC : 0;
  const int wv = NCOL == 2 ? wave % WPC : wave;
  const int g = (lane >> 4) & 1;
  const int p0 = wv * 32 + (lane >> 5) * 16 + (lane & 15);
  int tabJ = -1;  // atom whose cluster tables the LDS holds (-1: none)
  const char* bval = reinterpret_cast<const char*>(a.bval);

  for (int64_t it = 0;; ++it) {
    int64_t base;
    int count;
    if (a.queue) {
      if (tid == 0) {
        int64_t sl = -1;
        int n = 0;
        while (tried < a.nqueue) {
          const int64_t qb = a.qbeg[q], qe = a.qbeg[q + 1];
          const int64_t left = qe - (qb + atomicAdd(&a.queue[q], 0));
          const int gsz = (left > 2 * NORB * wgq) ? NORB : ((left > wgq) ? NCOL : 1);
          const int64_t cand = qb + atomicAdd(&a.queue[q], gsz);
          if (cand < qe) {
            sl = cand;
            n = (int)min((int64_t)gsz, qe - cand);
            break;
          }
          q = (q + 1) % a.nqueue;
          ++tried;
        }
        s_misc[0] = (int)sl;
        s_misc[2] = n;
      }
      __syncthreads();
      base = uni(s_misc[0]);
      count = uni(s_misc[2]);
      __syncthreads();
      if (base < 0) break;
    } else {
      if (it > 0) break;
      // the first workgroups take the first position of each group and those
      // after it of the same atom, the others one of the rest, if it is still to
      // be done
      const int64_t ngr = (a.ncols + a.group - 1) / a.group;
      const int64_t rest = (int64_t)blockIdx.x - ngr;
      base = rest < 0 ? (int64_t)blockIdx.x * a.group
                      : rest / (a.group - 1) * a.group + 1 + rest % (a.group - 1);
      if (base >= a.ncols) break;
      auto atom = [&](int64_t p) { return uni(a.cols[a.slots ? (int64_t)a.slots[p] : p]) >> 2; };
      const int64_t first = base / a.group * a.group;
      const int64_t last = min(first + a.group, a.ncols);
      const int J0 = atom(first);
      int64_t end = first + 1;
      while (end < last && atom(end) == J0) ++end;
      if (base != first && base < end) break;
      count = base == first ? (int)(end - first) : 1;
    }
    if (base >= a.ncols) break;

    for (int u = 0; u < count;) {
      // the next column, and the one after it if it belongs to the same atom
      int64_t slots[2] = {base + u, -1};
      if (a.slots) slots[0] = uni(a.slots[slots[0]]);
      const int j0 = uni(a.cols[slots[0]]);
      const int J = j0 >> 2;
      int jc[2] = {j0, j0};
      int nact = 1;
      if (NCOL == 2 && u + 1 < count) {
        const int64_t s1 = a.slots ? (int64_t)uni(a.slots[base + u + 1]) : base + u + 1;
        const int j1 = uni(a.cols[s1]);
        if ((j1 >> 2) == J) {
          slots[1] = s1;
          jc[1] = j1;
          nact = 2;
        }
      }
      u += nact;
      const int64_t c0 = uni(a.clus_ptr[J]);
      const int nat = uni((int)(a.clus_ptr[J + 1] - c0));
      const int nC = NORB * nat;
      if (nat > CLUSTER_MAX || nC > ROWS || nat <= 0) {
        if (tid == 0) {
          atomicOr(a.err, (int)KERR_CAPACITY);
          for (int i = 0; i < nact; ++i) a.nu_eff[slots[i]] = 0;
        }
        continue;
      }
      const int ntile = (nat + 3) >> 2;
      const int nbJ = uni(a.bptr[J + 1] - a.bptr[J]);

      if (J != tabJ) {
        // ---- prologue: cluster atoms and their block rows (gather of H_C,
        // S_C).  A half wave reads one global block row, one block per lane,
        // looks the column atoms up in a hash of the cluster, and the ballot
        // of the hits places them.
        tabJ = -1;
        __syncthreads();  // the pool may still hold the last column's data
        int32_t* s_hk = reinterpret_cast<int32_t*>(s_pool);
        int32_t* s_hv = s_hk + HASH;
        for (int i = tid; i < HASH; i += KTPB) s_hk[i] = -1;
        if (tid < CLUSTER_MAX) {
          s_key[tid] = 0;
          s_patb[tid] = -1;
          s_len[tid] = 0;
          s_blen[tid] = 0;
        }
        __syncthreads();
        const int ptid = opaque(tid);
        if (ptid < nat) {
          const int I = a.clus_atoms[c0 + ptid];
          const int b0 = a.bptr[I];
          s_atoms[ptid] = I;
          s_brow[ptid] = b0;
          s_blen[ptid] = (uint8_t)(a.bptr[I + 1] - b0);
        }
        if (ptid == 0) s_misc[1] = -1;
        __syncthreads();
        if (ptid < nat) {
          const int I = s_atoms[ptid];
          unsigned hs = ((unsigned)I * 2654435761u) >> 23;
          for (;;) {
            const int old = atomicCAS(&s_hk[hs], -1, I);
            if (old == -1) break;
            hs = (hs + 1) & (HASH - 1);
          }
          s_hv[hs] = ptid;
          if (I == J) s_misc[1] = ptid;
        }
        constexpr int NQ = ROWS / 64;
        const int hw = ptid >> 5, l32 = ptid & 31;
        int kl[NQ];
#pragma unroll
        for (int qq = 0; qq < NQ; ++qq) {
          const int i = hw + 16 * qq;
          kl[qq] = -1;
          if (i < nat && l32 < (int)s_blen[i]) kl[qq] = a.bcol[s_brow[i] + l32];
        }
        __syncthreads();
#pragma unroll
        for (int qq = 0; qq < NQ; ++qq) {
          const int key = kl[qq];
          int found = -1;
          if (key >= 0) {
            unsigned hs = ((unsigned)key * 2654435761u) >> 23;
            for (;;) {
              const int k2 = s_hk[hs];
              if (k2 == key) {
                found = s_hv[hs];
                break;
              }
              if (k2 < 0) break;
              hs = (hs + 1) & (HASH - 1);
            }
          }
          kl[qq] = found;
        }
#pragma unroll
        for (int qq = 0; qq < NQ; ++qq) {
          const int i = hw + 16 * qq;
          const unsigned mask = (unsigned)(__ballot(kl[qq] >= 0) >> (ptid & 32));
          if (l32 == 0 && i < nat) s_key[i] = (uint16_t)((__popc(mask) << 8) | (255 - i));
        }
        __syncthreads();
        // rank of each atom by blocks (descending), ties by cluster order
        if (ptid < 2 * CLUSTER_MAX) {
          const int i = ptid >> 1;
          const int key = s_key[i];
          const uint4* kp = reinterpret_cast<const uint4*>(s_key) + (ptid & 1) * (CLUSTER_MAX / 16);
          int r = 0;
#pragma unroll 4
          for (int v = 0; v < CLUSTER_MAX / 16; ++v) {
            const uint4 k8 = kp[v];
            r += ((int)(k8.x & 0xffff) > key) + ((int)(k8.x >> 16) > key);
            r += ((int)(k8.y & 0xffff) > key) + ((int)(k8.y >> 16) > key);
            r += ((int)(k8.z & 0xffff) > key) + ((int)(k8.z >> 16) > key);
            r += ((int)(k8.w & 0xffff) > key) + ((int)(k8.w >> 16) > key);
          }
          r += __shfl_xor(r, 1, 64);
          if ((ptid & 1) == 0 && i < nat) {
            s_pos[i] = (uint8_t)r;
            s_orig[r] = (uint8_t)i;
            s_len[r] = (uint8_t)(key >> 8);
          }
        }
        __syncthreads();
        const int jl = uni(s_misc[1]);
        const int nbJl = jl >= 0 ? uni((int)(s_key[jl] >> 8)) : -1;
        // tiles: their units (two pairs of blocks) follow each other in the
        // table, wave after wave (tile t belongs to wave t % KW), a few dummy
        // units after each wave's.  Lane t computes tile t; every lane reads
        // all lengths.
        if (wave == 0) {
          const int pl = opaque(lane);
          const uint4* lp = reinterpret_cast<const uint4*>(s_len);
          int ub = (pl % KW) * PAD_UNITS, nun = KW * PAD_UNITS, mynp = 0;
          unsigned ne = 0;
#pragma unroll 2
          for (int v = 0; v < CLUSTER_MAX / 16; ++v) {
            const uint4 l4 = lp[v];
            const unsigned d[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const int t = 4 * v + c;
              const int np = (int)((d[c] & 255) + 1) >> 1;
              const int un = (np + 1) >> 1;
              if (t % KW < pl % KW || (t % KW == pl % KW && t < pl)) ub += un;
              if (t == pl) mynp = np;
              nun += un;
              ne = __builtin_amdgcn_sad_u8(d[c], 0, ne);
            }
          }
          if (pl < ntile) s_tile[pl] = make_ushort2((unsigned short)ub, (unsigned short)mynp);
          if (pl == 0) {
            s_misc[3] = nun;
            s_misc[4] = (int)ne;
          }
          if (pl < KW) s_ubase[pl] = ub;  // tile w is the first of wave w
        }
        __syncthreads();
        const int nent = uni(s_misc[4]);
        if (nent > ENT_MAX || jl < 0 || nbJl != nbJ) {
          if (tid == 0) {
            atomicOr(a.err, (int)(nent > ENT_MAX ? KERR_CAPACITY : KERR_PATTERN));
            a.nu_eff[slots[0]] = 0;
            if (nact > 1) a.nu_eff[slots[1]] = 0;
          }
          __syncthreads();
          continue;
        }
        // table entries; a row that ends before its tile is filled up with the
        // zero operand past the last row
        uint32_t* tabw = reinterpret_cast<uint32_t*>(s_pool);
        constexpr uint32_t DUMMY = (uint32_t)(ROWS / 4) * 32 * 0x10001u;
        for (int i = ptid; i < s_misc[3] * (TAB_UNIT / 4); i += KTPB)
          tabw[i] = i % (TAB_UNIT / 4) < TAB_B / 4 ? DUMMY : 0u;
        __syncthreads();
        uint16_t* tab16 = reinterpret_cast<uint16_t*>(s_pool);
#pragma unroll
        for (int qq = 0; qq < NQ; ++qq) {
          const int i = hw + 16 * qq;
          const unsigned mask = (unsigned)(__ballot(kl[qq] >= 0) >> (ptid & 32));
          if (kl[qq] >= 0) {
            const int ps = s_pos[i], pk = s_pos[kl[qq]];
            const int e = __popc(mask & ((1u << l32) - 1u));
            const int un = (int)s_tile[ps >> 2].x + (e >> 2);
            tab16[un * (TAB_UNIT / 2) + (ps & 3) * 4 + (e & 1) * 2 + ((e >> 1) & 1)] =
                (uint16_t)(pk * 32);
            tabw[un * (TAB_UNIT / 4) + TAB_B / 4 + (ps & 3) * 4 + (e & 1) * 2 + ((e >> 1) & 1)] =
                (uint32_t)(s_brow[i] + l32) * 16u;
            if (i == jl) s_patb[pk] = (int16_t)l32;
          }
        }
        tabJ = J;
        __syncthreads();
      }
      const int jl = uni(s_misc[1]);
      const int ebytes = uni(s_misc[3]) * TAB_UNIT;
      const char* tab = reinterpret_cast<const char*>(s_pool);
      char* U = reinterpret_cast<char*>(s_pool) + ebytes;
      char* s_x = U;
      double* s_w = reinterpret_cast<double*>(U + 2 * XB);
      char* s_cache = U + 2 * XB + w_bytes(ROWS);
      const int ellr = NORB * uni((int)s_pos[jl]);  // row of the atom's first orbital

      // ---- operands: both buffers and the product zero, q_0 = e_l
      for (int i = opaque(tid); i < 2 * XB / 8; i += KTPB) reinterpret_cast<double*>(s_x)[i] = 0.0;
      for (int i = opaque(tid); i < NCOL * ROWS; i += KTPB) s_w[i] = 0.0;
      // The wave's units in order, and which of them end a tile; the first ones
      // stay in the wave's share of the LDS, the others stream
      uint64_t uend = 0;
      int nun = 0;
#pragma unroll
      for (int ti = 0; ti < TPW; ++ti) {
        const int t = wave + ti * KW;
        if (t < ntile) {
          nun += (__builtin_amdgcn_readfirstlane((int)s_tile[t].y) + 1) >> 1;
          uend |= 1ull << (nun - 1);
        }
      }
      const char* tabu = tab + __builtin_amdgcn_readfirstlane(s_ubase[wave]) * TAB_UNIT;
      const int room = (int)(a.pool - ebytes - 2 * XB - (int)w_bytes(ROWS));
      const int share = min(a.cache_cap, max(room - 2 * PAIR_CACHE, 0) / (2 * PAIR_CACHE)) /
                        KW;  // units of a wave
      s_cache += wave * share * 2 * PAIR_CACHE;
      const int ncu = min(share, nun);
      // blocks of unit un in the lanes' places; w: 0 for H, 128 for S
      auto unit_blocks = [&](double2(&v)[2], int un, int la, int w) __attribute__((always_inline)) {
        const uint2 e = *reinterpret_cast<const uint2*>(tabu + TAB_B + un * TAB_UNIT +
                                                        ((la >> 1) & 6) * 8 + (la >> 5) * 8);
        const char* hp = bval + (((la >> 4) & 1) * 64 + (la & 3) * 16 + w);
        v[0] = ld_glb2(hp + ((uint64_t)e.x << 4));
        v[1] = ld_glb2(hp + ((uint64_t)e.y << 4));
      };
      {
        const int la = opaque(lane);
        double2* cd = reinterpret_cast<double2*>(s_cache) + la;
        for (int c = 0; c < ncu; c += 4) {
          double2 v[4][2];
#pragma unroll
          for (int e = 0; e < 4; ++e) unit_blocks(v[e], min(c + e, ncu - 1), la, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            if (c + e < ncu) {
              cd[(c + e) * 128] = v[e][0];
              cd[(c + e) * 128 + 64] = v[e][1];
            }
          }
        }
      }
      __syncthreads();
      if (tid < nact) {
        const int ell = ellr + ((tid == 0 ? jc[0] : jc[1]) & 3);
        *reinterpret_cast<double*>(s_x + ((ell >> 1) & 1) * PL + (ell >> 2) * 32 + tid * 16 +
                                   (ell & 1) * 8) = 1.0;
      }

      double qv[RPL][NB];
      const int64_t slot = (NCOL == 2 && col == 1) ? slots[1] : slots[0];
      const bool mine = slot >= 0;
      const int myell = ellr + (((NCOL == 2 && col == 1) ? jc[1] : jc[0]) & 3);
#pragma unroll
      for (int m = 0; m < RPL; ++m) {
#pragma unroll
        for (int t = 0; t < NB; ++t) qv[m][t] = 0.0;
        if (mine && g == 0 && p0 + LROWS * m == myell) qv[m][0] = 1.0;
      }
      const int nu_max = min(a.nu, nC);
      int nu_eff = nu_max;
      bool act = mine;
      double beta_prev = 0.0;
      double* hcol = a.hs + slot * (int64_t)(2 * cap * cap);
      double* scol = hcol + cap * cap;
      __syncthreads();

      // Gram-Schmidt pieces, on the basis columns 0 .. k: the dots of w (and
      // |w|^2) of this wave into s_red, then the column's totals (slot = value
      // of the lane's row) and w -= Q c, |c|^2
      // (up to 7 vectors of a lane: eight values reduced, else sixteen; the
      // last slot is the norm)
      auto dots = [&](const double(&w)[RPL], int k, double* rd,
                      auto norm) __attribute__((always_inline)) {
        double nn = 0.0;
#pragma unroll
        for (int m = 0; m < RPL; ++m)
          if (decltype(norm)::value) nn = fma(w[m], w[m], nn);
        auto dot = [&](int t) __attribute__((always_inline)) {
          double d = 0.0;
          if (t < NB) {
            d = qv[0][t < NB ? t : 0] * w[0];
#pragma unroll
            for (int m = 1; m < RPL; ++m) d = fma(qv[m][t < NB ? t : 0], w[m], d);
          }
          return d;
        };
        const int la = opaque(lane);
        if (k < 14) {
          double v[8];
#pragma unroll
          for (int t = 0; t < 7; ++t) v[t] = dot(t);
          v[7] = nn;
          const double r = red8(v);
          rd[red8_index(la)] = r;  // (the lanes that share a place hold the same value)
        } else {
          double v[16];
#pragma unroll
          for (int t = 0; t < 11; ++t) v[t] = dot(t);
          if (k >= 22) {
#pragma unroll
            for (int t = 11; t < 15; ++t) v[t] = dot(t);
          } else {
            v[11] = v[12] = v[13] = v[14] = 0.0;
          }
          v[15] = nn;
          const double r = red16(v, (la & 2) != 0);
          rd[red16_index(la)] = r;
          if constexpr (NSET > 1) {
            if (k >= 30) {
#pragma unroll
              for (int t = 0; t < 16; ++t) v[t] = dot(15 + t);
              const double r1 = red16(v, (la & 2) != 0);
              rd[16 + red16_index(la)] = r1;
            }
          }
        }
      };
      auto totals = [&](double(&hv)[NSET], int k) __attribute__((always_inline)) {
        const int la = opaque(lane);
        const double* rp = &s_red[NCOL == 2 ? col : 0][0][g][0] + (la & (k < 14 ? 7 : 15));
#pragma unroll
        for (int set = 0; set < NSET; ++set) {
          hv[set] = 0.0;
          if (set == 0 || k >= 30) {
            double acc = rp[set * 16];
#pragma unroll
            for (int v = 1; v < WPC; ++v) acc += rp[v * 2 * 16 * NSET + set * 16];
            hv[set] = acc;
          }
        }
      };
      auto subtract = [&](double(&w)[RPL], const double(&hv)[NSET], int k) __attribute__((always_inline)) {
        double csq = (opaque(lane) & 15) < (k < 14 ? 7 : 15) ? hv[0] * hv[0] : 0.0;
        if (NSET > 1) csq = fma(hv[NSET - 1], hv[NSET - 1], csq);
        double s[RPL];
#pragma unroll
        for (int m = 0; m < RPL; ++m) s[m] = 0.0;
        auto add = [&](auto ti) __attribute__((always_inline)) {
          constexpr int t = decltype(ti)::value;
          const double c = row_bcast<(t < 15 ? t : t - 15)>(hv[t < 15 ? 0 : NSET - 1]);
#pragma unroll
          for (int m = 0; m < RPL; ++m) s[m] = fma(qv[m][t], c, s[m]);
        };
        static_for<0, (NB < 7 ? NB : 7)>(add);
        if constexpr (NB > 7) {
          if (k >= 14) static_for<7, (NB < 11 ? NB : 11)>(add);
        }
        if constexpr (NB > 11) {
          if (k >= 22) static_for<11, (NB < 15 ? NB : 15)>(add);
        }
        if constexpr (NB > 15) {
          if (k >= 30) static_for<15, NB>(add);
        }
#pragma unroll
        for (int m = 0; m < RPL; ++m) w[m] -= swap16_add(s[m], s[m]);
        csq = row_allreduce(csq);
        return swap16_add(csq, csq);
      };
      // q_cn = w into its register column (none of them unless put) and, in the
      // lanes of `own_x`, the operand buffer xb
      auto store_q = [&](const double(&w)[RPL], int cn, bool put, bool own_x,
                         char* xb) __attribute__((always_inline)) {
        const int tn = __builtin_amdgcn_readfirstlane(put ? cn >> 1 : NU);
        const uint64_t own = (cn & 1) ? 0xffff0000ffff0000ull : 0x0000ffff0000ffffull;
        static_for<0, (NB + 1) / 2>([&](auto ti) __attribute__((always_inline)) {
          constexpr int T = decltype(ti)::value, t0 = 2 * T;
          constexpr int n3 = RPL % 2 ? 3 : 0;  // rows 0-2 together when RPL is odd
          double none[3];  // the odd column past the last one
          auto odd = [&](int m) __attribute__((always_inline)) -> double& {
            return t0 + 1 < NB ? qv[m][t0 + 1 < NB ? t0 + 1 : t0] : none[m % 3];
          };
          if constexpr (t0 + 1 >= NB) none[0] = none[1] = none[2] = 0.0;
          if constexpr (n3 == 3)
            put3<T>(qv[0][t0], qv[1][t0], qv[2][t0], odd(0), odd(1), odd(2), w[0], w[1], w[2], tn,
                    own);
          if constexpr (RPL - n3 >= 2)
            put2<T>(qv[n3][t0], qv[n3 + 1][t0], odd(n3), odd(n3 + 1), w[n3], w[n3 + 1], tn, own);
          if constexpr (RPL - n3 >= 4)
            put2<T>(qv[n3 + 2][t0], qv[n3 + 3][t0], odd(n3 + 2), odd(n3 + 3), w[n3 + 2],
                    w[n3 + 3], tn, own);
          if constexpr (RPL - n3 >= 6)
            put2<T>(qv[n3 + 4][t0], qv[n3 + 5][t0], odd(n3 + 4), odd(n3 + 5), w[n3 + 4],
                    w[n3 + 5], tn, own);
        });
        if (own_x) {
          const int pr = opaque(p0);
          char* xo = xb + ((pr >> 1) & 1) * PL + (pr >> 2) * 32 + (NCOL == 2 ? col : 0) * 16 +
                     (pr & 1) * 8;
#pragma unroll
          for (int m = 0; m < RPL; ++m) *reinterpret_cast<double*>(xo + LROWS * m * 8) = w[m];
        }
      };
      // the residual of a column's last step for the exact gradient
      auto store_last = [&](const double(&w)[RPL], bool last) __attribute__((always_inline)) {
        if (g == 0 && last) {
#pragma unroll
          for (int m = 0; m < RPL; ++m) {
            const int r = p0 + LROWS * m;
            if (r < nC)
              a.adj_r[slot * (int64_t)a.adj_rows + NORB * s_orig[r >> 2] + (r & 3)] = w[m];
          }
        }
      };

      // the next basis vector from the orthogonalized w, if the column goes on
      auto advance = [&](double(&w)[RPL], double b2, int k, bool go, bool own_x)
          __attribute__((always_inline)) {
        const double inv = go ? rsqrt(b2) : 1.0;
        beta_prev = go ? b2 * inv : beta_prev;
        if (ADJ && go && wv == 0 && lane == 0) a.adj_beta[slot * (int64_t)cap + k] = beta_prev;
#pragma unroll
        for (int m = 0; m < RPL; ++m) w[m] *= inv;
        store_q(w, k + 1, go, own_x, s_x + ((k & 1) ^ 1) * XB);
      };
      // a condition that all lanes share, as a scalar up to nu = 30; beyond that it
      // stays in the lanes (forces of 3,600 atoms at nu = 40: 16.0 against 16.3 ms)
      auto any = [](bool c) { return NU > 30 ? c : __builtin_amdgcn_ballot_w64(c) != 0; };
      bool more = true;
      for (int k = 0; k < nu_max && more; ++k) {
        char* xb = s_x + (k & 1) * XB;
        // ---- w = H_C q_k for both columns, tile by tile
        {
          double al = 0.0, ww = 0.0;
          const int la = opaque(lane);
          const int x = la & 3, b = (la >> 2) & 3, y = la >> 4;
          const char* xl = xb + (y & 1) * PL + (x & 1) * 16;
          const char* tp = tabu + (b * 2 + (y >> 1)) * 4;
          const char* ch = s_cache + la * 16;
          auto words = [&](int i) __attribute__((always_inline)) {
            return *(const __attribute__((address_space(3))) uint32_t*)(tp + i * TAB_UNIT);
          };
          auto xload = [&](double2(&v)[2], uint32_t wd) __attribute__((always_inline)) {
            v[0] = ld_lds2(xl + (wd & 0xffffu));
            v[1] = ld_lds2(xl + (wd >> 16));
          };
          // the first streamed units are on their way while the cached ones
          // are used
          double2 hs[RING][2];
#pragma unroll
          for (int i = 0; i < RING; ++i)
            if (ncu + i < nun) unit_blocks(hs[i], ncu + i, la, 0);
          double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
          // the running tile's own operand and product rows
          const char* xk = xb + (y >> 1) * PL + (4 * wave + b) * 32 + (x & 1) * 16 + (y & 1) * 8;
          double* wp = s_w + (x & 1) * ROWS + 16 * wave + 4 * b + y;
          uint64_t fend = uend;
          auto unit = [&](const double2(&h)[2], const double2(&v)[2]) __attribute__((always_inline)) {
            a0 = __builtin_amdgcn_mfma_f64_4x4x4f64(h[0].x, v[0].x, a0, 0, 0, 0);
            a1 = __builtin_amdgcn_mfma_f64_4x4x4f64(h[0].y, v[0].y, a1, 0, 0, 0);
            a2 = __builtin_amdgcn_mfma_f64_4x4x4f64(h[1].x, v[1].x, a2, 0, 0, 0);
            a3 = __builtin_amdgcn_mfma_f64_4x4x4f64(h[1].y, v[1].y, a3, 0, 0, 0);
            if (fend & 1) {  // the tile's last unit
              const double wr = (a0 + a1) + (a2 + a3);
              const double xv = ld_lds(xk);
              al = fma(wr, xv, al);
              ww = fma(wr, wr, ww);
              *wp = wr;  // (lanes x and x + 2 write the same value)
              a0 = a1 = a2 = a3 = 0.0;
              xk += KW * 128;
              wp += KW * 16;
            }
            fend >>= 1;
          };
          // operands and cached blocks one unit ahead, table entries two
          double2 xa[2], xc[2], ha[2], hc[2];
          uint32_t wn = words(0);
          xload(xa, wn);
          wn = words(1);
          tp += 2 * TAB_UNIT;
          ha[0] = ld_lds2(ch);
          ha[1] = ld_lds2(ch + PAIR_CACHE);
          int un = 0;
          for (; un + 1 < ncu; un += 2) {
            xload(xc, wn);
            wn = words(0);
            hc[0] = ld_lds2(ch + 2 * PAIR_CACHE);
            hc[1] = ld_lds2(ch + 3 * PAIR_CACHE);
            __builtin_amdgcn_sched_barrier(0);
            unit(ha, xa);
            xload(xa, wn);
            wn = words(1);
            ha[0] = ld_lds2(ch + 4 * PAIR_CACHE);
            ha[1] = ld_lds2(ch + 5 * PAIR_CACHE);
            __builtin_amdgcn_sched_barrier(0);
            unit(hc, xc);
            tp += 2 * TAB_UNIT;
            ch += 4 * PAIR_CACHE;
          }
          if (un < ncu) {
            unit(ha, xa);
            xload(xa, wn);
            wn = words(0);
            tp += TAB_UNIT;
            ++un;
          }
          for (; un < nun; un += RING) {
#pragma unroll
            for (int i = 0; i < RING; ++i) {
              if (un + i < nun) {
                xload((i & 1) ? xa : xc, wn);
                wn = words(i);
                __builtin_amdgcn_sched_barrier(0);
                unit(hs[i], (i & 1) ? xc : xa);
                if (un + i + RING < nun) unit_blocks(hs[i], un + i + RING, la, 0);
              }
            }
            tp += RING * TAB_UNIT;
          }
          // q_k^T w and |w|^2 of each column over the wave's tiles
          double v = swap32_add(al, ww);
          v = swap16_add(v, v);
          v += dpp_f64<DPP_ROW_ROR8>(v);
          v += dpp_f64<DPP_ROW_ROR4>(v);
          if ((lane & 31) < 2) s_part[lane >> 5][lane & 1][wave] = v;
        }
        __syncthreads();

        // ---- local subtraction, then full Gram-Schmidt passes: one, and more
        // only for a column whose pass removed more than half of |w|^2
        double w[RPL];
        double alpha = 0.0, ww1 = 0.0;
        {
          const char* xo = s_x + ((k & 1) ^ 1) * XB;
          const int la = opaque(lane);
          double pt = s_part[(la >> 3) & 1][NCOL == 2 ? col : 0][la & 7];
          pt += dpp_f64<DPP_ROW_HALF_MIRROR>(pt);
          pt += dpp_f64<DPP_QUAD_XOR2>(pt);
          pt += dpp_f64<DPP_QUAD_XOR1>(pt);
          alpha = lane_value(pt, 0);
          ww1 = lane_value(pt, 8);
          const int pr = opaque(p0);
          const int xr = ((pr >> 1) & 1) * PL + (pr >> 2) * 32 + (NCOL == 2 ? col : 0) * 16 +
                         (pr & 1) * 8;
          const char* xko = xb + xr;
          const char* xpo = xo + xr;
          const double* wp = s_w + (NCOL == 2 ? col : 0) * ROWS + pr;
#pragma unroll
          for (int m = 0; m < RPL; ++m) {
            const double xk = ld_lds(xko + LROWS * m * 8);
            const double xp = ld_lds(xpo + LROWS * m * 8);
            w[m] = fma(-beta_prev, xp, fma(-alpha, xk, wp[LROWS * m]));
          }
        }
        int st = ST_DONE;
        double hv[NSET], norm = 0.0, beta2 = 0.0;
        double* red = &s_red[NCOL == 2 ? col : 0][wv][g][0];
        if (act) dots(w, k, red, std::true_type{});
        __syncthreads();
        if (act) {
          totals(hv, k);
          norm = lane_value(hv[0], k < 14 ? 7 : 15);
          if (wv == 0 && lane < 32) {
#pragma unroll
            for (int set = 0; set < NSET; ++set) {
              const int sl = lane & 15;
              const int i = 2 * (set == 0 ? sl : 15 + sl) + g;
              if ((set > 0 || sl < (k < 14 ? 7 : 15)) && i <= k) {
                double hval = hv[set];
                if (i == k) hval += alpha;
                if (i + 1 == k) hval += beta_prev;
                hcol[(int64_t)k * cap + i] = hval;
                if (ADJ) a.adj_h[slot * (int64_t)cap * cap + (int64_t)k * cap + i] = hval;
              }
            }
          }
          beta2 = norm - subtract(w, hv, k);
          const bool finite = isfinite(ww1);
          if (!finite && wv == 0 && lane == 0) atomicOr(a.err, (int)KERR_NONFINITE);
          const bool half = !(beta2 > 0.5 * norm);
          const bool small = !(beta2 > a.breakdown * a.breakdown * ww1);
          st = any(!finite) || k + 1 >= nu_max
                   ? (int)ST_DONE
                   : (any(half) ? (int)ST_AGAIN : (any(small) ? (int)ST_DONE : (int)ST_GO));
          advance(w, beta2, k, st == ST_GO, g == 0 && st == ST_GO);
          nu_eff = st == ST_DONE ? k + 1 : nu_eff;
          if (ADJ) store_last(w, st == ST_DONE);
        }
        if (wv == 0 && lane == 0) s_ctl[NCOL == 2 ? col : 0] = st;
        __syncthreads();
        int c_0 = __builtin_amdgcn_readfirstlane(s_ctl[0]);
        int c_1 = NCOL == 2 ? __builtin_amdgcn_readfirstlane(s_ctl[1]) : (int)ST_DONE;
        if (__builtin_expect(c_0 == ST_AGAIN || c_1 == ST_AGAIN, 0)) {
          // rare: almost invariant spaces.  The partner's w goes along, unused
          const bool again = (NCOL == 2 && col == 1 ? c_1 : c_0) == ST_AGAIN;
          for (int pass = 0; pass < 2; ++pass) {
            dots(w, k, red, std::true_type{});
            __syncthreads();
            totals(hv, k);
            norm = lane_value(hv[0], k < 14 ? 7 : 15);
            beta2 = norm - subtract(w, hv, k);
            __syncthreads();
          }
          const int go = any(beta2 > a.breakdown * a.breakdown * ww1) ? (int)ST_GO : (int)ST_DONE;
          st = again ? go : st;
          advance(w, beta2, k, again && st == ST_GO, again && g == 0);
          nu_eff = again && st == ST_DONE ? k + 1 : nu_eff;
          if (ADJ) store_last(w, again && st == ST_DONE);
          if (wv == 0 && lane == 0) s_ctl[NCOL == 2 ? col : 0] = st;
          __syncthreads();
          c_0 = __builtin_amdgcn_readfirstlane(s_ctl[0]);
          c_1 = NCOL == 2 ? __builtin_amdgcn_readfirstlane(s_ctl[1]) : (int)ST_DONE;
        }
        act = (NCOL == 2 && col == 1 ? c_1 : c_0) == ST_GO;
        more = c_0 == ST_GO || c_1 == ST_GO;
      }

      // ---- nu_eff, row l of Q, the pattern (or all) rows of Q, and the
      // whole basis for the exact gradient
      if (mine) {
        if (wv == 0 && lane == 0) {
          a.nu_eff[slot] = nu_eff;
          if (a.npat) a.npat[slot] = a.full ? nC : NORB * nbJ;
        }
        const int pr = opaque(p0);
#pragma unroll
        for (int m = 0; m < RPL; ++m) {
          const int r = pr + LROWS * m;
          if (r < nC) {
            if (r == myell) {
              double* ur = a.urow + slot * (int64_t)cap;
#pragma unroll
              for (int t = 0; t < NB; ++t) ur[2 * t + g] = qv[m][t];
            }
            const int ro = NORB * s_orig[r >> 2] + (r & 3);
            const int pb = s_patb[r >> 2];
            const int p = a.full ? ro : (pb >= 0 ? NORB * pb + (r & 3) : -1);
            if (p >= 0) {
              double* dst = a.qpat + (slot * (int64_t)a.pat_stride + p) * cap;
#pragma unroll
              for (int t = 0; t < NB; ++t) dst[2 * t + g] = qv[m][t];
            }
            if (ADJ) {
              double* dq = a.adj_q + slot * (int64_t)cap * a.adj_rows + ro;
#pragma unroll
              for (int t = 0; t < NB; ++t) dq[(int64_t)(2 * t + g) * a.adj_rows] = qv[m][t];
            }
          }
        }
      }

      // ---- s = Q^T (S_C Q), CB vectors of each column at a time: the
      // vectors go to LDS (over the operands and the cached blocks), S_C
      // streams once per pass through the matrix cores, and the products,
      // written over the vectors, are dotted with the basis
      char* s_q = U;
      char* s_z = s_q + (ROWS / 4 + 1) * PA;
      double* s_sred = reinterpret_cast<double*>(s_z + (ROWS / 4) * PA);
      // byte offset of row r in s_q and s_z
      auto prow = [&](int r) __attribute__((always_inline)) {
        return (r >> 2) * PA + ((r >> 1) & 1) * PQ + (r & 1) * 8;
      };
      __syncthreads();
      for (int i = opaque(tid); i < (ROWS / 4 + 1) * PA / 8; i += KTPB)
        *reinterpret_cast<double*>(s_q + (ROWS / 4) * PA + i * 8) = 0.0;
      for (int cc = 0; cc * CB < nu_max; ++cc) {
        __syncthreads();
#pragma unroll
        for (int gg = 0; gg < (NU + CB - 1) / CB; ++gg) {
          if (gg == cc) {
            char* dst = s_q + prow(opaque(p0)) + ((NCOL == 2 ? col : 0) * CB + g * (CB / 2)) * 16;
#pragma unroll
            for (int m = 0; m < RPL; ++m) {
#pragma unroll
              for (int v = 0; v < CB / 2; ++v) {
                const int t = gg * (CB / 2) + v;
                double qe = 0.0;
                if (t < NB) qe = qv[m][t < NB ? t : 0];
                *reinterpret_cast<double*>(dst + (LROWS / 4) * m * PA + v * 16) = qe;
              }
            }
          }
        }
        __syncthreads();
        // groups of four of the NCOL * CB vectors
        constexpr int NG = NCOL * CB / 4;
        const int la = opaque(lane);
        const int x = la & 3, b = (la >> 2) & 3, y = la >> 4;
        {
          // vector 4 gr + x of the lane's orbital pair
          const char* qb = s_q + (y & 1) * PQ + x * 16;
          const char* tp = tabu + (b * 2 + (y >> 1)) * 4;
          char* zr = s_z + prow(16 * wave + 4 * b + y) + x * 16;
          // a unit's blocks are on their way while the one before is used
          double2 sn[2];
          unit_blocks(sn, 0, la, 128);
          double acc[NG][2];
#pragma unroll
          for (int gr = 0; gr < NG; ++gr) acc[gr][0] = acc[gr][1] = 0.0;
          uint64_t fend = uend;
          uint32_t wd = *(const __attribute__((address_space(3))) uint32_t*)tp;
          for (int un = 0; un < nun; ++un) {
            const double2 sc[2] = {sn[0], sn[1]};
            double2 xq[2][NG];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
              // the operand's atom: its byte offset / 32, times PA bytes
              const char* qr = qb + __umul24(v ? wd >> 16 : wd & 0xffffu, PA / 32);
#pragma unroll
              for (int gr = 0; gr < NG; ++gr) xq[v][gr] = ld_lds2(qr + gr * 64);
            }
            tp += TAB_UNIT;
            wd = *(const __attribute__((address_space(3))) uint32_t*)tp;
            if (un + 1 < nun) unit_blocks(sn, un + 1, la, 128);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int v = 0; v < 2; ++v) {
#pragma unroll
              for (int gr = 0; gr < NG; ++gr)
                acc[gr][0] =
                    __builtin_amdgcn_mfma_f64_4x4x4f64(sc[v].x, xq[v][gr].x, acc[gr][0], 0, 0, 0);
#pragma unroll
              for (int gr = 0; gr < NG; ++gr)
                acc[gr][1] =
                    __builtin_amdgcn_mfma_f64_4x4x4f64(sc[v].y, xq[v][gr].y, acc[gr][1], 0, 0, 0);
            }
            if (fend & 1) {
#pragma unroll
              for (int gr = 0; gr < NG; ++gr) {
                *reinterpret_cast<double*>(zr + gr * 64) = acc[gr][0] + acc[gr][1];
                acc[gr][0] = acc[gr][1] = 0.0;
              }
              zr += KW * 4 * PA;
            }
            fend >>= 1;
          }
        }
        __syncthreads();
        for (int jj = 0; jj < CB; ++jj) {
          const int j = cc * CB + 2 * (jj & (CB / 2 - 1)) + jj / (CB / 2);
          if (mine && j < nu_eff) {
            double z[RPL];
            const char* zp = s_z + prow(opaque(p0)) + ((NCOL == 2 ? col : 0) * CB + jj) * 16;
#pragma unroll
            for (int m = 0; m < RPL; ++m) z[m] = ld_lds(zp + (LROWS / 4) * m * PA);
            dots(z, j, s_sred + ((jj * KW + wave) * 2 + g) * 16 * NSET, std::false_type{});
          }
        }
        __syncthreads();
        for (int idx = wv * 64 + lane; idx < CB * 32 * NSET; idx += WPC * 64) {
          const int jj = idx / (32 * NSET), rem = idx % (32 * NSET);
          const int gg = rem / (16 * NSET), sl = rem % (16 * NSET);
          const int j = cc * CB + 2 * (jj & (CB / 2 - 1)) + jj / (CB / 2);
          // (slots as the dots leave them: vector t of set 0, 15 + t of set 1)
          const int i = 2 * (sl < 16 ? sl : sl - 1) + gg;
          if (mine && j < nu_eff && i <= j && sl != 15 && !(j < 14 && sl >= 7)) {
            const double* rp = s_sred + ((jj * KW + (wave - wv)) * 2 + gg) * 16 * NSET + sl;
            double acc = rp[0];
            for (int v = 1; v < WPC; ++v) acc += rp[v * 2 * 16 * NSET];
            scol[(int64_t)j * cap + i] = acc;
          }
        }
      }
      __syncthreads();
    }
  }
}

// Workgroup shapes: eight waves, two columns of an atom in up to 768 rows for
// nu <= 30 (half of the basis vectors of RPL rows in a lane: nu = 30 takes 60,
// 120, 150 or 180 registers for clusters of up to 64, 128, 160 or 192 atoms).
// Two columns take 200 registers at nu = 40 and 160 atoms, 192 at nu = 48 and 128:
// some of the rest then lives in scratch, which still costs less than a
// workgroup for one column (3,892 atoms, r = 6, nu = 40: 15.9 against 17.3 ms).
// Beyond that a cluster takes the whole workgroup for one column.  A column's
// shape follows from nu and its cluster's size alone: a smaller shape has fewer instructions per step and
// holds more of H in LDS, so the smallest that holds a cluster is the fastest
// one (160-atom clusters at nu = 30: 7.3 ms with 5 rows against 9.9 ms with 6).
struct ShapeDef {
  int cap, ncol, rpl;
};
static constexpr ShapeDef kShapes[] = {
    {12, 2, 2}, {12, 2, 4}, {12, 2, 6},
    {20, 2, 2}, {20, 2, 4}, {20, 2, 5}, {20, 2, 6},
    {30, 2, 2}, {30, 2, 4}, {30, 2, 5}, {30, 2, 6},
    {40, 2, 2}, {40, 2, 4}, {40, 2, 5}, {40, 1, 3},
    {48, 2, 2}, {48, 2, 4}, {48, 1, 3},
};
constexpr int kNumShapes = (int)(sizeof(kShapes) / sizeof(kShapes[0]));

template <int I>
static const void* kfn(bool adj) {
  constexpr ShapeDef s = kShapes[I];
  if constexpr (s.cap <= 30) {
    if (adj) return reinterpret_cast<const void*>(&krylov_kernel<s.cap, s.ncol, s.rpl, true>);
  }
  return adj ? nullptr
             : reinterpret_cast<const void*>(&krylov_kernel<s.cap, s.ncol, s.rpl, false>);
}

// the kernel of shape `id`; adj: the variant that also leaves each column's
// basis, h, beta and last residual for the exact gradient (nu <= 30 shapes only)
template <int I = 0>
static const void* shape_fn(int id, bool adj = false) {
  if constexpr (I < kNumShapes) {
    return id == I ? kfn<I>(adj) : shape_fn<I + 1>(id, adj);
  } else {
    return nullptr;
  }
}

static int shape_rows(int id) { return 32 * (KW / kShapes[id].ncol) * kShapes[id].rpl; }

int krylov_shapes(int cap, KrylovShapeInfo* out, int max_out) {
  int n = 0;
  for (int i = 0; i < kNumShapes; ++i) {
    if (kShapes[i].cap != cap) continue;
    if (n < max_out) {
      out[n].cap = cap;
      out[n].tpb = KTPB;
      out[n].r = kShapes[i].rpl;
      out[n].nrows = shape_rows(i);
      out[n].id = i;
    }
    ++n;
  }
  return n;
}

size_t krylov_static_lds(int id) {
  hipFuncAttributes attr{};
  if (hipFuncGetAttributes(&attr, shape_fn(id)) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return attr.sharedSizeBytes;
}

size_t krylov_pool_min(int id) {
  return pool_bytes(shape_rows(id), kShapes[id].ncol, (kShapes[id].cap / 2) / 16 + 1);
}

// cluster blocks cached in `dyn` bytes at the most (four per tile block)
int krylov_cache_blocks(int id, size_t dyn) {
  const int rows = shape_rows(id);
  const size_t fixed = 2 * x_bytes(rows) + w_bytes(rows) + 2 * PAIR_CACHE;
  return dyn > fixed ? (int)((dyn - fixed) / (2 * PAIR_CACHE) / KW) * KW * KRYLOV_UNIT_BLOCKS : 0;
}

// workgroups of shape `id` that fit on one CU with `dyn` bytes of dynamic
// LDS each (0 if the launch would not fit); also raises the kernel's dynamic
// LDS limit to `dyn`
int krylov_occupancy(int id, size_t dyn) {
  const void* fn = shape_fn(id);
  if (!fn) return 0;
  // the kernel's dynamic LDS limit only ever rises, so a query never lowers
  // it below what an earlier plan launches with
  static size_t dyn_set[kNumShapes] = {};
  if (dyn > dyn_set[id]) {
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn) !=
        hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    // the exact-gradient variant launches with the same plans
    const void* fa = shape_fn(id, true);
    if (fa && hipFuncSetAttribute(fa, hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn) !=
                  hipSuccess) {
      (void)hipGetLastError();
      return 0;
    }
    dyn_set[id] = dyn;
  }
  int nb = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, fn, KTPB, dyn) != hipSuccess) {
    (void)hipGetLastError();
    return 0;
  }
  return nb;
}

hipError_t launch_krylov(const KrylovArgs& a, int id, size_t dyn, int grid, hipStream_t s) {
  const void* fn = shape_fn(id, a.adj_q != nullptr);
  if (!fn || grid <= 0 || dyn < krylov_pool_min(id) || (!a.queue && a.group < 1))
    return hipErrorInvalidValue;
  KrylovArgs copy = a;
  copy.pool = (int)dyn;
  void* args[] = {&copy};
  return hipLaunchKernel(fn, dim3(grid), dim3(KTPB), args, dyn, s);
}

int krylov_capacity(int nu) {
  static const int caps[] = {12, 20, 30, 40, 48};
  for (int c : caps)
    if (nu <= c) return c;
  return 0;
}

}  // namespace mag
