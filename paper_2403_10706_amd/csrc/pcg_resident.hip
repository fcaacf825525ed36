// Resident form of the Gauss-Newton PCG: a whole solve (every iteration) in one launch.
//
// The vectors of a volume fit the register files and the LDS of the chip (256 CUs with 512 KB of
// registers and 160 KB of LDS each), so one workgroup per CU takes a unit of the plane march
// (T plane positions times XL planes, see MarchGeo), keeps r, w, d, the couplings and x of its
// nodes in registers and p in LDS, and reads the bands once per solve instead of moving ten
// vectors through memory on every iteration.  What leaves a workgroup per iteration is p at its
// faces and seven partial sums.
//
// Exchange.  Values cross workgroups as 8-byte words of 32 data bits and a 32-bit tag (the
// iteration's number within the solve's launch sequence), written and polled with relaxed
// agent-scope atomics: a word is valid exactly when its tag is the awaited one, so no fence, no
// flag and no ordering between words is needed.  Words are double-buffered by iteration parity:
// iteration i + 2 is written only after every workgroup's sums of iteration i + 1 arrived, and
// those were written after its reads of iteration i.  Tags only grow from launch to launch; the
// words are cleared once at the start of a solve.
//
// Residency.  Every workgroup publishes its arrival; the volume's first workgroup waits for all
// arrivals and then publishes the decision to go.  Past that point all workgroups are resident and
// every wait ends.  If other work keeps them from becoming resident for kArriveTicks, it decides
// against it: the others leave and the first one solves the volume alone from memory.
//
// What bounds it (rgp_pcg_solve with 20 iterations, us per iteration, stepped against resident):
//   25x25x17 FP32 14.5 / 5.1   72x84x56 17.9 / 7.0   144x168x111 33.9 / 14.1   200x200x132 54 / 28
//   32x32x24 FP64 19 / 5.5     90x90x90 FP64 31 / 12.2
// Small volumes: two exchanges per iteration (outer p and sums), about 1 us of latency each, and
// the workgroup barriers between.  144x168x111: of 12.7 us, 3.3 wait for the outer p (8 MB of words
// each way), 2 for the sums, 2.3 + 1.6 are the stencil and its reduction (FP64 issue), 2.8 the update.
// Above that d and the couplings no longer fit the registers and are read again from the L2, a group
// of planes ahead of their use (200x200x132: stencil 8 and update 7 of 25 us; with a position's
// planes read together, right before their use, 9.6 and 12 of 35).
//
// Arithmetic: node for node that of the stepped form (pcg.hip), with the block sums formed over
// this form's own partition.
#include "rgp_internal.hpp"
#include "rgp_launch.hpp"
#include "rgp_solver.hpp"
#include "batch.hpp"

#include <algorithm>

#pragma clang fp contract(off)

#include "pcg_scalar.hpp"

namespace rgp {

namespace {

typedef unsigned long long u64;

constexpr int kResBlock = 512;
constexpr u64 kArriveTicks = 2000000;    // 20 ms of the 100 MHz clock
constexpr u64 kWaitTicks = 200000000;    // 2 s

__device__ __forceinline__ void word_put(u64* p, u64 v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 word_get(const u64* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ u64 tagged(uint32_t tag, uint32_t v) { return ((u64)tag << 32) | v; }

// A field value as words (one per 32 bits) at index n of `w`.
// (Byte offsets stay below 2^32: a volume here has at most kMaxResUnits * kResBlock * 48 nodes.)
__device__ __forceinline__ u64* word_at(u64* w, uint32_t byte) {
  return reinterpret_cast<u64*>(reinterpret_cast<char*>(w) + byte);
}
__device__ __forceinline__ const u64* word_at(const u64* w, uint32_t byte) {
  return reinterpret_cast<const u64*>(reinterpret_cast<const char*>(w) + byte);
}
__device__ __forceinline__ void value_put(u64* w, uint32_t n, float v, uint32_t tag) {
  word_put(word_at(w, 8u * n), tagged(tag, __float_as_uint(v)));
}
__device__ __forceinline__ void value_put(u64* w, uint32_t n, double v, uint32_t tag) {
  word_put(word_at(w, 16u * n), tagged(tag, (uint32_t)__double2loint(v)));
  word_put(word_at(w, 16u * n + 8u), tagged(tag, (uint32_t)__double2hiint(v)));
}
__device__ __forceinline__ float value_of(const u64 (&u)[1]) { return __uint_as_float((uint32_t)u[0]); }
__device__ __forceinline__ double value_of(const u64 (&u)[2]) {
  return __hiloint2double((int)(uint32_t)u[1], (int)(uint32_t)u[0]);
}

// Waits for K values at indexes n[] of `w` (kNullOff: not wanted, gives 0); all loads of a round
// are in flight together.  False when the wait was given up after `spins` rounds.  (Rounds and not
// time: none pass while the device runs something else.)
template <typename TR, int K>
__device__ __forceinline__ bool values_get(const u64* w, const uint32_t (&n)[K], uint32_t tag,
                                           uint32_t spins, TR (&v)[K]) {
  constexpr int W = sizeof(TR) / 4;
  u64 u[K][W];
#pragma unroll
  for (int k = 0; k < K; ++k)
#pragma unroll
    for (int j = 0; j < W; ++j)
      u[k][j] = word_get(word_at(w, 8u * (W * (n[k] != kNullOff ? n[k] : 0u) + j)));
  auto arrived = [&](int k) -> bool {
    bool ok = true;
#pragma unroll
    for (int j = 0; j < W; ++j) ok &= (uint32_t)(u[k][j] >> 32) == tag;
    return ok || n[k] == kNullOff;
  };
  for (uint32_t spin = 0;; ++spin) {
    bool ok = true;
#pragma unroll
    for (int k = 0; k < K; ++k) ok &= arrived(k);
    if (ok) break;
    if (spin == spins) return false;
    // only what has not arrived is read again
    __builtin_amdgcn_s_sleep(1);
#pragma unroll
    for (int k = 0; k < K; ++k)
      if (!arrived(k)) {
#pragma unroll
        for (int j = 0; j < W; ++j) u[k][j] = word_get(word_at(w, 8u * (W * n[k] + j)));
      }
  }
#pragma unroll
  for (int k = 0; k < K; ++k) v[k] = n[k] != kNullOff ? value_of(u[k]) : TR(0);
  return true;
}

// A value that is the same in every lane, held in a scalar register.
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniform(float v) {
  return __int_as_float(uniform(__float_as_int(v)));
}
__device__ __forceinline__ double uniform(double v) {
  return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}

// Waits for the sums of the units (kResSumStride words each: sum k's two halves at 2 k and 2 k + 1).
// Thread t takes word t % 16 of units t / 16, t / 16 + 32, ... (J of them), so that loads are
// consecutive; returns the sum over its units of sum (t % 16) / 2, on even threads.
template <int J>
__device__ __forceinline__ bool sums_get(const u64* part, int units, uint32_t tag, uint32_t spins,
                                         double& s) {
  uint32_t n[J];
  float f[J];
  const int t = threadIdx.x;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int u = t / 16 + j * (kResBlock / 16);
    n[j] = u < units && (t & 15) < 14 ? (uint32_t)(u * kResSumStride + (t & 15)) : kNullOff;
  }
  const bool ok = values_get<float, J>(part, n, tag, spins, f);
  s = 0.0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int own = (int)__float_as_uint(f[j]);
    const int next = __builtin_amdgcn_update_dpp(0, own, 0xB1, 0xF, 0xF, false);   // lane ^ 1
    s += __hiloint2double(next, own);
  }
  return ok;
}

// A unit: whole rows of the plane (`teff` positions from f0) times np planes from o0.
struct ResUnit {
  int f0, teff, o0, np;
};
__device__ __forceinline__ ResUnit res_unit(const ResArgs& a, int u) {
  ResUnit r;
  const int ti = u / a.noc, oc = u - ti * a.noc;
  r.f0 = uniform(ti * a.T);
  r.teff = uniform(min(a.T, a.P - r.f0));
  r.o0 = uniform(oc * a.XL);
  r.np = uniform(min(a.XL, a.no - r.o0));
  return r;
}

// w = H p at one node, accumulated in FP64 and rounded once (as in the stepped form).  ol, ou:
// the couplings to the lower and upper PE neighbour.
template <typename TR>
__device__ __forceinline__ TR res_stencil(int ROLE, TR d, TR pk, TR pom, TR pop, TR pam, TR pap, TR pbm,
                                          TR pbp, TR ol, TR ou, TR c_o, TR c_a, TR c_b) {
  double wd = (double)d * (double)pk;
  if (ROLE == 0) {
    wd = fmad((double)ol, (double)pom, wd);
    wd = fmad((double)ou, (double)pop, wd);
    wd = fmad(-(double)c_a, (double)pam + (double)pap, wd);
    wd = fmad(-(double)c_b, (double)pbm + (double)pbp, wd);
  } else if (ROLE == 1) {
    wd = fmad((double)ol, (double)pam, wd);
    wd = fmad((double)ou, (double)pap, wd);
    wd = fmad(-(double)c_o, (double)pom + (double)pop, wd);
    wd = fmad(-(double)c_b, (double)pbm + (double)pbp, wd);
  } else {
    wd = fmad((double)ol, (double)pbm, wd);
    wd = fmad((double)ou, (double)pbp, wd);
    wd = fmad(-(double)c_o, (double)pom + (double)pop, wd);
    wd = fmad(-(double)c_a, (double)pam + (double)pap, wd);
  }
  return (TR)wd;
}

template <typename TR>
__device__ __forceinline__ void res_sums(double (&acc)[7], TR pk, TR w, TR r, TR z, TR rd) {
  const double rr = (double)r, ww = (double)w, zz = (double)z, id = (double)rd;
  acc[0] = fmad((double)pk, ww, acc[0]);
  acc[1] = fmad(zz, ww, acc[1]);
  acc[2] = fmad(ww * ww, id, acc[2]);
  acc[3] = fmad(rr, ww, acc[3]);
  acc[4] = fmad(ww, ww, acc[4]);
  acc[5] = fmad(rr, zz, acc[5]);
  acc[6] = fmad(rr, rr, acc[6]);
}

struct ResShared {
  double sh[kResBlock / 16][8];
  int flag;
};

// Sum k of the rows' partial sums, on lane 8 k of every wavefront: eight lanes per sum.
__device__ __forceinline__ double res_row_sum(const double (*sh)[8]) {
  const int lane = threadIdx.x & (kWave - 1);
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < kResBlock / 128; ++j) s += sh[(lane & 7) + 8 * j][lane >> 3];
  s += dpp_row<0xB1>(s);    // lane ^ 1
  s += dpp_row<0x4E>(s);    // lane ^ 2
  s += dpp_row<0x141>(s);   // mirrored within 8
  return s;
}

// This workgroup's sums of acc: sum k is valid on lane 8 k.  Lane pairs, then quads, split the
// eight values (one of them 0) between them while they add, so that a lane ends with two values
// of its 16-lane row instead of reducing all seven over 64 lanes.
__device__ __forceinline__ double res_block_sum(const double (&acc)[7], double (*sh)[8]) {
  const int lane = threadIdx.x & (kWave - 1);
  const bool b0 = lane & 1, b1 = lane & 2;
  double h[4], q[2];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double lo = acc[k], hi = k < 3 ? acc[k < 3 ? k + 4 : 0] : 0.0;
    h[k] = (b0 ? hi : lo) + dpp_row<0xB1>(b0 ? lo : hi);   // lane ^ 1
  }
#pragma unroll
  for (int k = 0; k < 2; ++k)
    q[k] = (b1 ? h[k + 2] : h[k]) + dpp_row<0x4E>(b1 ? h[k] : h[k + 2]);   // lane ^ 2
#pragma unroll
  for (int k = 0; k < 2; ++k) q[k] += dpp_row<0x128>(q[k]);   // row rotations by 8 and 4
#pragma unroll
  for (int k = 0; k < 2; ++k) q[k] += dpp_row<0x124>(q[k]);
  const int row = threadIdx.x / 16;
  if ((lane & 15) < 4) {
    const int v = 4 * (lane & 1) + (lane & 2);
    sh[row][v] = q[0];
    sh[row][v + 1] = q[1];
  }
  __syncthreads();
  return res_row_sum(sh);
}

// The cross-axis couplings along the march's axes (0 along the PE axis).
template <typename TR>
__device__ __forceinline__ void res_couplings(const ResArgs& a, int role, TR& c_o, TR& c_a,
                                              TR& c_b) {
  const TR cx = (TR)a.cx, cy = (TR)a.cy;
  c_o = role == 0 ? TR(0) : cx;
  c_a = role == 0 ? cx : (role == 1 ? TR(0) : cy);
  c_b = role == 2 ? TR(0) : cy;
}

__device__ __forceinline__ void res_outputs(const ResArgs& a, const PcgSlot& c) {
  a.st->pcg_iters = c.iters;
  a.st->relres = c.relres;
  if (a.iters_out) *a.iters_out = c.iters;
  if (a.relres_out) *a.relres_out = c.relres;
}

// The whole solve by one workgroup, from memory (the decision against residency): vectors r and p
// in the two spare arrays, w in the first word array, which is cleared again at the end.
template <typename TR>
__device__ __forceinline__ void res_alone(const ResArgs& a, ResShared& m) {
  double (*sh)[8] = m.sh;
  const int role = a.role;
  const int t = threadIdx.x, na = a.na, nb = a.nb, no = a.no, P = a.P;
  const TR* __restrict__ dg = static_cast<const TR*>(a.diag);
  const TR* __restrict__ of = static_cast<const TR*>(a.off);
  const TR* __restrict__ rhs = static_cast<const TR*>(a.rhs);
  TR* x = static_cast<TR*>(a.x);
  TR* r = static_cast<TR*>(a.spare_r);
  TR* p = static_cast<TR*>(a.spare_p);
  TR* w = reinterpret_cast<TR*>(a.words);
  TR c_o, c_a, c_b;
  res_couplings<TR>(a, role, c_o, c_a, c_b);
  const uint32_t n = a.nnode;
  for (uint32_t i = t; i < n; i += kResBlock) {
    const TR rv = (TR)a.rhs_sign * rhs[i];
    r[i] = rv;
    p[i] = fmad(TR(0), TR(0), rv * (TR(1) / dg[i]));
    x[i] = TR(0);
  }
  __syncthreads();
  PcgSlot cur{};
  for (int it = 1; it <= a.maxit; ++it) {
    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
    for (uint32_t k = t; k < n; k += kResBlock) {
      const int o = (int)(k / (uint32_t)P), f = (int)(k - (uint32_t)o * (uint32_t)P);
      const int ia = f / nb, ib = f - ia * nb;
      const TR pk = p[k], d = dg[k];
      const TR pom = o > 0 ? p[k - P] : TR(0), pop = o < no - 1 ? p[k + P] : TR(0);
      const TR pam = ia > 0 ? p[k - nb] : TR(0), pap = ia < na - 1 ? p[k + nb] : TR(0);
      const TR pbm = ib > 0 ? p[k - 1] : TR(0), pbp = ib < nb - 1 ? p[k + 1] : TR(0);
      TR ol = TR(0);
      if (role == 0 && o > 0) ol = of[k - P];
      if (role == 1 && ia > 0) ol = of[k - nb];
      if (role == 2 && ib > 0) ol = of[k - 1];
      const TR wv = res_stencil<TR>(role, d, pk, pom, pop, pam, pap, pbm, pbp, ol, of[k], c_o, c_a,
                                    c_b);
      w[k] = wv;
      const TR rd = TR(1) / d, rv = r[k];
      res_sums<TR>(acc, pk, wv, rv, rv * rd, rd);
    }
    const double s = res_block_sum(acc, sh);
    double ts[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) ts[k] = read_lane(s, 8 * k);
    __syncthreads();
    bool fin = false;
    cur = pcg_advance(cur, ts, it, a.maxit, a.rtol, fin);
    if (cur.status == kPcgDone) break;
    const TR al = (TR)cur.alpha, be = (TR)cur.beta;
    for (uint32_t i = t; i < n; i += kResBlock) {
      const TR pv = p[i];
      if (fin) {
        x[i] = x[i] + al * pv;
      } else {
        x[i] = fmad(al, pv, x[i]);
        const TR rv = fmad(-al, w[i], r[i]);
        r[i] = rv;
        p[i] = fmad(be, pv, rv * (TR(1) / dg[i]));
      }
    }
    __syncthreads();
    if (fin) break;
  }
  __syncthreads();
  for (uint32_t i = t; i < n; i += kResBlock) w[i] = TR(0);
  if (t == 0) res_outputs(a, cur);
}

// Makes v opaque to the compiler: values derived from it are not kept across iterations.
template <typename TR>
__device__ __forceinline__ void keep_single(TR& v) {
  __asm__ volatile("" : "+v"(v));
}

// KEEP bits: what a thread keeps in registers for the whole solve besides r and w of its nodes: d,
// 1/d, the couplings.  What is not kept is read again (or formed again) on every iteration.
enum ResKeep : int { kKeepDiag = 1, kKeepRecip = 2, kKeepOff = 4, kKeepAll = 7 };
constexpr int kResGroup = 4;   // planes handled as one straight run of code

// A kernel variant: plane positions per thread, most planes, KEEP bits, positions whose x is kept
// in LDS (the others': registers), and the stride of an LDS plane of p.  Such a plane holds one row
// before the tile, the tile, one row after it and, last, a slot that stays 0 for missing
// neighbours; its stride is a constant, so that every plane of a neighbour is one base address and
// an immediate offset.
struct ResTier {
  int npt, xl, keep, xlds, stride;
};

// One unit's share of the solve (see the head of the file): at most NPT plane positions per thread
// and XL planes.  A thread's position i is (t + i * kResBlock + nb) mod T, so that the rows next
// to other units (the tile's first and last) belong to the last positions, which an update takes
// and publishes first.  True when this (the volume's first) workgroup is to solve it alone.
template <typename TR, int ROLE, int NPT, int XL, int KEEP, int XN, int S>
__device__ __forceinline__ bool res_body(const ResArgs& a, int ub, ResShared& m) {
  constexpr bool KD = (KEEP & kKeepDiag) != 0, KR = (KEEP & kKeepRecip) != 0,
                 KO = (KEEP & kKeepOff) != 0;
  constexpr uint32_t kSz = sizeof(TR);
  extern __shared__ unsigned char res_lds[];
  TR* lds = reinterpret_cast<TR*>(res_lds);
  double (*sh)[8] = m.sh;
  int& flag = m.flag;
  const int t = threadIdx.x;
  const uint32_t tag0 = a.tag;
  if (t == 0) {
    word_put(a.sync + ub, tagged(tag0, 1u));
    flag = 0;
  }
  const int nb = uniform(a.nb), no = uniform(a.no);
  int P = uniform(a.P);
  const ResUnit un = res_unit(a, ub);
  int np = un.np;
  // planes 0 .. XL - 1 and one more; x of position i < XN, plane q, behind them
  TR* xlds = lds + (XL + 1) * S + t;
  for (int k = t; k < (XL + 1) * S; k += kResBlock) lds[k] = TR(0);
  const uint32_t nbytes = a.nnode * kSz;
  const BRes rD = bres(a.diag, nbytes), rO = bres(a.off, nbytes), rR = bres(a.rhs, nbytes);
  const BRes rX = bres(a.x, nbytes);
  const bool gn = a.gn_mode != 0;

  double lsum[5];
  if (gn) load_partials_rm<5>(lsum, a.lf.part, a.lf.nprod);

  // Own: the thread has this position; Edge: in the tile's first or last row; NoLo, NoHi: an
  // a-neighbour is missing; Bm, Bp: the b-neighbours exist (bits of one register per position: as
  // masks they would hold scalar registers throughout).  lc: LDS offset of the position.
  enum { kOwn = 1, kEdge = 2, kNoLo = 4, kNoHi = 8, kBm = 16, kBp = 32 };
  uint32_t pos[NPT], bits[NPT];
  int lc[NPT];
#pragma unroll
  for (int i = 0; i < NPT; ++i) {
    const int j = t + i * kResBlock;
    const bool mine = j < un.teff;
    int l = j + nb;
    if (l >= un.teff) l -= un.teff;
    if (!mine) l = 0;
    const int f = un.f0 + l, ib = f - (f / nb) * nb;
    bits[i] = (mine ? kOwn : 0) | (l < nb || l >= un.teff - nb ? kEdge : 0) | (f < nb ? kNoLo : 0) |
              (f >= P - nb ? kNoHi : 0) | (ib > 0 ? kBm : 0) | (ib < nb - 1 ? kBp : 0);
    pos[i] = (uint32_t)un.o0 * (uint32_t)P + (uint32_t)f;
    lc[i] = nb + l;
  }
  auto has = [&](int i, int what) -> bool { return (bits[i] & (uint32_t)what) != 0; };
  auto node = [&](int q, int i) -> uint32_t { return pos[i] + (uint32_t)q * (uint32_t)P; };
  auto at = [&](bool ok, uint32_t n) -> uint32_t { return ok ? n * kSz : kNullOff; };
  // coupling to the lower PE neighbour in the plane (roles 1 and 2; 0 at the lower end)
  auto lower = [&](int q, int i) -> TR {
    if (ROLE == 1) return bld<TR>(rO, at(!has(i, kNoLo), node(q, i) - (uint32_t)nb));
    if (ROLE == 2) return bld<TR>(rO, at(has(i, kBm), node(q, i) - 1u));
    return TR(0);
  };

  TR r[XL][NPT], w[XL][NPT], d[KD ? XL : 1][NPT];
  TR rd[KR ? XL : 1][NPT], oc[KO ? XL : 1][NPT], ob[KO && ROLE != 0 ? XL : 1][NPT];
  TR x[XL][NPT > XN ? NPT - XN : 1], om[NPT];
#pragma unroll
  for (int q = 0; q < XL; ++q)
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int qc = min(q, np - 1);   // (planes past the unit: r = 0, and w is held at 0)
      if (KD) d[KD ? q : 0][i] = bld<TR>(rD, node(qc, i) * kSz);
      r[q][i] = bld<TR>(rR, at(q < np && has(i, kOwn), node(qc, i)));
      if (KO) {
        oc[q][i] = bld<TR>(rO, node(qc, i) * kSz);
        if (ROLE != 0) ob[q][i] = lower(qc, i);
      }
      if (i >= XN) x[q][i >= XN ? i - XN : 0] = TR(0);
      w[q][i] = TR(0);
    }
#pragma unroll
  for (int i = 0; i < NPT; ++i)
    om[i] = ROLE == 0 ? bld<TR>(rO, at(has(i, kOwn) && un.o0 > 0, pos[i] - (uint32_t)P)) : TR(0);

  if (gn) {
    const bool stop = load_flag(&a.st->gn_stop) != 0;
    block_sum<5, kResBlock>(lsum);
    const bool viol = finalize_loss_sums(a.lf, lsum, !stop && ub == 0);
    if (stop || viol) return false;   // the same in every workgroup
  }

  // residency: all arrived, or the first workgroup alone
  if (ub == 0) {
    bool ok = true;
    if (t < a.units) {
      const u64 t0 = wall_clock64();
      while ((uint32_t)(word_get(a.sync + t) >> 32) != tag0) {
        if (wall_clock64() - t0 > kArriveTicks + a.patience) {
          ok = false;
          break;
        }
      }
    }
    __syncthreads();
    if (!ok) flag = 1;
    __syncthreads();
    const bool alone = flag != 0;
    if (t == 0) word_put(a.sync + kMaxResUnits, tagged(tag0, alone ? 2u : 1u));
    if (alone) return true;
  } else {
    if (t == 0) {
      u64 v = 0;
      const u64 t0 = wall_clock64();
      int go = 0;
      while (true) {
        v = word_get(a.sync + kMaxResUnits);
        if ((uint32_t)(v >> 32) == tag0) {
          go = (uint32_t)v == 1u;
          break;
        }
        if (wall_clock64() - t0 > kWaitTicks) break;
      }
      flag = go ? 0 : 1;
    }
    __syncthreads();
    if (flag) return false;
  }

  TR c_o, c_a, c_b;
  res_couplings<TR>(a, ROLE, c_o, c_a, c_b);
  const TR sg = (TR)a.rhs_sign;
  const size_t wstride = (size_t)a.nnode * (kSz / 4);   // words per parity
  const uint32_t pstride = (uint32_t)kResSumStride * kMaxResUnits;

  // Keeps addresses from being formed once before the iterations and held in registers.
  auto opaque = [&]() {
    P = uniform(P);
    np = uniform(np);
    __asm__ volatile("" : "+s"(P), "+s"(np));
#pragma unroll
    for (int i = 0; i < NPT; ++i) __asm__ volatile("" : "+v"(pos[i]), "+v"(bits[i]), "+v"(lc[i]));
  };
  // p of one node to LDS and, at the unit's faces, to the neighbours
  auto put_p = [&](int q, int i, TR p, u64* words, uint32_t tag) {
    lds[q * S + lc[i]] = p;
    if (has(i, kEdge) || q == 0 || q == np - 1) value_put(words, node(q, i), p, tag);
  };
  // planes in the order in which an update takes them: the outer ones first (in their order where
  // the diagonal is read again, group by group)
  auto nth = [](int k) -> int {
    return !KD && !KR ? k : (k == 0 ? 0 : (k == 1 ? XL - 1 : k - 1));
  };
  {
    u64* words = a.words + (size_t)((tag0 + 1u) & 1u) * wstride;
#pragma unroll
    for (int i = NPT - 1; i >= 0; --i)
#pragma unroll
      for (int k = 0; k < XL; ++k) {
        const int q = nth(k);
        const TR inv = TR(1) / (KD ? d[KD ? q : 0][i] : bld<TR>(rD, node(min(q, np - 1), i) * kSz));
        r[q][i] = sg * r[q][i];
        if (KR) rd[KR ? q : 0][i] = inv;
        if (q < np && has(i, kOwn)) put_p(q, i, fmad(TR(0), TR(0), r[q][i] * inv), words, tag0 + 1u);
        if (i < XN) xlds[(i * XL + q) * kResBlock] = TR(0);
      }
  }

  // What is not kept in registers is read again group by group of planes, one group ahead of its
  // use (a group takes longer than a read from the L2).  Every read is unconditional, so that none
  // is moved to its use.
  struct Stream {
    TR d[kResGroup], o[kResGroup], l[kResGroup];
  };
  auto fetch = [&](int i, int g, bool couplings) -> Stream {
    Stream f{};
#pragma unroll
    for (int j = 0; j < kResGroup; ++j) {
      const int q = min(g * kResGroup + j, np - 1);
      if (!KD) f.d[j] = bld<TR>(rD, node(q, i) * kSz);
      if (KO || !couplings) continue;
      f.o[j] = bld<TR>(rO, node(q, i) * kSz);
      f.l[j] = lower(q, i);
    }
    return f;
  };
  constexpr bool kStream = !KD || !KO;

  double bn = 0.0, rel = 0.0;
  int its = 0;
  bool lost = false;
  const int hn = 2 * nb * np;   // positions of the outer rows, all planes
  for (int it = 1; it <= a.maxit; ++it) {
    const uint32_t tag = tag0 + (uint32_t)it;
    opaque();
    const u64* words = a.words + (size_t)(tag & 1u) * wstride;
    Stream now = fetch(0, 0, true);
    // p at the planes before and after the unit and in the rows before and after its tile, all in
    // flight together; p after the unit and the rows go to LDS (the former to slots that only this
    // thread reads)
    TR pm[NPT];
    {
      constexpr int kRows = XL >= 12 ? 3 : (XL > 2 ? XL / 2 : 1);
      uint32_t n[2 * NPT + kRows];
      TR v[2 * NPT + kRows];
      int to[kRows];
#pragma unroll
      for (int i = 0; i < NPT; ++i) {
        n[i] = has(i, kOwn) && un.o0 > 0 ? pos[i] - (uint32_t)P : kNullOff;
        n[NPT + i] = has(i, kOwn) && un.o0 + np < no ? node(np, i) : kNullOff;
      }
      for (int h0 = 0;;) {
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
          const uint32_t hh = (uint32_t)(h0 + j * kResBlock + t);
          const uint32_t q = fdiv(hh, a.by_2nb);
          const int h = (int)(hh - q * (uint32_t)(2 * nb));
          const int f = h < nb ? un.f0 - nb + h : un.f0 + un.teff + (h - nb);
          const bool ok = hh < (uint32_t)hn && f >= 0 && f < P;
          n[2 * NPT + j] = ok ? (uint32_t)(un.o0 + (int)q) * (uint32_t)P + (uint32_t)f : kNullOff;
          to[j] = (int)q * S + (h < nb ? h : un.teff + h);
        }
        lost = !values_get<TR, 2 * NPT + kRows>(words, n, tag, a.spins, v) || lost;
#pragma unroll
        for (int j = 0; j < kRows; ++j)
          if (n[2 * NPT + j] != kNullOff) lds[to[j]] = v[2 * NPT + j];
        h0 += kRows * kResBlock;
        if (h0 >= hn) break;
      }
#pragma unroll
      for (int i = 0; i < NPT; ++i) {
        pm[i] = v[i];
        if (has(i, kOwn)) lds[np * S + lc[i]] = v[NPT + i];
      }
    }
    if (lost) flag = 1;
    __syncthreads();
    if (flag) break;

    // w = H p and the sums
    double acc[7] = {0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const TR* cc = lds + lc[i];
      const TR* cam = lds + (has(i, kNoLo) ? S - 1 : lc[i] - nb);
      const TR* cap = lds + (has(i, kNoHi) ? S - 1 : lc[i] + nb);
      const TR* cbm = lds + (has(i, kBm) ? lc[i] - 1 : S - 1);
      const TR* cbp = lds + (has(i, kBp) ? lc[i] + 1 : S - 1);
      TR pom = pm[i], pk = cc[0], ol = om[i];
#pragma unroll
      for (int q0 = 0; q0 < XL; q0 += kResGroup) {
        if (!kStream && q0 >= np) continue;
        const Stream f = now;
        if (kStream) {
          const bool more = q0 + kResGroup < XL;
          if (more || i + 1 < NPT) now = fetch(more ? i : i + 1, more ? q0 / kResGroup + 1 : 0, true);
          __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int q = q0; q < q0 + kResGroup && q < XL; ++q) {
          const TR pop = cc[(q + 1) * S], pam = cam[q * S], pap = cap[q * S];
          const TR pbm = cbm[q * S], pbp = cbp[q * S];
          // what is derived from the kept values (their FP64 forms, 1/d) is formed here each time
          if (KD) keep_single(d[KD ? q : 0][i]);
          if (KR) keep_single(rd[KR ? q : 0][i]);
          if (KO) keep_single(oc[KO ? q : 0][i]);
          if (KO && ROLE != 0) keep_single(ob[KO && ROLE != 0 ? q : 0][i]);
          const TR ou = KO ? oc[KO ? q : 0][i] : f.o[q - q0];
          if (ROLE != 0) ol = KO ? ob[KO && ROLE != 0 ? q : 0][i] : f.l[q - q0];
          const TR dk = KD ? d[KD ? q : 0][i] : f.d[q - q0];
          TR wv = res_stencil<TR>(ROLE, dk, pk, pom, pop, pam, pap, pbm, pbp, ol, ou, c_o, c_a,
                                  c_b);
          wv = has(i, kOwn) && q < np ? wv : TR(0);
          w[q][i] = wv;
          const TR inv = KR ? rd[KR ? q : 0][i] : TR(1) / dk;
          res_sums<TR>(acc, pk, wv, r[q][i], r[q][i] * inv, inv);
          pom = pk;
          pk = pop;
          if (ROLE == 0) ol = ou;
        }
        __builtin_amdgcn_sched_barrier(0);   // bounds the values held in registers
      }
    }
    // all-reduce: this unit's sums to every workgroup, theirs to this one
    const double s = res_block_sum(acc, sh);
    u64* part = a.part + (size_t)(tag & 1u) * pstride;
    if (t < 56 && (t & 7) == 0) {
      u64* mine = part + ub * kResSumStride + t / 4;
      word_put(mine, tagged(tag, (uint32_t)__double2loint(s)));
      word_put(mine + 1, tagged(tag, (uint32_t)__double2hiint(s)));
    }
    if (!KD && !KR) now = fetch(NPT - 1, 0, false);   // the update's, under the wait
    double us;
    const bool got = a.units <= 64    ? sums_get<2>(part, a.units, tag, a.spins, us)
                     : a.units <= 128 ? sums_get<4>(part, a.units, tag, a.spins, us)
                                      : sums_get<8>(part, a.units, tag, a.spins, us);
    if (!got) flag = 1;
    __syncthreads();   // (the row sums of this unit are read)
    if ((t & 1) == 0) sh[t / 16][(t & 15) / 2] = us;
    __syncthreads();
    if (flag) break;
    const double tot = res_row_sum(sh);
    double ts[7];
#pragma unroll
    for (int k = 0; k < 7; ++k) ts[k] = read_lane(tot, 8 * k);
    PcgSlot prev{};
    prev.bnorm2 = bn;
    prev.relres = rel;
    bool fin = false;
    const PcgSlot cur = pcg_advance(prev, ts, it, a.maxit, a.rtol, fin);
    bn = uniform(cur.bnorm2);
    rel = uniform(cur.relres);
    its = uniform(cur.iters);
    const bool done = uniform(cur.status) == kPcgDone;   // keep x
    const TR al = uniform((TR)cur.alpha), be = uniform((TR)cur.beta);
    fin = uniform(fin ? 1 : 0) != 0;
    if (done) break;
    u64* next = a.words + (size_t)((tag + 1u) & 1u) * wstride;
    opaque();
#pragma unroll
    for (int i = NPT - 1; i >= 0; --i) {
#pragma unroll
      for (int k0 = 0; k0 < XL; k0 += kResGroup) {
        const Stream f = now;
        if (!KD && !KR) {
          const bool more = k0 + kResGroup < XL;
          if (more || i > 0) now = fetch(more ? i : i - 1, more ? k0 / kResGroup + 1 : 0, false);
          __builtin_amdgcn_sched_barrier(0);
        }
        TR po[kResGroup], xv[kResGroup];
#pragma unroll
        for (int j = 0; j < kResGroup && k0 + j < XL; ++j) {
          const int q = nth(k0 + j);
          po[j] = lds[q * S + lc[i]];
          xv[j] = i < XN ? xlds[(i * XL + q) * kResBlock] : x[q][i >= XN ? i - XN : 0];
        }
#pragma unroll
        for (int j = 0; j < kResGroup && k0 + j < XL; ++j) {
          const int q = nth(k0 + j);
          const TR xw = fin ? xv[j] + al * po[j] : fmad(al, po[j], xv[j]);
          if (i < XN)
            xlds[(i * XL + q) * kResBlock] = xw;
          else
            x[q][i >= XN ? i - XN : 0] = xw;
          if (!KR && KD) keep_single(d[KD ? q : 0][i]);
          const TR rv = fmad(-al, w[q][i], r[q][i]);
          r[q][i] = rv;
          const TR inv = KR ? rd[KR ? q : 0][i]
                            : TR(1) / (KD ? d[KD ? q : 0][i] : f.d[j]);
          const TR pn = fmad(be, po[j], rv * inv);
          if (q < np && !fin && has(i, kOwn)) put_p(q, i, pn, next, tag + 1u);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (fin) break;
  }
  // A wait was given up: some workgroup stands still.  A level stops with b unchanged and a status; a
  // plain solve shows it in all its outputs: x of this unit and the residual NaN, -1 iterations.
  const bool failed = lost || flag;
  if (failed && t == 0) {
    if (gn) {
      __hip_atomic_store(&a.st->gn_stop, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (a.st->status == 0) a.st->status = RGP_EHIP;
    }
    if (a.iters_out) *a.iters_out = -1;
    if (a.relres_out) *a.relres_out = __longlong_as_double(0x7ff8000000000000LL);
  }
#pragma unroll
  for (int q = 0; q < XL; ++q)
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const TR xv = i < XN ? xlds[(i * XL + q) * kResBlock] : x[q][i >= XN ? i - XN : 0];
      bst<TR>(rX, at(q < np && has(i, kOwn), node(q, i)), failed ? (TR)__builtin_nan("") : xv);
    }
  if (failed) return false;
  if (ub == 0 && t == 0) {
    PcgSlot c{};
    c.iters = its;
    c.relres = rel;
    res_outputs(a, c);
  }
  return false;
}

template <typename TR, int NPT, int XL, int KEEP, int XN, int S>
__global__ __launch_bounds__(kResBlock, XL <= 2 ? 4 : 2) void k_pcg_resident(ResBatch b) {
  int p = 0;
  while (p + 1 < b.n && (int)blockIdx.x >= b.start[p + 1]) ++p;
  const ResArgs& a = b.v[p];
  const int ub = (int)blockIdx.x - b.start[p];
  if (ub >= a.units) return;
  __shared__ ResShared m;
  bool alone;
  if (a.role == 0)
    alone = res_body<TR, 0, NPT, XL, KEEP, XN, S>(a, ub, m);
  else if (a.role == 1)
    alone = res_body<TR, 1, NPT, XL, KEEP, XN, S>(a, ub, m);
  else
    alone = res_body<TR, 2, NPT, XL, KEEP, XN, S>(a, ub, m);
  if (alone) res_alone<TR>(a, m);
}

__global__ __launch_bounds__(kBlock) void k_clear_words(uint4* p, uint64_t n, u64* q, uint32_t nq) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  const uint64_t i0 = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  for (uint64_t i = i0; i < n; i += stride) p[i] = uint4{0u, 0u, 0u, 0u};
  for (uint64_t i = i0; i < nq; i += stride) q[i] = 0ull;
}

}  // namespace

namespace {

// The variants, in the order in which the planner tries them.  A thread has 256 registers; r and w
// of its nodes take two each, everything kept seven.  Up to 8 planes (16 nodes) all of it fits;
// at 12 planes x moves to LDS (without that 40 registers spilled and the update took 5.4 instead
// of 1.9 us), at 16 the couplings and, with a third position per thread, d are read again.  Units of at least 2 planes: with one
// the sums come from twice the workgroups.
constexpr ResTier kTiersF32[] = {{2, 2, kKeepAll, 0, 1537},  {2, 4, kKeepAll, 0, 1537},
                                 {2, 8, kKeepAll, 0, 1537},  {2, 12, kKeepAll, 2, 1537},
                                 {2, 16, kKeepDiag | kKeepRecip, 2, 1385}, {3, 16, 0, 1, 1824}};
constexpr ResTier kTiersF64[] = {{1, 2, kKeepAll, 0, 1033}, {1, 4, kKeepAll, 0, 1033},
                                 {1, 8, kKeepAll, 0, 1033}};

}  // namespace

// The unit shape of the resident form, a function of the geometry and the field type only: the
// first variant whose units fit one per CU, with rows and planes spread evenly over the units.
ResPlan plan_resident(const Geom& g, DType real) {
  ResPlan L{};
  const MarchGeo m = march_geo(g, 1, 1);
  if (m.nb > 256 || g.nnode > (int64_t)kMaxResUnits * kResBlock * 48) return L;
  const bool f64 = real == DType::F64;
  if (!f64 && real != DType::F32) return L;
  const ResTier* tiers = f64 ? kTiersF64 : kTiersF32;
  const int nt = f64 ? (int)(sizeof(kTiersF64) / sizeof(ResTier)) : (int)(sizeof(kTiersF32) / sizeof(ResTier));
  for (int k = 0; k < nt; ++k) {
    const ResTier& r = tiers[k];
    // rows of a tile
    const int most = std::min(r.npt * kResBlock / m.nb, (r.stride - 1) / m.nb - 2);
    if (most < 1) continue;
    const int ntile = (m.na + most - 1) / most;
    const int rows = (m.na + ntile - 1) / ntile;
    const int noc_max = kMaxResUnits / ntile;
    if (noc_max < 1) continue;
    int xl = (m.no + noc_max - 1) / noc_max;
    if (xl > r.xl) continue;
    if (k == 0 && xl < r.xl) xl = r.xl;
    const int T = rows * m.nb;
    const size_t lds = ((size_t)(r.xl + 1) * r.stride + (size_t)r.xlds * r.xl * kResBlock) *
                       dsize_real(real);
    if (lds > kMaxResLds) continue;
    L.m = march_geo(g, T, xl);
    L.lds = lds;
    L.tier = k;
    L.ok = true;
    return L;
  }
  return L;
}

ResArgs make_res_args(const Geom& g, const ResPlan& L, double alpha) {
  ResArgs a{};
  a.no = L.m.no;
  a.na = L.m.na;
  a.nb = L.m.nb;
  a.role = L.m.role;
  a.P = (int32_t)L.m.P;
  a.T = L.m.T;
  a.XL = L.m.XL;
  a.noc = L.m.noc;
  a.units = (int32_t)L.m.units;
  a.nnode = (uint32_t)g.nnode;
  a.ncell = (uint32_t)g.ncell;
  a.by_2nb = make_fastdiv((uint32_t)(2 * L.m.nb));
  a.spins = kResSpins;
  a.cx = alpha * g.vol / (g.hx * g.hx);
  a.cy = alpha * g.vol / (g.hy * g.hy);
  return a;
}

hipError_t launch_clear_words(void* words, int64_t nnode, DType real, void* sync, hipStream_t s) {
  if (active_recorder())
    return record_other([words, nnode, real, sync](hipStream_t s2) {
      return launch_clear_words(words, nnode, real, sync, s2);
    });
  // two parities of one word per 32 bits of the field, in 16-byte stores
  const uint64_t n = (uint64_t)nnode * (real == DType::F64 ? 2 : 1);
  const uint64_t blocks = n ? (n + kBlock - 1) / kBlock : 1;
  hipLaunchKernelGGL(k_clear_words, dim3((unsigned)(blocks < 2048 ? blocks : 2048)), dim3(kBlock), 0,
                     s, static_cast<uint4*>(words), n, static_cast<u64*>(sync),
                     (uint32_t)kResSyncWords);
  return hipGetLastError();
}

hipError_t launch_pcg_resident_one(const ResArgs& a, const ResPlan& L, DType real, hipStream_t s) {
  if (active_recorder()) {
    return record_launch(RecKind::kPcgSolve, a, (unsigned)a.units, kResBlock, L.lds, (int)real,
                         L.tier, 0, nullptr);
  }
  ResBatch b{};
  b.n = 1;
  b.start[1] = a.units;
  b.v[0] = a;
  return launch_pcg_resident(b, real, L.tier, L.lds, s);
}

hipError_t launch_pcg_resident(const ResBatch& b, DType real, int tier, size_t lds, hipStream_t s) {
  if (b.n < 1 || b.n > kMaxResVolumes || lds > kMaxResLds) return hipErrorInvalidValue;
  for (int p = 0; p < b.n; ++p)
    if (b.v[p].units > kMaxResUnits || b.start[p + 1] - b.start[p] != b.v[p].units)
      return hipErrorInvalidValue;
  const unsigned grid = (unsigned)b.start[b.n];
  int64_t cells = 0, nodes = 0;
  for (int p = 0; p < b.n; ++p) {
    cells += b.v[p].ncell;
    nodes += b.v[p].nnode;
  }
#define RGP_RES(TR, ...)                                                                        \
  do {                                                                                          \
    const hipError_t e_ = hipFuncSetAttribute(                                                  \
        reinterpret_cast<const void*>(&k_pcg_resident<TR, __VA_ARGS__>),                      \
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxResLds);                           \
    if (e_ != hipSuccess) return e_;                                                            \
    RGP_LAUNCH_TN(kKindPcgSolve, b.v[0].maxit, cells, nodes, (k_pcg_resident<TR, __VA_ARGS__>), \
                  grid, kResBlock, lds, s, b);                                                  \
  } while (0)
  // (tier indexes kTiersF32, kTiersF64)
#define RGP_RES_TIER(TR, TIERS, K) \
  if (tier == K)                   \
  RGP_RES(TR, TIERS[K].npt, TIERS[K].xl, TIERS[K].keep, TIERS[K].xlds, TIERS[K].stride)
  if (tier < 0) return hipErrorInvalidValue;
  if (real == DType::F32) {
    RGP_RES_TIER(float, kTiersF32, 0);
    RGP_RES_TIER(float, kTiersF32, 1);
    RGP_RES_TIER(float, kTiersF32, 2);
    RGP_RES_TIER(float, kTiersF32, 3);
    RGP_RES_TIER(float, kTiersF32, 4);
    RGP_RES_TIER(float, kTiersF32, 5);
    if (tier > 5) return hipErrorInvalidValue;
  } else if (real == DType::F64) {
    RGP_RES_TIER(double, kTiersF64, 0);
    RGP_RES_TIER(double, kTiersF64, 1);
    RGP_RES_TIER(double, kTiersF64, 2);
    if (tier > 2) return hipErrorInvalidValue;
  } else {
    return hipErrorInvalidValue;
  }
#undef RGP_RES_TIER
#undef RGP_RES
  return hipGetLastError();
}

}  // namespace rgp
