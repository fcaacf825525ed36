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
// every wait ends.  If other work (another process, a kernel of another stream that holds CUs) keeps
// some of them out for kArriveTicks, those that have arrived share the units and work from memory
// (res_share), and whoever arrives later joins at the next iteration: no workgroup has to be
// resident but the first.  All sums are formed unit by unit in the same order, so the results are
// the same bits however many take part.
//
// What bounds it.  rgp_pcg_solve with 20 iterations, us per iteration, in one launch per iteration
// (a graph of them) and in this form, whose fixed costs are about 12 us of the 20 iterations:
//   25x25x17 FP32 6.6 / 5.0   72x84x56 11.2 / 6.5   144x168x111 27.5 / 13.3   200x200x132 48 / 24-25
//   32x32x24 FP64 7.4 / 4.4   90x90x90 FP64 22.2 / 10.6
// One workgroup's phases, us per iteration (read with wall_clock64 in a copy, which adds 0.1 to 1):
//                wait for outer p   stencil   its sums   wait for all sums   update   sum
//   25x25x17            1.4           0.5       0.4            1.0             1.0     4.3
//   72x84x56            2.1           0.5       0.5            2.0             1.0     6.0
//   144x168x111         4.0           2.2       1.6            2.1             2.5    12.4
//   200x200x132         4.9           6.1       3.4            2.3             6.1    22.7
// Small volumes: the two exchanges, about 1 us of latency each at least.  144x168x111: the outer p (8 MB
// of words each way), then FP64 issue.  Above that d and the couplings no longer fit the registers and
// are read again from the L2, a group of planes ahead of their use (with a position's planes read
// together, right before their use, the stencil took 9.6 and the update 12).
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
// 0.2 ms of the 100 MHz clock: about what a solve takes when all workgroups run, and less than what
// sharing it costs more than that
constexpr u64 kArriveTicks = 20000;
constexpr uint32_t kDecisionPolls = 1u << 28;   // (it comes, or the first workgroup never ran)

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
  int rank;                         // res_wait's answer
  int step, members;                // res_share: what the first workgroup published
  int arrived[kResBlock / kWave];   // res_share: newcomers seen by each wavefront
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

// How a solve goes on, as the first workgroup publishes it.
enum ResHow : uint32_t { kHowResident = 1, kHowShared = 2, kHowOver = 3 };
constexpr int kGoResident = -2, kLeave = -1;

// (Thread 0 of a workgroup but the first.)  Waits for the decision: kGoResident, this workgroup's
// rank among those that share the solve, or kLeave when the solve is over.
__device__ __forceinline__ int res_wait(const ResArgs& a, int ub) {
  for (uint32_t n = 0; n < kDecisionPolls; ++n) {
    const u64 how = word_get(a.sync + kResHow);
    if ((uint32_t)(how >> 32) == a.tag) {
      if ((uint32_t)how == kHowResident) return kGoResident;
      if ((uint32_t)how == kHowOver) return kLeave;
      const uint32_t mine = (uint32_t)word_get(a.sync + ub);
      if (mine >= kResMember) return (int)(mine - kResMember);
    }
    __builtin_amdgcn_s_sleep(1);
  }
  return kLeave;
}

// A given-up wait, in the outputs: a level stops with b unchanged and a status; a plain solve gives
// -1 iterations, a residual that is NaN, and (by the caller) NaN in x.
__device__ __forceinline__ void res_failed(const ResArgs& a) {
  if (a.gn_mode) {
    __hip_atomic_store(&a.st->gn_stop, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (a.st->status == 0) a.st->status = RGP_EHIP;
  }
  if (a.iters_out) *a.iters_out = -1;
  if (a.relres_out) *a.relres_out = __longlong_as_double(0x7ff8000000000000LL);
}

// (res_share; res_body has the same lines in place: called from there, with the addresses formed on
// each iteration, 144x168x111 took 2.5 % longer.)  The sums of all units, added in a fixed order, on
// every thread.  False (and `flag` set) when the wait for one was given up.
__device__ __forceinline__ bool res_totals(const ResArgs& a, uint32_t tag, double (*sh)[8], int& flag,
                                           double (&ts)[7]) {
  const u64* part = a.part + (size_t)(tag & 1u) * (kResSumStride * kMaxResUnits);
  const int t = threadIdx.x;
  double us;
  const bool got = a.units <= 64    ? sums_get<2>(part, a.units, tag, a.spins, us)
                   : a.units <= 128 ? sums_get<4>(part, a.units, tag, a.spins, us)
                                    : sums_get<8>(part, a.units, tag, a.spins, us);
  if (!got) flag = 1;
  __syncthreads();   // (the row sums of this unit are read)
  if ((t & 1) == 0) sh[t / 16][(t & 15) / 2] = us;
  __syncthreads();
  if (flag) return false;
  const double tot = res_row_sum(sh);
#pragma unroll
  for (int k = 0; k < 7; ++k) ts[k] = read_lane(tot, 8 * k);
  return true;
}
__device__ __forceinline__ void res_put_sums(const ResArgs& a, int ub, uint32_t tag, double s) {
  const int t = threadIdx.x;
  if (t < 56 && (t & 7) == 0) {
    u64* mine = a.part + (size_t)(tag & 1u) * (kResSumStride * kMaxResUnits) + ub * kResSumStride + t / 4;
    word_put(mine, tagged(tag, (uint32_t)__double2loint(s)));
    word_put(mine + 1, tagged(tag, (uint32_t)__double2hiint(s)));
  }
}

// The solve by the workgroups that have arrived, `rank` being this one's place among them (the first
// workgroup has 0): member r of k takes the units r, r + k, ...  The vectors are in memory: r and p in
// the two spare arrays, w in the first word array (its nodes are cleared again at the end).  A step
// is the start of the vectors (step 0) or an iteration.  The first workgroup opens each step: it
// waits until every member has finished the one before, admits newcomers, and publishes the number
// of members and the scalars that a newcomer lacks.  A member's stores are released before it says
// that it has finished and acquired when the next step opens, so units may change hands; within a
// step the exchange of the sums parts the reads of the old p from the stores of the new one.
// 20 iterations at 144x168x111 FP32: 1.15 ms by 128 workgroups and 5.2 ms by 16 (resident 0.27, one
// launch per iteration 0.53); 72x84x56: 0.52 and 1.1 ms (0.13, 0.36).  The code of the smallest
// variants stays within their 128 registers with 2 planes (FP32) and 1 (FP64) at a time.
template <typename TR>
__device__ __forceinline__ void res_share(const ResArgs& a, int rank, ResShared& m) {
  constexpr uint32_t kSz = sizeof(TR);
  constexpr int kG = sizeof(TR) == 4 ? 2 : 1;   // planes whose loads are in flight together
  const int t = threadIdx.x, role = a.role, na = a.na, nb = a.nb, no = a.no, P = a.P;
  const uint32_t nbytes = a.nnode * kSz;
  const BRes rD = bres(a.diag, nbytes), rO = bres(a.off, nbytes), rB = bres(a.rhs, nbytes);
  const BRes rX = bres(a.x, nbytes), rR = bres(a.spare_r, nbytes), rP = bres(a.spare_p, nbytes);
  const BRes rW = bres(a.words, nbytes);
  const TR sg = (TR)a.rhs_sign;
  TR c_o, c_a, c_b;
  res_couplings<TR>(a, role, c_o, c_a, c_b);
  auto at = [&](bool ok, uint32_t n) -> uint32_t { return ok ? n * kSz : kNullOff; };
  // body(plane position, node in the unit's first plane) over this thread's positions of a unit, which
  // are those of the resident form
  auto positions = [&](const ResUnit& un, auto body) {
    for (int j = t; j < un.teff; j += kResBlock) {
      const int l = j + nb < un.teff ? j + nb : j + nb - un.teff;
      const int f = un.f0 + l;
      body(f, (uint32_t)un.o0 * (uint32_t)P + (uint32_t)f);
    }
  };
  bool in = t == 0;   // (first workgroup: workgroup t is a member)
  bool lost = false;
  int k = 1, it = rank == 0 ? 0 : -1;
  double bn = 0.0, rel = 0.0;
  PcgSlot cur{};
  while (true) {
    bool late = false;
    if (rank == 0) {
      if (it > 0 && t > 0 && t < k) {
        late = true;
        for (uint32_t n = 0; n <= a.spins && late; ++n) {
          late = (uint32_t)(word_get(a.sync + kResDone + t) >> 32) != a.tag + (uint32_t)it - 1u;
          if (late) __builtin_amdgcn_s_sleep(1);
        }
      }
      const int room = min(a.units, a.most + it * a.grow), wv = t / kWave;
      const bool want = t > 0 && t < a.units && !in && word_get(a.sync + t) == tagged(a.tag, 1u);
      const u64 b = __ballot(want);
      if ((t & (kWave - 1)) == 0) m.arrived[wv] = __popcll(b);
      __syncthreads();
      int r = k + __popcll(b & ((1ull << (t & (kWave - 1))) - 1ull)), all = k;
      for (int j = 0; j < kResBlock / kWave; ++j) {
        r += j < wv ? m.arrived[j] : 0;
        all += m.arrived[j];
      }
      if (want && r < room) {
        word_put(a.sync + t, tagged(a.tag, kResMember + (uint32_t)r));
        in = true;
      }
      k = uniform(min(all, room));
      if (t == 0) {
        const uint32_t tag = a.tag + (uint32_t)it;
        word_put(a.sync + kResScal + 0, tagged(tag, (uint32_t)__double2loint(bn)));
        word_put(a.sync + kResScal + 1, tagged(tag, (uint32_t)__double2hiint(bn)));
        word_put(a.sync + kResScal + 2, tagged(tag, (uint32_t)__double2loint(rel)));
        word_put(a.sync + kResScal + 3, tagged(tag, (uint32_t)__double2hiint(rel)));
        word_put(a.sync + kResStep, tagged(tag, (uint32_t)k));
      }
    } else {
      if (t == 0) {
        late = true;
        for (uint32_t n = 0; n <= a.spins && late; ++n) {
          const u64 v = word_get(a.sync + kResStep);
          const uint32_t st = (uint32_t)(v >> 32) - a.tag;
          late = it < 0 ? st > (uint32_t)a.maxit || (uint32_t)v <= (uint32_t)rank : st != (uint32_t)it;
          m.step = (int)st;
          m.members = (int)(uint32_t)v;
          if (late) __builtin_amdgcn_s_sleep(1);
        }
      }
      __syncthreads();
      it = uniform(m.step);
      k = uniform(m.members);
    }
    lost = __syncthreads_or(late);
    if (lost) break;
    if (rank > 0) {
      const uint32_t n[2] = {0u, 1u};
      double v[2];
      late = !values_get<double, 2>(a.sync + kResScal, n, a.tag + (uint32_t)it, a.spins, v);
      bn = v[0];
      rel = v[1];
      lost = __syncthreads_or(late);
      if (lost) break;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    if (it == 0) {
      for (int u = rank; u < a.units; u += k) {
        const ResUnit un = res_unit(a, u);
        positions(un, [&](int, uint32_t n0) {
          for (int q = 0; q < un.np; ++q) {
            const uint32_t o = (n0 + (uint32_t)q * (uint32_t)P) * kSz;
            const TR rv = sg * bld<TR>(rB, o);
            bst<TR>(rR, o, rv);
            bst<TR>(rP, o, fmad(TR(0), TR(0), rv * (TR(1) / bld<TR>(rD, o))));
            bst<TR>(rX, o, TR(0));
          }
        });
      }
    } else {
      const uint32_t tag = a.tag + (uint32_t)it;
      for (int u = rank; u < a.units; u += k) {   // w = H p and the unit's sums
        const ResUnit un = res_unit(a, u);
        double acc[7] = {0, 0, 0, 0, 0, 0, 0};
        positions(un, [&](int f, uint32_t n0) {
          const int ia = f / nb, ib = f - ia * nb;
          TR pom = bld<TR>(rP, at(un.o0 > 0, n0 - (uint32_t)P)), pk = bld<TR>(rP, n0 * kSz);
          TR ol = role == 0 ? bld<TR>(rO, at(un.o0 > 0, n0 - (uint32_t)P)) : TR(0);
          for (int q0 = 0; q0 < un.np; q0 += kG) {
            TR pop[kG], pam[kG], pap[kG], pbm[kG], pbp[kG], d[kG], ou[kG], lo[kG], r[kG];
#pragma unroll
            for (int g = 0; g < kG; ++g) {
              const bool on = q0 + g < un.np;
              const uint32_t n = n0 + (uint32_t)(q0 + g) * (uint32_t)P;
              pop[g] = bld<TR>(rP, at(on && un.o0 + q0 + g < no - 1, n + (uint32_t)P));
              pam[g] = bld<TR>(rP, at(on && ia > 0, n - (uint32_t)nb));
              pap[g] = bld<TR>(rP, at(on && ia < na - 1, n + (uint32_t)nb));
              pbm[g] = bld<TR>(rP, at(on && ib > 0, n - 1u));
              pbp[g] = bld<TR>(rP, at(on && ib < nb - 1, n + 1u));
              d[g] = bld<TR>(rD, at(on, n));
              ou[g] = bld<TR>(rO, at(on, n));
              lo[g] = bld<TR>(rO, at(on && ((role == 1 && ia > 0) || (role == 2 && ib > 0)),
                                     n - (role == 1 ? (uint32_t)nb : 1u)));
              r[g] = bld<TR>(rR, at(on, n));
            }
#pragma unroll
            for (int g = 0; g < kG; ++g) {
              if (q0 + g >= un.np) break;
              if (role != 0) ol = lo[g];
              const TR wv = res_stencil<TR>(role, d[g], pk, pom, pop[g], pam[g], pap[g], pbm[g],
                                            pbp[g], ol, ou[g], c_o, c_a, c_b);
              bst<TR>(rW, (n0 + (uint32_t)(q0 + g) * (uint32_t)P) * kSz, wv);
              const TR inv = TR(1) / d[g];
              res_sums<TR>(acc, pk, wv, r[g], r[g] * inv, inv);
              pom = pk;
              pk = pop[g];
              if (role == 0) ol = ou[g];
            }
          }
        });
        res_put_sums(a, u, tag, res_block_sum(acc, m.sh));
        __syncthreads();   // m.sh is read
      }
      double ts[7];
      if (!res_totals(a, tag, m.sh, m.flag, ts)) {
        lost = true;
        break;
      }
      PcgSlot prev{};
      prev.bnorm2 = bn;
      prev.relres = rel;
      bool fin = false;
      cur = pcg_advance(prev, ts, it, a.maxit, a.rtol, fin);
      bn = cur.bnorm2;
      rel = cur.relres;
      if (cur.status == kPcgDone) break;   // keep x
      const TR al = (TR)cur.alpha, be = (TR)cur.beta;
      for (int u = rank; u < a.units; u += k) {
        const ResUnit un = res_unit(a, u);
        positions(un, [&](int, uint32_t n0) {
          for (int q0 = 0; q0 < un.np; q0 += kG) {
            TR x[kG], r[kG], p[kG], w[kG], d[kG];
#pragma unroll
            for (int g = 0; g < kG; ++g) {
              const uint32_t o = at(q0 + g < un.np, n0 + (uint32_t)(q0 + g) * (uint32_t)P);
              x[g] = bld<TR>(rX, o);
              r[g] = bld<TR>(rR, o);
              p[g] = bld<TR>(rP, o);
              w[g] = bld<TR>(rW, o);
              d[g] = bld<TR>(rD, o);
            }
#pragma unroll
            for (int g = 0; g < kG; ++g) {
              const uint32_t o = at(q0 + g < un.np, n0 + (uint32_t)(q0 + g) * (uint32_t)P);
              const TR rv = fmad(-al, w[g], r[g]);
              bst<TR>(rX, o, fin ? x[g] + al * p[g] : fmad(al, p[g], x[g]));
              bst<TR>(rR, o, rv);
              bst<TR>(rP, o, fmad(be, p[g], rv * (TR(1) / d[g])));
            }
          }
        });
      }
      if (fin) break;
    }
    __syncthreads();
    if (t == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      if (rank > 0) word_put(a.sync + kResDone + rank, tagged(a.tag + (uint32_t)it, 1u));
    }
    ++it;
  }
  for (int u = rank; u < a.units; u += k) {
    const ResUnit un = res_unit(a, u);
    positions(un, [&](int, uint32_t n0) {
      for (int q = 0; q < un.np; ++q) {
        const uint32_t o = (n0 + (uint32_t)q * (uint32_t)P) * kSz;
        bst<TR>(rW, o, TR(0));
        if (lost) bst<TR>(rX, o, (TR)__builtin_nan(""));
      }
    });
  }
  if (t == 0) {
    if (lost)
      res_failed(a);
    else if (rank == 0)
      res_outputs(a, cur);
    if (rank == 0) word_put(a.sync + kResHow, tagged(a.tag, kHowOver));
  }
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
// and publishes first.  Returns this workgroup's rank among those that share the solve, where not
// all could become resident; else negative.
template <typename TR, int ROLE, int NPT, int XL, int KEEP, int XN, int S>
__device__ __forceinline__ int res_body(const ResArgs& a, int ub, ResShared& m) {
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
    if (stop || viol) return kLeave;   // the same in every workgroup
  }

  // residency: all arrived, or those that have share the solve
  if (ub == 0) {
    bool ok = a.most >= a.units;
    if (ok && t < a.units) {
      const u64 t0 = wall_clock64();
      while ((uint32_t)(word_get(a.sync + t) >> 32) != tag0) {
        if (wall_clock64() - t0 > kArriveTicks + a.patience) {
          ok = false;
          break;
        }
      }
    }
    const bool share = __syncthreads_or(!ok);
    if (t == 0) word_put(a.sync + kResHow, tagged(tag0, share ? kHowShared : kHowResident));
    if (share) return 0;
  } else {
    if (t == 0) m.rank = res_wait(a, ub);
    __syncthreads();
    const int rank = uniform(m.rank);
    if (rank != kGoResident) return rank;
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
  const bool failed = lost || flag;   // some workgroup stands still
  if (failed && t == 0) res_failed(a);
#pragma unroll
  for (int q = 0; q < XL; ++q)
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const TR xv = i < XN ? xlds[(i * XL + q) * kResBlock] : x[q][i >= XN ? i - XN : 0];
      bst<TR>(rX, at(q < np && has(i, kOwn), node(q, i)), failed ? (TR)__builtin_nan("") : xv);
    }
  if (failed) return kLeave;
  if (ub == 0 && t == 0) {
    PcgSlot c{};
    c.iters = its;
    c.relres = rel;
    res_outputs(a, c);
  }
  return kLeave;
}

template <typename TR, int NPT, int XL, int KEEP, int XN, int S>
__global__ __launch_bounds__(kResBlock, XL <= 2 ? 4 : 2) void k_pcg_resident(ResBatch b) {
  int p = 0;
  while (p + 1 < b.n && (int)blockIdx.x >= b.start[p + 1]) ++p;
  const ResArgs& a = b.v[p];
  const int ub = (int)blockIdx.x - b.start[p];
  if (ub >= a.units) return;
  __shared__ ResShared m;
  int rank;
  if (a.role == 0)
    rank = res_body<TR, 0, NPT, XL, KEEP, XN, S>(a, ub, m);
  else if (a.role == 1)
    rank = res_body<TR, 1, NPT, XL, KEEP, XN, S>(a, ub, m);
  else
    rank = res_body<TR, 2, NPT, XL, KEEP, XN, S>(a, ub, m);
  if (rank >= 0) res_share<TR>(a, rank, m);
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
  a.most = (int32_t)L.m.units;
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
