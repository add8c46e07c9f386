// mg_eval_lane.h -- the evaluation kernel in the lane-per-link layout: cost
// and adjoint of every (candidate, waypoint row) of a batch in one launch.
// Instantiated per lane layout in mg_eval_l*.hip so the variants compile in
// parallel.
#pragma once

#include "mg_eval.h"

namespace mg {
namespace {

// Copy of a lane's 3x4 transform from the lane `OFF` below (row_shr) or
// above (row_shl) within the 16-lane DPP row.
template <int CTRL>
__device__ __forceinline__ void dpp12(const float* src, float* dst) {
#pragma unroll
  for (int e = 0; e < 12; ++e) dst[e] = dpp<CTRL>(src[e]);
}

// One Hillis-Steele step of the prefix product along a chain:
// P <- P(lane - OFF) * P for lanes at least OFF past their chain start.
template <int OFF>
__device__ __forceinline__ void scan_step(float* P, bool active) {
  float Q[12];
  dpp12<0x110 + OFF>(P, Q);          // row_shr:OFF
  float R[12];
#pragma unroll
  for (int r = 0; r < 3; ++r) {
    const float q0 = Q[r * 4 + 0], q1 = Q[r * 4 + 1], q2 = Q[r * 4 + 2], q3 = Q[r * 4 + 3];
    R[r * 4 + 0] = q0 * P[0] + q1 * P[4] + q2 * P[8];
    R[r * 4 + 1] = q0 * P[1] + q1 * P[5] + q2 * P[9];
    R[r * 4 + 2] = q0 * P[2] + q1 * P[6] + q2 * P[10];
    R[r * 4 + 3] = q0 * P[3] + q1 * P[7] + q2 * P[11] + q3;
  }
#pragma unroll
  for (int e = 0; e < 12; ++e) P[e] = active ? R[e] : P[e];
}

// One step of the suffix sum of a 6-vector along a chain (row_shl:OFF).
template <int OFF>
__device__ __forceinline__ void suffix_step(float* W, bool active) {
#pragma unroll
  for (int e = 0; e < 6; ++e) {
    const float v = dpp<0x100 + OFF>(W[e]);
    W[e] = active ? W[e] + v : W[e];
  }
}

// Pose of this lane's link at its joint value q: the local transform
// F_l Rz(q) from the Tab.6 closed form (columns 0 and 1 mix, 2 and 3 are
// F's), then the prefix product along the chain (pos = lanes past the chain
// start).  Lanes without a link hold the identity.
template <int LPE>
__device__ __forceinline__ void link_pose(const float4& f0, const float4& f1, const float4& f2, bool on, int pos,
                                          float q, float* T) {
  const float sn = __sinf(q), cs = __cosf(q);
  T[0] = f0.x * cs + f0.y * sn;  T[1] = f0.y * cs - f0.x * sn;  T[2] = f0.z;  T[3] = f0.w;
  T[4] = f1.x * cs + f1.y * sn;  T[5] = f1.y * cs - f1.x * sn;  T[6] = f1.z;  T[7] = f1.w;
  T[8] = f2.x * cs + f2.y * sn;  T[9] = f2.y * cs - f2.x * sn;  T[10] = f2.z; T[11] = f2.w;
  if (!on) identity(T);
  scan_step<1>(T, pos >= 1);
  scan_step<2>(T, pos >= 2);
  scan_step<4>(T, pos >= 4);
  if (LPE > 8) scan_step<8>(T, pos >= 8);
}

// The same pose formed link by link from the root, with the operations of the
// wave-per-link layout's chain_fk (`steps` links follow the first on the longest
// chain): bit for bit its pose.
__device__ __forceinline__ void link_pose_serial(const float4& f0, const float4& f1, const float4& f2, bool on,
                                                 int pos, int steps, float q, float* T) {
  const float sn = __sinf(q), cs = __cosf(q);
  T[0] = f0.x * cs + f0.y * sn;  T[1] = f0.y * cs - f0.x * sn;  T[2] = f0.z;  T[3] = f0.w;
  T[4] = f1.x * cs + f1.y * sn;  T[5] = f1.y * cs - f1.x * sn;  T[6] = f1.z;  T[7] = f1.w;
  T[8] = f2.x * cs + f2.y * sn;  T[9] = f2.y * cs - f2.x * sn;  T[10] = f2.z; T[11] = f2.w;
  // (step i leaves the poses of the chains' first i + 1 links as they are)
  for (int i = 0; i < steps; ++i) {
    float P[12];
    dpp12<0x111>(T, P);                // row_shr:1, the parent's pose
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const float t0 = P[r * 4 + 0], t1 = P[r * 4 + 1], t2 = P[r * 4 + 2], t3 = P[r * 4 + 3];
      const float u0 = t0 * f0.x + t1 * f1.x + t2 * f2.x;
      const float u1 = t0 * f0.y + t1 * f1.y + t2 * f2.y;
      const float u2 = t0 * f0.z + t1 * f1.z + t2 * f2.z;
      const float u3 = t0 * f0.w + t1 * f1.w + t2 * f2.w + t3;
      T[r * 4 + 0] = pos >= 1 ? u0 * cs + u1 * sn : T[r * 4 + 0];
      T[r * 4 + 1] = pos >= 1 ? u1 * cs - u0 * sn : T[r * 4 + 1];
      T[r * 4 + 2] = pos >= 1 ? u2 : T[r * 4 + 2];
      T[r * 4 + 3] = pos >= 1 ? u3 : T[r * 4 + 3];
    }
  }
  if (!on) identity(T);
}

// Lane l of an evaluation owns link l (its pose, sphere ball, joint and
// pose terms); an evaluation takes LPE lanes (8 or 16, one per link) times H
// copies that split the world's cuboids, and a wave holds 64 / (LPE H)
// evaluations, so everything an evaluation needs stays inside one wave: the
// four waves of a workgroup only share the staged rows, tables and cuboid
// tile (one barrier per tile).
//
// What bounds this kernel is the vector work on (sphere, cuboid) pairs.  Of
// the M N pairs of an evaluation only a few per cent lie within r + eta, but
// which ones differs from lane to lane, so a loop over cuboids that the
// whole wave walks runs the exact distance for nearly every pair that any of
// its lanes needs.  The pairs are therefore compacted in three steps, each
// spreading its work over the wave's 64 lanes through queues in LDS:
//   1. (link, cuboid) pairs, one per lane: the ball around the link's
//      spheres over a group of the wave's evaluations against the cuboid;
//   2. (evaluation, link, cuboid), one per lane: the evaluation's own balls
//      around the two parts of the link's spheres;
//   3. (evaluation, part, cuboid) items, one per lane (several lanes per item,
//      each with a share of the spheres, when few are left): the face test
//      of every sphere of the part and, where it passes, the exact term.
// With swept collision the spheres whose trace may take a step (one in ten
// of those that pass the face test, where segments are short) go through a
// second queue, one (sphere, cuboid) pair and side per lane.  (Traced where
// the exact term is, 64 lanes waited for the few that step: 6144 rows of two
// arms among 500 cuboids, K = 4, took 579 us, 440 with the queue.)  A wave
// then holds neighbouring rows of one candidate and shares their poses, which
// lets three workgroups into a CU's LDS instead of two (410 us, now 315; over
// other inputs of these sizes a launch takes 240 to 315).
// The lanes' sums go back to the owners (evaluation, link) through an LDS
// row per lane: each owner finds its rows from six ballots of the owners'
// bits and adds them in lane order, so the results are deterministic.  (LDS
// float atomics cost 194 cycles per wave instruction on gfx950, whatever the
// addresses: eight of them per 64 pairs bounded this kernel, 411 us against
// the figure below on 524288 inverse-kinematics evaluations.)
// The culls are exact: the signed distance is 1-Lipschitz, so a ball whose
// centre is further from a cuboid than its radius and eta holds no sphere that
// matters (for spheres max(|p| - h), which bounds the distance from below,
// does), and a pair they drop adds no cost and cannot lower the clearance
// clamped at eta.
//
// Measured, us per launch (cost and gradient of every candidate), this layout
// with its best number of copies against the best wave-per-link layout:
//   524288 single configurations, 40 cuboids (4096 x 32 seeds, K = 4)  216 / 634
//   64 problems, 84616 rows, 5 to 200 cuboids each, K = 4              151 / 236
//   two arms, 120 spheres, 500 cuboids, swept, 6144 rows, K = 4        315 / 1074
//   the same without the sweep                                         180 / 298
//   128 seeds x 32, 40 cuboids, K = 8                                  16.1 / 24.1
//   32 seeds x 32, 40 cuboids, K = 8                                   11.1 / 11.6
//   4 seeds x 32, 10 cuboids, K = 4                                    7.6 / 9.4
// Large batches are bound by the vector instructions issued (some 280 per
// evaluation, half of them kinematics, joint and pose terms, at one per four
// cycles and SIMD), small ones by one wave's chain of them.

// Compiler fence between LDS writes and reads of different lanes of one wave
// (the hardware runs a wave's LDS instructions in order).
__device__ __forceinline__ void wave_lds_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// Sum (or minimum) over the H copies of an evaluation: the lanes that differ
// in the bits from LPE to LPE H / 2.  Every lane gets the same bits.
template <int BIT>
__device__ __forceinline__ float lane_xor(float v, int lane) {
  if constexpr (BIT == 8) return dpp<0x128>(v);    // row_ror:8
  const auto r = BIT == 16 ? __builtin_amdgcn_permlane16_swap(__float_as_int(v), __float_as_int(v), false, false)
                           : __builtin_amdgcn_permlane32_swap(__float_as_int(v), __float_as_int(v), false, false);
  return __int_as_float((int)(lane & BIT ? r[0] : r[1]));
}
template <int LPE, int H, typename OP>
__device__ __forceinline__ float copies_op(float v, OP op) {
  const int lane = threadIdx.x % kWave;
  if constexpr (H >= 2) v = op(v, lane_xor<LPE>(v, lane));
  if constexpr (H >= 4) v = op(v, lane_xor<2 * LPE>(v, lane));
  if constexpr (H >= 8) v = op(v, lane_xor<4 * LPE>(v, lane));
  return v;
}
// Minimum of each of v[0..N) over GE (a power of two) neighbouring evaluations
// of a wave, STRIDE lanes each.
template <int STRIDE, int N>
__device__ __forceinline__ void evals_min(float* v, int GE) {
  if (STRIDE <= 8 && GE * STRIDE > 8) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = fminf(v[i], dpp<0x128>(v[i]));   // row_ror:8
  }
  if (STRIDE <= 16 && GE * STRIDE > 16) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = swap16_min(v[i]);
  }
  if (STRIDE <= 32 && GE * STRIDE > 32) {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = swap32_min(v[i]);
  }
}
// Stores and loads that meet between workgroups of one launch (the XCDs' L2
// caches are not coherent): through to memory, past the caches.
__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int lanes_below(uint64_t m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0));
}

constexpr int kLplWaves = kBlock / kWave;
constexpr int kLplTile = 64;      // cuboids staged per tile
constexpr int kLplPairs = 2 * kWave;   // entries of the (group, link, cuboid) queue
constexpr int kLplTrace = 5 * kWave / 2;   // entries of the trace queue (two spheres are tested between checks)
// float4 between the rows of a staged tile (one more than the cuboids: the
// four rows of a cuboid, read together, then lie in different banks)
constexpr int kLplStride = kLplTile + 1;

// Most groups of evaluations a wave's links are bounded over (one where the
// balls of several would cost a workgroup per CU).
__host__ __device__ constexpr int lpl_groups(int lpe, int H) {
  const int epw = kWave / (lpe * H);
  return lpe > 8 ? 1 : epw < 4 ? epw : 4;
}

// LDS of a lane-per-link workgroup, float offsets (kept a multiple of 4).
// Shared: rows of x and of d (or the particle variance), limits and start,
// goals, tool transforms, sphere slots, the cuboid tile [4][kLplStride]
// float4, in particle mode the draws; then per wave: link poses (and with
// swept collision the poses before the wave's rows, after them and of the
// start, the trace's reach and where each evaluation's neighbours are), the
// evaluations' and the links' balls, the lanes' sums, and the queues.
struct LplLds {
  int x, d, lim, goal, etf, slot, box, eps, wave, wave_size, total;
};
__host__ __device__ inline LplLds lpl_lds(int lpe, int H, int rb, int kb, int D, int slots, bool sw, bool pm,
                                         bool grad) {
  LplLds o;
  const int rs = rb + 8, ow = kWave / H;
  int at = 0;
  auto take = [&at](int n) {
    const int r = at;
    at += (n + 3) & ~3;
    return r;
  };
  o.x = take(rs * D);
  o.d = take(rs * D);
  o.lim = take(3 * D);
  o.goal = take(kMaxEE * 7);
  o.etf = take(kMaxEE * 12);
  o.slot = take(lpe * slots * 4);
  o.box = take(kLplStride * 16);
  o.eps = take(pm ? kb * rs * D : 0);
  o.wave = at;
  o.wave_size = 12 * ow + (sw ? 36 * lpe + (ow + 3) / 4 * 4 + 8 : 0) + 8 * ow +
                4 * lpe * (sw ? 1 : lpl_groups(lpe, H)) + (grad ? 8 : 4) * (kWave + 2) + (sw ? kLplTrace / 2 : 0) +
                (kLplPairs + 3 * kWave) / 2;
  o.total = at + kLplWaves * o.wave_size;
  return o;
}

// One sphere against one cuboid in the box frame: cost, clearance and, with
// GRAD, the box-frame force b (d cost / d centre) and its moment m about the
// box origin, all accumulated, and the distance sdf.  ax.. = |p| - h, m3 their
// maximum.
template <bool GRAD>
__device__ __forceinline__ void pair_term(float px, float py, float pz, float ax, float ay, float az, float m3,
                                          float r, float w, float eta, float inv_eta, float& cost, float& mc,
                                          float* b, float* m, float& sdf) {
  const float qx = fmaxf(ax, 0.0f), qy = fmaxf(ay, 0.0f), qz = fmaxf(az, 0.0f);
  const float n2 = qx * qx + qy * qy + qz * qz;
  const bool out = n2 > 0.0f;
  const float n = __builtin_amdgcn_sqrtf(n2);
  sdf = out ? n : m3;
  mc = fminf(mc, sdf - r);
  // Eq.(10): the slope u / eta clamped to [0, 1], the cost its integral
  const float u = r - sdf + eta;
  const float slope = fminf(fmaxf(u * inv_eta, 0.0f), 1.0f);
  cost = fmaf(w * slope, fmaf(-0.5f * eta, slope, u), cost);
  if (GRAD) {
    const float f = -w * slope;
    const float fo = out ? f * __builtin_amdgcn_rcpf(n) : f;
    // inside: the nearest face, lowest axis on ties
    const bool ix = ax == m3, iy = !ix && ay == m3;
    const float vx = fo * (out ? qx : ix ? 1.0f : 0.0f);
    const float vy = fo * (out ? qy : iy ? 1.0f : 0.0f);
    const float vz = fo * (out ? qz : (ix || iy) ? 0.0f : 1.0f);
    const float gx = px >= 0.0f ? vx : -vx, gy = py >= 0.0f ? vy : -vy, gz = pz >= 0.0f ? vz : -vz;
    b[0] += gx; b[1] += gy; b[2] += gz;
    m[0] = fmaf(py, gz, fmaf(-pz, gy, m[0]));
    m[1] = fmaf(pz, gx, fmaf(-px, gz, m[1]));
    m[2] = fmaf(px, gy, fmaf(-py, gx, m[2]));
  }
}

// A link-frame point in the world: row r of the pose (a, w) times (x, y, z, 1).
// (Spelled out, as the compiler contracts the same sum in the wave-per-link
// kernels: left to itself it picks the order of the products by their operands.)
__device__ __forceinline__ float dot3(float ax, float ay, float az, float x, float y, float z) {
  return fmaf(az, z, fmaf(ax, x, ay * y));
}
__device__ __forceinline__ float row_point(const float4& a, const float4& p) {
  return dot3(a.x, a.y, a.z, p.x, p.y, p.z) + a.w;
}

// The trace toward one neighbouring waypoint (Alg.11-12): direction u (world,
// unscaled), from p (box frame) with distance sdf; the samples' gradients in
// the box frame.  (The operations of the wave-per-link layout's
// sweep_pair_box: where a sample lies decides whether it counts at all.)
template <bool GRAD>
__device__ __forceinline__ void trace_term(float ux, float uy, float uz, const float4& A0, const float4& A1,
                                           const float4& A2, int steps, float px, float py, float pz,
                                           const float4& Hh, float sdf, float r, float w, float eta, float inv_eta,
                                           float& cost, float* b) {
  const float rh = r + eta;
  const float len = sqrtf(dot3(ux, uy, uz, ux, uy, uz));
  const float half = 0.5f * len;
  float j = sdf < rh ? rh : sdf - rh;
  if (!(len > 0.0f && j < half)) return;
  const float il = 1.0f / len;
  ux *= il; uy *= il; uz *= il;
  const float vx = dot3(A0.x, A0.y, A0.z, ux, uy, uz);
  const float vy = dot3(A1.x, A1.y, A1.z, ux, uy, uz);
  const float vz = dot3(A2.x, A2.y, A2.z, ux, uy, uz);
  for (int st = 0; st < steps && j < half; ++st) {
    const float qx = fmaf(j, vx, px), qy = fmaf(j, vy, py), qz = fmaf(j, vz, pz);
    float s2;
    if (GRAD) {
      float gx, gy, gz;
      s2 = box_sdf(qx, qy, qz, fabsf(qx) - Hh.x, fabsf(qy) - Hh.y, fabsf(qz) - Hh.z, gx, gy, gz);
      dc_term_box(s2, gx, gy, gz, r, w, eta, inv_eta, cost, b[0], b[1], b[2]);
    } else {
      s2 = box_dist(fabsf(qx) - Hh.x, fabsf(qy) - Hh.y, fabsf(qz) - Hh.z);
      dc_cost(s2, r, w, eta, inv_eta, cost);
    }
    j += s2 - rh > 0.0f ? s2 - rh : rh;
  }
}

template <int LPE, int H, bool CAND, bool GRAD, bool SW>
__global__ __launch_bounds__(kBlock) void eval_kernel(const EvalArgs a) {
  constexpr int EPW = kWave / (LPE * H);           // evaluations per wave
  constexpr int OW = EPW * LPE;                    // owners (evaluation, link) per wave
  extern __shared__ float s_mem[];
  warm_kernargs<sizeof(EvalArgs)>();

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  const int lane = tid % kWave;
  const int l = lane % LPE, sub = lane / LPE % H, ew = lane / (LPE * H);
  const int owner = ew * LPE + l;
  const int D = a.rb.dof, L = a.rb.n_links, slots = 2 * a.ln.used, n_ee = a.rb.n_ee;
  const int KB = a.ln.kb, RB = a.ln.rb;            // candidates and rows per workgroup (KB RB evaluations)
  const int bx = blockIdx.x;

  // ---- this workgroup's problem: by arithmetic when all problems have one
  //      size, else from the table of first workgroups (64 entries a step) ----
  int p = 0, c = bx;
  if (a.ln.uni_rows > 0) {
    if (a.P > 1) {
      const int cpp = (a.ln.uni_rows + RB - 1) / RB;
      p = bx / cpp;
      c = bx - p * cpp;
    }
  } else {
    int lo = 0, n = a.P;                            // the last p in [lo, lo + n) with prefix[p] <= bx
    while (n > 1) {
      const int st = (n + kWave - 1) / kWave;
      const int i = lo + min(lane * st, n - 1);
      const bool le = lane * st < n && a.chunk_prefix[i] <= bx;
      const int k = __popcll(__ballot(le)) - 1;
      lo += k * st;
      n = min(st, n - k * st);
    }
    p = __builtin_amdgcn_readfirstlane(lo);
    c = bx - a.chunk_prefix[p];
  }
  int S, T, row0, seed0, w0, w1;
  if (a.wl.one.S > 0) {
    const v4i pr = ((cv4i*)(a.prob))[1];
    S = a.wl.one.S; T = a.wl.one.T; row0 = 0; seed0 = 0; w0 = pr.y; w1 = pr.z;
  } else {
    cv4i* pr = (cv4i*)(a.prob + p);
    const v4i p0 = pr[0], p1 = pr[1];
    S = p0.x; T = p0.y; row0 = p0.w; seed0 = p1.x; w0 = p1.y; w1 = p1.z;
  }
  Problem pb;
  pb.S = S; pb.T = T; pb.world = 0; pb.row0 = row0; pb.seed0 = 0; pb.box_lo = w0; pb.box_hi = w1; pb.pad = 0;
  const int nrows = S * T, first = c * RB;         // this workgroup's first row within the problem

  // evaluation of this lane: candidates of a row side by side
  // (swept: a wave's evaluations are neighbouring rows of one candidate, so
  // that a row's neighbours are evaluations of the wave but at its ends)
  const int ei = wave * EPW + ew;
  const bool by_row = SW && T > 1;
  const int k = blockIdx.y * KB + (by_row ? ei / RB : ei % KB);
  const int rloc = first + (by_row ? ei % RB : ei / KB);
  const bool valid = rloc < nrows;
  const int rl = valid ? rloc : nrows - 1;
  const int t = rl % T;                            // waypoint t + 1 of its seed
  const int row = row0 + rl;
  const bool pm = CAND && !GRAD && a.var != nullptr;

  const LplLds o = lpl_lds(LPE, H, RB, KB, D, slots, SW, pm, GRAD);
  float* s_x = s_mem + o.x;
  float* s_d = s_mem + o.d;
  float* s_lim = s_mem + o.lim;
  float* s_goal = s_mem + o.goal;
  float* s_etf = s_mem + o.etf;
  float4* s_slot = reinterpret_cast<float4*>(s_mem + o.slot);
  float4* s_box = reinterpret_cast<float4*>(s_mem + o.box);
  float* s_eps = s_mem + o.eps;
  float* s_w = s_mem + o.wave + wave * o.wave_size;
  float4* s_T = reinterpret_cast<float4*>(s_w);                            // [3][OW]
  float4* s_X = s_T + 3 * OW;                                              // [3][3 LPE] (SW)
  float4* s_ball = s_X + (SW ? 9 * LPE : 0);                               // [2][OW], by part
  // [groups][L]; swept, only rows of one point have groups, and no neighbours
  float4* s_lown = s_ball + 2 * OW;
  float4* s_lball = SW && T == 1 ? s_X : s_lown;
  float4* s_res = s_lown + LPE * (SW ? 1 : lpl_groups(LPE, H));                                           // [2 with GRAD][kWave + 2]
  unsigned short* s_tq = reinterpret_cast<unsigned short*>(s_res + (GRAD ? 2 : 1) * (kWave + 2));   // [kLplTrace] (SW)
  float* s_ext = reinterpret_cast<float*>(s_tq + (SW ? kLplTrace : 0));    // [OW] (SW)
  int* s_nb = reinterpret_cast<int*>(s_ext + (SW ? (OW + 3) / 4 * 4 : 0));  // [EPW] (SW)
  unsigned short* s_pq = reinterpret_cast<unsigned short*>(s_nb + (SW ? 8 : 0));         // [kLplPairs]
  unsigned short* s_q = s_pq + kLplPairs;                                  // [3 kWave]

  // ---- one round of loads: this lane's link tables, and the staging ----
  const int lj = l < L ? l : 0;
  const v4i info = *(const v4i*)(a.ln.info + l);   // chain start, chain end, spheres, end effector
  const float4 F0 = reinterpret_cast<const float4*>(a.rb.fixed_tf + lj * 12)[0];
  const float4 F1 = reinterpret_cast<const float4*>(a.rb.fixed_tf + lj * 12)[1];
  const float4 F2 = reinterpret_cast<const float4*>(a.rb.fixed_tf + lj * 12)[2];
  const float4* bls = a.ln.sphere + LPE * slots + 3 * l;
  const float4 bl = bls[0], bl0 = bls[1], bl1 = bls[2];
  const int r_lo = max(row0, row0 + first - 4);
  const int r_hi = min(row0 + nrows - 1, row0 + first + RB - 1 + 4);
  const int n_st = (r_hi - r_lo + 1) * D;
  const float* dsrc = pm ? a.var : a.d;
  for (int i = tid; i < n_st; i += kBlock) {
    const float xv = a.x[(size_t)r_lo * D + i];
    const float dv = CAND ? dsrc[(size_t)r_lo * D + i] : 0.0f;
    s_x[i] = xv;
    if (CAND) s_d[i] = dv;
  }
  if (tid < 3 * D) s_lim[tid] = tid < D ? a.rb.q_lo[tid] : tid < 2 * D ? a.rb.q_hi[tid - D] : a.q_start[(size_t)p * D + tid - 2 * D];
  else if (tid >= kWave && tid < kWave + n_ee * 7) s_goal[tid - kWave] = a.goal[(size_t)p * n_ee * 7 + tid - kWave];
  else if (tid >= 2 * kWave && tid < 2 * kWave + n_ee * 12) s_etf[tid - 2 * kWave] = a.rb.ee_tf[tid - 2 * kWave];
  for (int i = tid; i < LPE * slots; i += kBlock) s_slot[i] = a.ln.sphere[i];
  auto stage_tile = [&](int tl) {
    const int nb = min(kLplTile, w1 - tl);
    const float4* src = reinterpret_cast<const float4*>(a.box + tl);
    for (int i = tid; i < 4 * nb; i += kBlock) s_box[(i & 3) * kLplStride + (i >> 2)] = src[i];
  };
  if (w0 < w1) stage_tile(w0);
  if (pm) {
    // the draws of every particle of the workgroup over its rows: from memory
    // or made here, one Philox block per four elements of [rows][D]
    const int rs = RB + 8, k0 = blockIdx.y * KB;
    if (a.d) {
      for (int i = tid; i < KB * n_st; i += kBlock) {
        const int kk = i / n_st, e = i - kk * n_st;
        s_eps[kk * rs * D + e] = a.d[(size_t)(k0 + kk) * a.d_stride + (size_t)r_lo * D + e];
      }
    } else {
      const long long e_lo = (long long)r_lo * D, e_hi = e_lo + n_st;
      const long long q_lo = e_lo >> 2;
      const int nq = (int)(((e_hi + 3) >> 2) - q_lo);
      for (int i = tid; i < nq * KB; i += kBlock) {
        const int kk = i / nq;
        const long long q = q_lo + (i - kk * nq);
        float w4[4];
        philox_draws4(a.pm_seed, k0 + kk, a.pm_it, (uint64_t)q, w4);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const long long e = 4 * q + u;
          if (e >= e_lo && e < e_hi) s_eps[kk * rs * D + (int)(e - e_lo)] = w4[u];
        }
      }
    }
  }
  __syncthreads();

  const float alpha = CAND ? a.alpha[k < kMaxK ? k : 0] : 0.0f;
  const int eps0 = pm ? (k - (int)blockIdx.y * KB) * (RB + 8) * D : 0;
  // candidate value of joint j at row r: clip(x + alpha d) for a line-search
  // candidate, clip(x + sqrt(var) eps_k) for a particle
  auto qval = [&](int r, int j) -> float {
    const int i = (r - r_lo) * D + j;
    float v = s_x[i];
    if (CAND) {
      if (pm) v = fmaf(sqrtf(s_d[i]), s_eps[eps0 + i], v);
      else v = fmaf(alpha, s_d[i], v);
      v = fminf(fmaxf(v, s_lim[j]), s_lim[D + j]);
    }
    return v;
  };

  // ---- kinematics: the local transform F_l Rz(q_l) (Tab.6) and the prefix
  //      product along the chain, for this waypoint (and its neighbours) ----
  const bool on = l < L;
  const int pos = l - info.x;
  const float ql = qval(row, lj);
  auto pose_at = [&](float q, float* To) {
    if (a.ln.serial) link_pose_serial(F0, F1, F2, on, pos, a.wl.max_depth - 1, q, To);
    else link_pose<LPE>(F0, F1, F2, on, pos, q, To);
  };
  float Tm[12];
  pose_at(ql, Tm);
  if (sub == 0) {
#pragma unroll
    for (int r = 0; r < 3; ++r)
      s_T[r * OW + owner] = make_float4(Tm[4 * r], Tm[4 * r + 1], Tm[4 * r + 2], Tm[4 * r + 3]);
  }
  float ext = 0.0f;
  if constexpr (SW) {
    if (T > 1) {
      // link poses at the neighbouring waypoints (the start before waypoint 1;
      // none after the last: its own pose, a segment of length zero): other
      // evaluations', or the three that lanes 0, LPE and 2 LPE on form here
      const int w_lo = first + wave * EPW % RB, g = lane / LPE;
      const int r_a = max(min(w_lo, nrows - 1) - 1, 0), r_b = min(w_lo + EPW, nrows - 1);
      const float qx = g == 2 ? s_lim[2 * D + lj] : qval(row0 + (g == 0 ? max(r_a, r_lo - row0) : r_b), lj);
      float Tx[12];
      pose_at(qx, Tx);
      if (g < 3) {
#pragma unroll
        for (int r = 0; r < 3; ++r)
          s_X[(3 * r + g) * LPE + l] = make_float4(Tx[4 * r], Tx[4 * r + 1], Tx[4 * r + 2], Tx[4 * r + 3]);
      }
      const int prev = t == 0 ? EPW + 2 : ew == 0 ? EPW : ew - 1;
      const int next = t + 1 == T ? ew : ew == EPW - 1 ? EPW + 1 : ew + 1;
      if (l == 0 && sub == 0) s_nb[ew] = prev | next << 8;
      wave_lds_fence();
      // the cull's reach: half the longest segment over the link's spheres
      // (slightly widened so rounding never culls a sample the trace takes)
      float4 dp[3], dn[3];
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        auto diff = [&](int sl) {
          const float4 v = sl < EPW ? s_T[r * OW + sl * LPE + l] : s_X[(3 * r + sl - EPW) * LPE + l];
          return make_float4(v.x - Tm[4 * r], v.y - Tm[4 * r + 1], v.z - Tm[4 * r + 2], v.w - Tm[4 * r + 3]);
        };
        dp[r] = diff(prev);
        dn[r] = diff(next);
      }
      float l2 = 0.0f;
      for (int s = 0; s < slots; ++s) {
        const float4 ls = s_slot[l * slots + s];
        if (ls.w <= -1e29f) continue;
        auto seg2 = [&](const float4* N) {
          const float ux = N[0].x * ls.x + N[0].y * ls.y + N[0].z * ls.z + N[0].w;
          const float uy = N[1].x * ls.x + N[1].y * ls.y + N[1].z * ls.z + N[1].w;
          const float uz = N[2].x * ls.x + N[2].y * ls.y + N[2].z * ls.z + N[2].w;
          return ux * ux + uy * uy + uz * uz;
        };
        l2 = fmaxf(l2, fmaxf(seg2(dp), seg2(dn)));
      }
      ext = 0.5f * sqrtf(l2) * 1.001f + 1e-6f;
    }
    if (sub == 0) s_ext[owner] = ext;
  }
  // the ball around the link's spheres, widened slightly so rounding never
  // drops a cuboid that matters (a lane without spheres never passes)
  const float eta = a.pr.eta, inv_eta = 1.0f / fmaxf(eta, 1e-30f), wc = a.pr.w_coll;
  const float cbx = Tm[0] * bl.x + Tm[1] * bl.y + Tm[2] * bl.z + Tm[3];
  const float cby = Tm[4] * bl.x + Tm[5] * bl.y + Tm[6] * bl.z + Tm[7];
  const float cbz = Tm[8] * bl.x + Tm[9] * bl.y + Tm[10] * bl.z + Tm[11];
  const float rball = (bl.w + eta) * 1.0001f + 1e-6f + ext;
  if (H == 1 || sub < 2) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      if (H > 1 && h != sub) continue;             // (two copies: a part each)
      const float4 q = h ? bl1 : bl0;
      s_ball[h * OW + owner] = make_float4(Tm[0] * q.x + Tm[1] * q.y + Tm[2] * q.z + Tm[3],
                                           Tm[4] * q.x + Tm[5] * q.y + Tm[6] * q.z + Tm[7],
                                           Tm[8] * q.x + Tm[9] * q.y + Tm[10] * q.z + Tm[11],
                                           (q.w + eta) * 1.0001f + 1e-6f + ext);
    }
  }
  // the wave's evaluations in groups whose links lie near one another: the
  // candidates of one row, and with trajectories neighbouring rows too (rows
  // of one point each have nothing in common: over two rows of 4 candidates 78
  // of 280 (link, cuboid) pairs passed the test below, by rows 11 of 560)
  const int GE = T == 1 ? max(min(KB, EPW), EPW / lpl_groups(LPE, H)) : EPW, NG = EPW / GE;
  if (EPW > 1) {
    // the link's ball over a group: centre of the bounding box of the centres,
    // half its diagonal more (widened as above)
    float mn[7] = {cbx, cby, cbz, -cbx, -cby, -cbz, -rball};
    evals_min<LPE * H, 7>(mn, GE);
    const float hx = -mn[3] - mn[0], hy = -mn[4] - mn[1], hz = -mn[5] - mn[2];
    if (l < L && sub == 0 && ew % GE == 0)
      s_lball[ew / GE * L + l] =
          make_float4(0.5f * (mn[0] - mn[3]), 0.5f * (mn[1] - mn[4]), 0.5f * (mn[2] - mn[5]),
                      0.5f * sqrtf(hx * hx + hy * hy + hz * hz) * 1.0001f + 1e-6f - mn[6]);
  } else if (lane < L) {
    s_lball[lane] = make_float4(cbx, cby, cbz, rball);
  }
  wave_lds_fence();

  // ---- the near pairs ----
  const int used = a.ln.used;                      // most spheres of a part
  // this lane's sums as an owner (copy sub of an evaluation adds the rows of
  // its share of the lanes): cost, clearance, force and moment about the
  // world origin
  float acc[8] = {0.0f, eta, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  // the lanes' v (owner ow, where act) added to their owners' sums
  auto deliver = [&](bool act, int ow, const float* v) {
    s_res[lane] = make_float4(v[0], v[1], v[2], v[3]);
    if (GRAD) s_res[kWave + 2 + lane] = make_float4(v[4], v[5], v[6], v[7]);
    // the rows of this owner: those whose owner agrees in all six bits
    const uint64_t va = __ballot(act);
    unsigned mlo = (unsigned)va, mhi = (unsigned)(va >> 32);
#pragma unroll
    for (int bit = 0; bit < 6; ++bit) {
      if ((1 << bit) >= OW) break;
      const uint64_t ob = __ballot((ow >> bit) & 1);
      const unsigned mine = (owner >> bit) & 1 ? ~0u : 0u;
      mlo &= ~((unsigned)ob ^ mine);
      mhi &= ~((unsigned)(ob >> 32) ^ mine);
    }
    wave_lds_fence();
    auto add = [&](unsigned i) {
      const float4 a4 = s_res[i];
      acc[0] += a4.x;
      acc[1] = fminf(acc[1], a4.y);
      if (GRAD) {
        const float4 b4 = s_res[kWave + 2 + i];
        acc[2] += a4.z; acc[3] += a4.w;
        acc[4] += b4.x; acc[5] += b4.y; acc[6] += b4.z; acc[7] += b4.w;
      }
    };
    // (no row left: row kWave, which holds nothing)
    if constexpr (H == 1) {
      while (__ballot((mlo | mhi) != 0)) {
        const unsigned i0 = min((unsigned)(__ffs(mlo) - 1), (unsigned)kWave);
        const unsigned i1 = min((unsigned)(__ffs(mhi) - 1), 32u) + 32;
        mlo &= mlo - 1;
        mhi &= mhi - 1;
        add(i0);
        add(i1);
      }
    } else {
      constexpr int SH = kWave / H;                // rows of a copy's share
      unsigned mw = sub * SH < 32 ? mlo >> (sub * SH & 31) : mhi >> (sub * SH & 31);
      if (SH < 32) mw &= (1u << (SH & 31)) - 1;
      while (__ballot(mw != 0)) {
        const unsigned i = mw ? (unsigned)(__ffs(mw) - 1 + sub * SH) : (unsigned)kWave;
        mw &= mw - 1;
        add(i);
      }
    }
    wave_lds_fence();
  };
  if (lane < 2) {
    s_res[kWave + lane] = make_float4(0.0f, 3.0e38f, 0.0f, 0.0f);
    if (GRAD) s_res[2 * kWave + 2 + lane] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
  int ntq = 0;                                     // traces pending (SW)
  // up to 32 (owner, sphere, cuboid), one per lane and side: the trace toward
  // the previous waypoint in the lower half of the wave, the next in the upper
  auto trace_chunk = [&](int base, int n) {
    if constexpr (SW) {
      const int ii = lane & 31, side = 1 + (lane >> 5);
      const bool act = ii < n;
      const unsigned it = act ? s_tq[base + ii] : 0;
      const int ow = it & 63, ob = (it >> 6) & 63, sl = it >> 12;
      const float4 A0 = s_box[ob], A1 = s_box[kLplStride + ob], A2 = s_box[2 * kLplStride + ob],
                   Hh = s_box[3 * kLplStride + ob];
      const float4 t0 = s_T[ow], t1 = s_T[OW + ow], t2 = s_T[2 * OW + ow];
      const int nb = s_nb[ow / LPE], nsl = side == 1 ? nb & 255 : nb >> 8;
      const float4* nt = nsl < EPW ? s_T + nsl * LPE + ow % LPE : s_X + (nsl - EPW) * LPE + ow % LPE;
      const int nst = nsl < EPW ? OW : 3 * LPE;
      const float4 n0 = nt[0], n1 = nt[nst], n2 = nt[2 * nst];
      const float4 ls = s_slot[(ow % LPE) * slots + sl];
      const float cx = row_point(t0, ls);
      const float cy = row_point(t1, ls);
      const float cz = row_point(t2, ls);
      const float px = fmaf(A0.x, cx, fmaf(A0.y, cy, fmaf(A0.z, cz, A0.w)));
      const float py = fmaf(A1.x, cx, fmaf(A1.y, cy, fmaf(A1.z, cz, A1.w)));
      const float pz = fmaf(A2.x, cx, fmaf(A2.y, cy, fmaf(A2.z, cz, A2.w)));
      // the segment to the neighbouring waypoint's centre
      const float ux = row_point(n0, ls) - cx;
      const float uy = row_point(n1, ls) - cy;
      const float uz = row_point(n2, ls) - cz;
      float cost = 0.0f, b[3] = {0.0f, 0.0f, 0.0f};
      if (act)
        trace_term<GRAD>(ux, uy, uz, A0, A1, A2, a.pr.sweep_steps, px, py, pz, Hh,
                         box_dist(fabsf(px) - Hh.x, fabsf(py) - Hh.y, fabsf(pz) - Hh.z), ls.w, wc, eta, inv_eta, cost,
                         b);
      const bool some = cost != 0.0f;
      if (__ballot(some)) {
        const float fx = A0.x * b[0] + A1.x * b[1] + A2.x * b[2];
        const float fy = A0.y * b[0] + A1.y * b[1] + A2.y * b[2];
        const float fz = A0.z * b[0] + A1.z * b[1] + A2.z * b[2];
        const float v[8] = {cost, 3.0e38f, fx, fy, fz, cy * fz - cz * fy, cz * fx - cx * fz, cx * fy - cy * fx};
        deliver(some, ow, v);
      }
    }
  };
  // n (owner, part, cuboid) items, one per lane, or 2, 4 or 8 lanes per item
  // with a share of the part's spheres each
  auto link_chunk = [&](const unsigned short* q, int n) {
    const int sh = n > 32 ? 0 : n > 16 ? 1 : n > 8 ? 2 : 3, per = kWave >> sh;
    const int ii = lane & (per - 1);
    const bool act = ii < n;
    const unsigned it = act ? q[ii] : 0;
    const int ow = it & 63, s_h = (it >> 6 & 1) * used, ob = it >> 7;
    const float4 A0 = s_box[ob], A1 = s_box[kLplStride + ob], A2 = s_box[2 * kLplStride + ob],
                 Hh = s_box[3 * kLplStride + ob];
    const float4 t0 = s_T[ow], t1 = s_T[OW + ow], t2 = s_T[2 * OW + ow];
    const float4* sl = s_slot + (ow % LPE) * slots + s_h;
    const float ext_o = SW ? s_ext[ow] : 0.0f;
    const float reach = act ? eta + ext_o : -1e30f;
    const int s1 = lane >> (6 - sh);               // this lane's spheres: s1, s1 + (1 << sh), ..
    float cost = 0.0f, mc = 3.0e38f, b[3] = {0.0f, 0.0f, 0.0f}, m[3] = {0.0f, 0.0f, 0.0f};
    // (the face test; an unused slot's radius is -1e30: it never passes)
    auto test = [&](int s, float4& ls, float* p, float& m3) -> bool {
      ls = sl[min(s, used - 1)];
      const float cx = row_point(t0, ls);
      const float cy = row_point(t1, ls);
      const float cz = row_point(t2, ls);
      p[0] = fmaf(A0.x, cx, fmaf(A0.y, cy, fmaf(A0.z, cz, A0.w)));
      p[1] = fmaf(A1.x, cx, fmaf(A1.y, cy, fmaf(A1.z, cz, A1.w)));
      p[2] = fmaf(A2.x, cx, fmaf(A2.y, cy, fmaf(A2.z, cz, A2.w)));
      m3 = fmaxf(fabsf(p[0]) - Hh.x, fmaxf(fabsf(p[1]) - Hh.y, fabsf(p[2]) - Hh.z));
      return s < used && m3 < ls.w + reach;
    };
    for (int s0 = 0; s0 < used; s0 += 2 << sh) {
      const int sa = s0 + s1, sb = sa + (1 << sh);
      float4 la, lb;
      float pa[3], pb[3], ma, mb;
      const bool ha = test(sa, la, pa, ma), hb = test(sb, lb, pb, mb);
      float da = 0.0f, db = 0.0f;
      if (ha)
        pair_term<GRAD>(pa[0], pa[1], pa[2], fabsf(pa[0]) - Hh.x, fabsf(pa[1]) - Hh.y, fabsf(pa[2]) - Hh.z, ma, la.w,
                        wc, eta, inv_eta, cost, mc, b, m, da);
      if (hb)
        pair_term<GRAD>(pb[0], pb[1], pb[2], fabsf(pb[0]) - Hh.x, fabsf(pb[1]) - Hh.y, fabsf(pb[2]) - Hh.z, mb, lb.w,
                        wc, eta, inv_eta, cost, mc, b, m, db);
      if constexpr (SW) {
        // the trace's first step, against half the link's longest segment
        const float ra = la.w + eta, rb = lb.w + eta;
        const bool wa = ha && (da < ra ? ra : da - ra) < ext_o, wb = hb && (db < rb ? rb : db - rb) < ext_o;
        const uint64_t ba = __ballot(wa), bb = __ballot(wb);
        if (wa) s_tq[ntq + lanes_below(ba)] = (unsigned short)(ow | ob << 6 | (s_h + sa) << 12);
        ntq += __popcll(ba);
        if (wb) s_tq[ntq + lanes_below(bb)] = (unsigned short)(ow | ob << 6 | (s_h + sb) << 12);
        ntq += __popcll(bb);
        if (ntq >= kWave / 2) {
          wave_lds_fence();
          while (ntq >= kWave / 2) {
            ntq -= kWave / 2;
            trace_chunk(ntq, kWave / 2);
          }
        }
      }
    }
    // force and moment about the world origin (the box origin is at
    // -A^T (A0.w, A1.w, A2.w)); items no sphere of which comes within r + eta
    // add nothing
    const bool some = mc < eta;
    if (__ballot(some)) {
      const float fx = A0.x * b[0] + A1.x * b[1] + A2.x * b[2];
      const float fy = A0.y * b[0] + A1.y * b[1] + A2.y * b[2];
      const float fz = A0.z * b[0] + A1.z * b[1] + A2.z * b[2];
      const float ox = -(A0.x * A0.w + A1.x * A1.w + A2.x * A2.w);
      const float oy = -(A0.y * A0.w + A1.y * A1.w + A2.y * A2.w);
      const float oz = -(A0.z * A0.w + A1.z * A1.w + A2.z * A2.w);
      const float v[8] = {cost, mc, fx, fy, fz,
                          A0.x * m[0] + A1.x * m[1] + A2.x * m[2] + (oy * fz - oz * fy),
                          A0.y * m[0] + A1.y * m[1] + A2.y * m[2] + (oz * fx - ox * fz),
                          A0.z * m[0] + A1.z * m[1] + A2.z * m[2] + (ox * fy - oy * fx)};
      deliver(some, ow, v);
    }
  };

  // ---- world collision (Eq.(10)/(11), summed over cuboids and spheres) ----
  for (int tl = w0; tl < w1; tl += kLplTile) {
    if (tl > w0) {
      __syncthreads();
      stage_tile(tl);
      __syncthreads();
    }
    const int nb = min(kLplTile, w1 - tl);
    // the cuboid's distance from a ball's centre against its radius
    auto reaches = [&](const float4& c4, const float4& A0, const float4& A1, const float4& A2, const float4& Hh,
                       bool exact) -> bool {
      const float px = fmaf(A0.x, c4.x, fmaf(A0.y, c4.y, fmaf(A0.z, c4.z, A0.w)));
      const float py = fmaf(A1.x, c4.x, fmaf(A1.y, c4.y, fmaf(A1.z, c4.z, A1.w)));
      const float pz = fmaf(A2.x, c4.x, fmaf(A2.y, c4.y, fmaf(A2.z, c4.z, A2.w)));
      const float ax = fabsf(px) - Hh.x, ay = fabsf(py) - Hh.y, az = fabsf(pz) - Hh.z;
      const bool face = fmaxf(ax, fmaxf(ay, az)) < c4.w;
      if (!exact) return face;
      const float qx = fmaxf(ax, 0.0f), qy = fmaxf(ay, 0.0f), qz = fmaxf(az, 0.0f);
      return face && fmaf(qx, qx, fmaf(qy, qy, qz * qz)) <= c4.w * c4.w;
    };
    // 1. (group, link, cuboid) pairs i = (g L + l) nb + o, as many as the queue
    //    holds at a time (the divisions by multiplication: exact for i < 2^13,
    //    nb <= 64 and g L + l < 2^7, L <= 16); the face test alone (the
    //    distance costs a third more here and spares less than that in 2.)
    const int n_lo = NG * L * nb;
    const unsigned magic = ((1u << 20) + nb - 1) / nb, magic_l = ((1u << 11) + L - 1) / L;
    int nq = 0;
    for (int i0 = 0; i0 < n_lo;) {
      int np = 0;
      for (; i0 < n_lo && np <= kLplPairs - kWave; i0 += kWave) {
        const int i = min(i0 + lane, n_lo - 1);
        const int gl = (i * magic) >> 20, ob = i - gl * nb;
        const bool hit = reaches(s_lball[gl], s_box[ob], s_box[kLplStride + ob], s_box[2 * kLplStride + ob],
                                 s_box[3 * kLplStride + ob], false) &&
                         i0 + lane < n_lo;
        const uint64_t bal = __ballot(hit);
        const int g = EPW == 1 ? 0 : (gl * magic_l) >> 11;
        if (hit) s_pq[np + lanes_below(bal)] = (unsigned short)((gl + g * (LPE - L)) | ob << 7);
        np += __popcll(bal);
      }
      wave_lds_fence();
      // 2. (evaluation, link, cuboid), kWave / GE pairs a step, both parts of
      //    the link; then 3.
      const int sh = __builtin_ctz(GE), step = kWave >> sh;
      for (int j0 = 0; j0 < np; j0 += step) {
        const int pj = j0 + (lane >> sh);
        const unsigned it = s_pq[min(pj, np - 1)];
        // (queued as g LPE + l: evaluation g GE + lane % GE)
        const unsigned gl = it & 127, g = gl / LPE;
        const int ow = (g * GE + (lane & (GE - 1))) * LPE + gl % LPE, ob = it >> 7;
        const float4 A0 = s_box[ob], A1 = s_box[kLplStride + ob], A2 = s_box[2 * kLplStride + ob],
                     Hh = s_box[3 * kLplStride + ob];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const bool hit = reaches(s_ball[h * OW + ow], A0, A1, A2, Hh, true) && pj < np;
          const uint64_t bal = __ballot(hit);
          if (hit) s_q[nq + lanes_below(bal)] = (unsigned short)(ow | h << 6 | ob << 7);
          nq += __popcll(bal);
        }
        if (nq >= kWave) {
          wave_lds_fence();
          while (nq >= kWave) {
            nq -= kWave;
            link_chunk(s_q + nq, kWave);
          }
        }
      }
    }
    if (nq > 0) {
      wave_lds_fence();
      link_chunk(s_q, nq);
    }
    if (SW && ntq > 0) {                           // (the next tile replaces the cuboids)
      wave_lds_fence();
      trace_chunk(0, ntq);
      ntq = 0;
    }
  }

  // ---- joint l: limit cost (Eq.(17)) and smoothness (Eq.(16)); every lane
  //      computes (clamped joint), lanes l >= D discard the result ----
  float cost = 0.0f, gsm = 0.0f;
  {
    float jc = 0.0f, js = 0.0f;
    joint_terms(a, pb, row, t, lj, ql, s_lim[lj], s_lim[D + lj], s_lim[2 * D + lj], qval, jc, js);
    cost = l < D ? jc : 0.0f;
    gsm = l < D ? js : 0.0f;
  }
  // wrench of this link about the world origin: F = sum of d cost / d point,
  // M = sum of point x (d cost / d point) (+ pure moments of the pose term)
  float F[3] = {0.0f, 0.0f, 0.0f}, M[3] = {0.0f, 0.0f, 0.0f};
  // ---- pose reaching cost at the last waypoint (Eq.(14)) ----
  if (info.w >= 0 && t == T - 1)
    pose_term_at(a, s_etf + info.w * 12, s_goal + info.w * 7, info.w, Tm, valid && sub == 0 ? row : -1, cost, F[0],
                 F[1], F[2], M[0], M[1], M[2]);
  // the copies' shares of the owner's sums
  if constexpr (H > 1) {
#pragma unroll
    for (int q = 0; q < (GRAD ? 8 : 2); ++q)
      acc[q] = q == 1 ? copies_op<LPE, H>(acc[q], [](float x, float y) { return fminf(x, y); })
                      : copies_op<LPE, H>(acc[q], [](float x, float y) { return x + y; });
  }
  cost += acc[0];
  const float mc = acc[1];

  // ---- adjoint: suffix sum of link wrenches, projection on joint l's axis ----
  float gradj = 0.0f;
  if (GRAD) {
    float W[6];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      W[q] = F[q] + acc[2 + q];
      W[3 + q] = M[q] + acc[5 + q];
    }
    const int left = info.y - 1 - l;               // links after this one on its chain
    suffix_step<1>(W, left >= 1);
    suffix_step<2>(W, left >= 2);
    suffix_step<4>(W, left >= 4);
    if (LPE > 8) suffix_step<8>(W, left >= 8);
    // revolute z (Tab.7): joint axis z and origin o are columns 2 and 3 of the
    // link pose; d/dq = z . (M - o x F)
    const float ux = W[3] - (Tm[7] * W[2] - Tm[11] * W[1]);
    const float uy = W[4] - (Tm[11] * W[0] - Tm[3] * W[2]);
    const float uz = W[5] - (Tm[3] * W[1] - Tm[7] * W[0]);
    gradj = l < D ? Tm[2] * ux + Tm[6] * uy + Tm[10] * uz + gsm : 0.0f;
  }

  const float csum = group_sum<LPE>(cost);
  const float mcmin = group_min<LPE>(mc);
  float gd = 0.0f;
  if (CAND && GRAD && l < D) gd = gradj * s_d[(row - r_lo) * D + l];
  if (CAND && GRAD) gd = group_sum<LPE>(gd);
  if (valid && sub == 0) {
    const size_t e = (size_t)k * a.rows + row;
    if (l == 0) {
      if (a.sum.count) {
        // (read by another workgroup below: written through to where every
        // XCD sees it)
        st_agent(a.cost_e + e, csum);
        st_agent(a.mc_e + e, mcmin);
        if (CAND && GRAD) st_agent(a.gd_e + e, gd);
      } else {
        a.cost_e[e] = csum;
        if (a.mc_e) a.mc_e[e] = mcmin;
        if (CAND && GRAD) a.gd_e[e] = gd;
      }
    }
    if (GRAD && l < D) a.grad_e[e * D + l] = gradj;
  }

  // ---- the seeds' sums: every workgroup adds its rows to its seeds' counts,
  //      and the one that completes a seed sums the rows, a wave per
  //      candidate, in the order of reduce_kernel (same bits) ----
  // What makes a row's three values visible to the workgroup that sums them,
  // wherever it runs:
  //   1. they are stored and loaded by agent-scope atomics (sc1 set: the store
  //      goes through this XCD's L2 to memory, the load is not served from a
  //      line that the reader's L2 or L1 kept), so no cache holds an older or a
  //      newer value of them, and none has to be written back or invalidated;
  //   2. every wave waits here until its stores are acknowledged (vmcnt 0), and
  //      the barrier makes all of the workgroup's waves have done so before its
  //      count is raised by an agent-scope atomic;
  //   3. the count reaches T only after every workgroup's addition, the adding
  //      wave waits for the value that its addition returns, and its workgroup
  //      loads the rows behind the barrier after that.
  // That is the order which a release and an acquire on the count would ask for,
  // without what those do besides: they write back and invalidate the whole
  // L2, gradients and all, once per workgroup (us per call so, and with
  // __ATOMIC_ACQ_REL: 32 x 32, K = 8 15.5 / 21.1; 256 x 32 13.5 / 18.6; 768 x 32
  // 19.6 / 25.8; 4 x 32 12.4 both).
  if (a.sum.count) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // (2)
    __syncthreads();
    int* s_done = reinterpret_cast<int*>(s_mem);
    const int sa = first / T, ns = (min(first + RB, nrows) - 1) / T - sa + 1;
    if (tid < ns) {
      const int seg = sa + tid, n = min(min(first + RB, nrows), (seg + 1) * T) - max(first, seg * T);
      int* cnt = a.sum.count + (size_t)(seed0 + seg) * a.K + blockIdx.y;
      // (whole seeds are taken off again, not the count cleared: it returns to
      // zero whatever launches of one batch overlap)
      const int old = __hip_atomic_fetch_add(cnt, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const bool done = (unsigned)old / T != (unsigned)(old + n) / T;
      if (done) __hip_atomic_fetch_add(cnt, -T, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_done[tid] = done;
    }
    __syncthreads();
    for (int i = wave; i < ns * KB; i += kLplWaves) {
      const int sg = i / KB, kk = blockIdx.y * KB + i % KB;
      if (!__builtin_amdgcn_readfirstlane(s_done[sg])) continue;
      const size_t e = (size_t)kk * a.rows + row0 + (sa + sg) * T + min(lane, T - 1);
      const float cv = ld_agent(a.cost_e + e), mv = ld_agent(a.mc_e + e);
      const float gv = CAND && GRAD && a.sum.gd ? ld_agent(a.gd_e + e) : 0.0f;
      const float cs = wave_sum(lane < T ? cv : 0.0f), ms = wave_min(mv);
      const float gs = CAND && GRAD ? wave_sum(lane < T ? gv : 0.0f) : 0.0f;
      if (lane == 0) {
        const size_t o = (size_t)kk * a.sum.n_seeds + seed0 + sa + sg;
        a.sum.cost[o] = cs;
        if (a.sum.min_clear) a.sum.min_clear[o] = ms;
        if (CAND && GRAD && a.sum.gd) a.sum.gd[o] = gs;
      }
    }
  }
}

template <int LPE, int H, bool SW>
hipError_t launch_eval_sw(const EvalArgs& a, int grid_x, bool cand, bool grad, hipStream_t s) {
  constexpr int epb = kLplWaves * kWave / (LPE * H);
  const bool pm = a.var != nullptr;
  // the workgroup's evaluations are KB candidates (a divisor of K) of RB rows
  const int K = cand ? a.K : 1;
  if (a.ln.kb < 1 || a.ln.kb * a.ln.rb != epb || K % a.ln.kb || (pm && (!cand || grad)) || a.ln.lpe != LPE ||
      a.ln.used > 8 || (SW && a.ln.rb % (epb / kLplWaves)) || a.rb.dof > a.rb.n_links || a.rb.n_links > LPE ||
      grid_x < 1)
    return hipErrorInvalidValue;
  const dim3 grid(grid_x, K / a.ln.kb), block(kBlock);
  const size_t lds = (size_t)lpl_lds(LPE, H, a.ln.rb, a.ln.kb, a.rb.dof, 2 * a.ln.used, SW, pm, grad).total * sizeof(float);
  auto go = [&](auto kern) -> hipError_t {
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    kern<<<grid, block, lds, s>>>(a);
    return hipGetLastError();
  };
  if (cand && grad) return go(eval_kernel<LPE, H, true, true, SW>);
  if (grad) return go(eval_kernel<LPE, H, false, true, SW>);
  if (!cand) return go(eval_kernel<LPE, H, false, false, SW>);
  return go(eval_kernel<LPE, H, true, false, SW>);   // particle costs
}

template <int LPE, int H>
hipError_t launch_eval_shape(const EvalArgs& a, int grid_x, bool cand, bool grad, hipStream_t s) {
  return a.pr.swept ? launch_eval_sw<LPE, H, true>(a, grid_x, cand, grad, s)
                    : launch_eval_sw<LPE, H, false>(a, grid_x, cand, grad, s);
}

}  // namespace
}  // namespace mg
