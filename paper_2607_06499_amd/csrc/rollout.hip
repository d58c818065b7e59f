// rollout.hip -- noise, forward simulation, cost and collision of every
// rollout (Alg. 1 [Rollouts], Eq. (3)-(5), Sec. II-B.1).  Each block also
// leaves a partial record (counts and sums for pruning and the reference
// point of Eq. (9)-(11)); the next kernel reduces those records.
//
// Layout: a rollout's steps are spread over lanes of a wavefront (the unicycle:
// 8, 16 or 32 lanes of 2 or 4 steps each, by horizon and rollout count; the arm:
// one step per lane, 32 or 64 lanes).  A
// lane owns the controls u_j of its steps and the states x_{j+1} they lead to:
// it draws their noise, the linear parts of the dynamics are prefix sums across
// lanes (the heading and position of the unicycle, the joint angles of the
// arm), and it evaluates their stage cost, contacts and (arm) forward
// kinematics.
#include "device.hpp"
#include "launch.hpp"

namespace cemppi {

// ---------------------------------------------------------------------------
// shared prologue: obstacles into LDS, finiteness, closest obstacle o*.  (The
// arm's helpers come first: the prologue uses them.)
struct ObsLds {
  float4 o[kMaxObs];     // (x, y, z, R^2) with R = robot/sphere radius + obstacle radius
  float4 v[kMaxObs];     // obstacle velocity (constant-velocity obstacles; else 0)
  float4 live[kMaxObs];  // the obstacles a rollout can reach, in index order
  float4 vlive[kMaxObs]; // their velocities
  int idx[kMaxObs];      // their obstacle indices
  int n_live;
};

// Arm forward kinematics: origins P0..P6 of the standard DH chain
// (A_i = Rz(q_i + off_i) Tz(d_i) Tx(a_i) Rx(alpha_i)); P6 is p_ee(q).
__device__ __forceinline__ void arm_origins(const Cfg& c, const float* q, float P[7][3],
                                            float* Re = nullptr) {
  float r00 = 1.f, r01 = 0.f, r02 = 0.f, r10 = 0.f, r11 = 1.f, r12 = 0.f, r20 = 0.f, r21 = 0.f,
        r22 = 1.f;
  float tx = 0.f, ty = 0.f, tz = 0.f;
  P[0][0] = P[0][1] = P[0][2] = 0.f;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    float st, ct;
    sincosf(q[i] + c.dh_off[i], &st, &ct);
    const float ca = c.dh_ca[i], sa = c.dh_sa[i], a = c.dh_a[i], d = c.dh_d[i];
    // translation of frame i in frame i-1: (a cos th, a sin th, d)
    const float lx = a * ct, ly = a * st, lz = d;
    tx += r00 * lx + r01 * ly + r02 * lz;
    ty += r10 * lx + r11 * ly + r12 * lz;
    tz += r20 * lx + r21 * ly + r22 * lz;
    // rotation Rz(th) Rx(alpha)
    const float a00 = ct, a01 = -st * ca, a02 = st * sa;
    const float a10 = st, a11 = ct * ca, a12 = -ct * sa;
    const float a21 = sa, a22 = ca;
    const float n00 = r00 * a00 + r01 * a10, n01 = r00 * a01 + r01 * a11 + r02 * a21,
                n02 = r00 * a02 + r01 * a12 + r02 * a22;
    const float n10 = r10 * a00 + r11 * a10, n11 = r10 * a01 + r11 * a11 + r12 * a21,
                n12 = r10 * a02 + r11 * a12 + r12 * a22;
    const float n20 = r20 * a00 + r21 * a10, n21 = r20 * a01 + r21 * a11 + r22 * a21,
                n22 = r20 * a02 + r21 * a12 + r22 * a22;
    r00 = n00; r01 = n01; r02 = n02;
    r10 = n10; r11 = n11; r12 = n12;
    r20 = n20; r21 = n21; r22 = n22;
    P[i + 1][0] = tx;
    P[i + 1][1] = ty;
    P[i + 1][2] = tz;
  }
  if (Re) {
    Re[0] = r00; Re[1] = r01; Re[2] = r02;
    Re[3] = r10; Re[4] = r11; Re[5] = r12;
    Re[6] = r20; Re[7] = r21; Re[8] = r22;
  }
}

// Orientation error of the pose cost (Sec. III-C): the angle of the relative
// rotation R_g^T R_ee, atan2(|v|, tr - 1) with tr its trace and v its
// antisymmetric part (|v| = 2 sin, tr - 1 = 2 cos); well conditioned at every
// angle in [0, pi].
__device__ __forceinline__ float rot_angle(const Cfg& c, const float* Re) {
  float tr = 0.f, vx = 0.f, vy = 0.f, vz = 0.f;
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const float g0 = c.Rg[3 * i], g1 = c.Rg[3 * i + 1], g2 = c.Rg[3 * i + 2];
    const float e0 = Re[3 * i], e1 = Re[3 * i + 1], e2 = Re[3 * i + 2];
    tr += g0 * e0 + g1 * e1 + g2 * e2;
    vx += g2 * e1 - g1 * e2;
    vy += g0 * e2 - g2 * e0;
    vz += g1 * e0 - g0 * e1;
  }
  return atan2f(sqrtf(vx * vx + vy * vy + vz * vz), tr - 1.f);
}

__device__ __forceinline__ void sphere_centre(const Cfg& c, const float P[7][3], int s, float& x,
                                              float& y, float& zz) {
  // the segment of sphere s is a kernel argument, so this switch is a
  // wave-uniform (scalar) branch
  const int sg = c.sph_seg[s];
  float ax, ay, az, bx, by, bz;
  switch (sg) {
#define CEMPPI_SEG(i)                                     \
  case i:                                                 \
    ax = P[i][0]; ay = P[i][1]; az = P[i][2];             \
    bx = P[i + 1][0]; by = P[i + 1][1]; bz = P[i + 1][2]; \
    break;
    CEMPPI_SEG(0)
    CEMPPI_SEG(1)
    CEMPPI_SEG(2)
    CEMPPI_SEG(3)
    CEMPPI_SEG(4)
    default:
      ax = P[5][0]; ay = P[5][1]; az = P[5][2];
      bx = P[6][0]; by = P[6][1]; bz = P[6][2];
      break;
#undef CEMPPI_SEG
  }
  const float t = c.sph_t[s];
  x = ax + t * (bx - ax);
  y = ay + t * (by - ay);
  zz = az + t * (bz - az);
}

__device__ __forceinline__ float limit_penalty(const Cfg& c, const float* q) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 6; ++i) {
    const float e = fabsf(q[i]) - c.qlim[i];
    s += e > 0.f ? e * e : 0.f;
  }
  return c.wlim * s;
}

// Prologue of a block, the work of one wave (all 64 lanes): stages the
// obstacles, checks the inputs and computes o* (smallest surface clearance,
// ties to the lowest index) and p(x_t); what it leaves in LDS is valid after
// the block's next barrier.  CVM: constant-velocity obstacles never (0), always
// (1) or as c.cv says (2).  Arm (DYN 1): *s_c0 receives the state part of the
// stage cost of x_t (with the pose cost, including its contact indicator).
// pub (block 0): also pushes the observation into the history ring and
// publishes the per-replan facts.
template <int DYN, int CVM = 2>
__device__ __forceinline__ void prologue(const Cfg& c, const Bufs& b, const float* __restrict__ x_t,
                                         const float* __restrict__ obs, int n_obs, bool pub, uint32_t step,
                                         ObsLds& L, int& s_bad, int& s_closest, float* s_p0,
                                         float* s_c0 = nullptr) {
  constexpr int P = DYN == 0 ? 2 : 3;
  const int lane = (int)(threadIdx.x & (kWave - 1));
  const bool mine = lane < n_obs;
  float o[4] = {0.f, 0.f, 0.f, 0.f};
  float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
  bool ok = true;
  if (mine) {
#pragma unroll
    for (int i = 0; i <= P; ++i) o[i] = obs[lane * (P + 1) + i];
    // constant-velocity obstacles: Eq. (17) for every obstacle over the ring
    // as it will be after this replan's push (the current observation is the
    // newest entry), telescoped to (o_t - o_{t-H'+1}) / ((H' - 1) dt)
    if (CVM == 2 ? c.cv != 0 : CVM == 1) {
      const Ctrl* ct = b.ctrl;
      const int cnt = (ct->hs_nobs == n_obs ? ct->hs_count : 0) + 1;
      const int Hp = cnt < c.H ? cnt : c.H;
      if (Hp >= 2) {
        const int h1 = (ct->hs_head - (Hp - 2) + 2 * c.H) % c.H;
        const float* old = b.hist + ((size_t)h1 * c.max_obs + lane) * P;
        const float den = (float)(Hp - 1) * c.dt;
        v.x = (o[0] - old[0]) / den;
        v.y = (o[1] - old[1]) / den;
        if (DYN != 0) v.z = (o[2] - old[2]) / den;
      }
    }
#pragma unroll
    for (int i = 0; i <= P; ++i) ok = ok && isfinite(o[i]);
  }
  if (lane < c.n) ok = ok && isfinite(x_t[lane]);
  const int bad = __ballot(!ok) != 0ull ? 1 : 0;
  const float rad = o[P], R = (DYN == 0 ? c.robot_r : c.rs) + rad;
  const float4 row = make_float4(o[0], o[1], DYN == 0 ? 0.f : o[2], R * R);
  if (mine) {
    L.o[lane] = row;
    L.v[lane] = v;
  }
  float cl = INFINITY;
  int idx = kInt32Max;
  float p0[3];
  if (DYN == 0) {
    p0[0] = x_t[0];
    p0[1] = x_t[1];
    p0[2] = 0.f;
    if (mine) {
      cl = sqrtf(dist2_2(p0[0], p0[1], row.x, row.y)) - rad;
      idx = lane;
    }
  } else {
    float q[6], Pm[7][3], Re[9];
    for (int i = 0; i < 6; ++i) q[i] = x_t[i];
    arm_origins(c, q, Pm, Re);
    for (int i = 0; i < 3; ++i) p0[i] = Pm[6][i];
    bool touch = false;
    for (int s = 0; s < c.ns; ++s) {
      float sx, sy, sz;
      sphere_centre(c, Pm, s, sx, sy, sz);
      const float d2 = dist2_3(sx, sy, sz, row.x, row.y, row.z);
      const float w = sqrtf(d2) - rad;
      cl = mine && w < cl ? w : cl;
      touch |= mine && d2 <= row.w;
    }
    if (mine) idx = lane;
    const bool icol0 = __ballot(touch) != 0ull;
    if (lane == 0 && s_c0) {
      const float d2g = sq(p0[0] - c.goal[0]) + sq(p0[1] - c.goal[1]) + sq(p0[2] - c.goal[2]);
      *s_c0 = c.pose ? c.Q[0] * sqrtf(d2g) + c.Q[1] * rot_angle(c, Re) + limit_penalty(c, q) +
                           (icol0 ? c.Q[2] : 0.f)
                     : c.Q[0] * d2g + limit_penalty(c, q);
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) {
    const float oc = __shfl_xor(cl, d, kWave);
    const int oi = __shfl_xor(idx, d, kWave);
    if (oc < cl || (oc == cl && oi < idx)) {
      cl = oc;
      idx = oi;
    }
  }
  const int closest = n_obs > 0 ? idx : -1;
  if (DYN == 0) {
    // Broad phase (unicycle): every state of a rollout lies within
    // reach = max|v| N dt of p(x_t), so an obstacle whose surface is farther
    // than that (with a margin far above the FP32 rounding of the positions)
    // is never in contact; it is left out of the collision loops.  The kept
    // obstacles stay in index order, so the lowest-index rule is unchanged.
    // A moving obstacle covers at most |v| N dt more.
    bool keep = mine;
    if (keep && c.reach < INFINITY) {
      const float d = sqrtf(dist2_2(p0[0], p0[1], row.x, row.y));
      const float ov = sqrtf(v.x * v.x + v.y * v.y) * ((float)c.N * c.dt);
      const float ext = c.reach + R + ov;
      keep = !(d > ext + (1e-3f * ext + 1e-3f));
    }
    const unsigned long long m = __ballot(keep);
    if (keep) {
      const int pos = __popcll(m & ((1ull << lane) - 1ull));
      L.live[pos] = row;
      L.vlive[pos] = v;
      L.idx[pos] = lane;
    }
    if (lane == 0) L.n_live = __popcll(m);
  }
  if (lane == 0) {
    s_bad = bad;
    s_closest = closest;
    for (int i = 0; i < 3; ++i) s_p0[i] = p0[i];
  }
  if (!pub) return;
  // the observation into the ring, and the facts of the prologue
  Ctrl* ct = b.ctrl;
  const int nh = (ct->hist_head + 1) % c.H;
  if (!bad && mine) {
    float* h = b.hist + ((size_t)nh * c.max_obs + lane) * P;
#pragma unroll
    for (int i = 0; i < P; ++i) h[i] = o[i];
  }
  if (lane == 0) {
    if (!bad) {
      const int count = ct->hist_nobs == n_obs ? ct->hist_count : 0;
      ct->hist_head = nh;
      ct->hist_count = count + 1 < c.H ? count + 1 : c.H;
      ct->hist_nobs = n_obs;
    }
    ct->n_obs = n_obs;
    ct->nonfinite = bad;
    ct->closest = closest;
    ct->p0[0] = p0[0];
    ct->p0[1] = p0[1];
    ct->p0[2] = p0[2];
    ct->step_used = step;
  }
}

// Per-rollout contribution to the block partial record.
__device__ __forceinline__ void rollout_contrib(float* rec, bool active, int col, int first,
                                                int closest, float S, const float* src, int P) {
  // every field as one select, written as three 16-byte stores
  const bool hit = active && col;
  const bool inA = hit && first == closest;
  const bool feas = active && !col;
  float4* r4 = reinterpret_cast<float4*>(rec);
  static_assert(kPart == 12 && P_NCOL == 0 && P_NREF == 1 && P_NFEAS == 2 && P_SMIN_ALL == 3 &&
                    P_SMIN_FEAS == 4 && P_SUM_REF == 5 && P_SUM_COL == 8,
                "record layout");
  const float s0 = src[0], s1 = src[1], s2 = P == 3 ? src[2] : 0.f;
  r4[0] = make_float4(hit ? 1.f : 0.f, inA ? 1.f : 0.f, feas ? 1.f : 0.f, active ? S : INFINITY);
  r4[1] = make_float4(feas ? S : INFINITY, inA ? s0 : 0.f, inA ? s1 : 0.f, inA ? s2 : 0.f);
  r4[2] = make_float4(hit ? s0 : 0.f, hit ? s1 : 0.f, hit ? s2 : 0.f, 0.f);
}

// Field f of the partial record of kGroup consecutive rollouts, summed in
// rollout order: the grouping (and so every rounding) is the same however the
// rollouts were spread over waves, blocks or rounds.
__device__ __forceinline__ float group_sum(const float (*recs)[kPart], int f) {
  const bool mn = f == P_SMIN_ALL || f == P_SMIN_FEAS;
  float acc = mn ? INFINITY : 0.f;
#pragma unroll
  for (int r = 0; r < kGroup; ++r) {
    const float v = recs[r][f];
    acc = mn ? fminf(acc, v) : acc + v;
  }
  return acc;
}

// The partial records of the rpb records of a block's rollouts bx*rpb ..
template <int NT>
__device__ __forceinline__ void write_group_partials(const Cfg& c, const Bufs& b, const float (*recs)[kPart],
                                                     int rpb, int bx) {
  __syncthreads();
  const int ng = rpb / kGroup;
  for (int t = threadIdx.x; t < ng * kPart; t += NT) {
    const int g = t / kPart, f = t - g * kPart;
    if (bx * ng + g < c.npart) b.part[((size_t)bx * ng + g) * kPart + f] = group_sum(recs + g * kGroup, f);
  }
}

// Unicycle perturbation (Eq. (3)) of one control step: e = L g, the clamp to
// the bounds (one v_med3_f32: the bounds are ordered) and the applied
// perturbation (clamped control - nominal).
__device__ __forceinline__ void perturb_clamp(const Cfg& c, float2 n, float g0, float g1, float& uv, float& uw,
                                              float& a0, float& a1) {
  const float e0 = c.L[0] * g0;
  const float e1 = c.L[2] * g0 + c.L[3] * g1;
  const float t0 = n.x + e0, t1 = n.y + e1;
  uv = __builtin_amdgcn_fmed3f(t0, c.umin[0], c.umax[0]);
  uw = __builtin_amdgcn_fmed3f(t1, c.umin[1], c.umax[1]);
  a0 = uv == t0 ? e0 : uv - n.x;
  a1 = uw == t1 ? e1 : uw - n.y;
}

// ---------------------------------------------------------------------------
// Unicycle rollouts (Sec. III-A): state (x, y, theta), control (v, omega).
//
// A rollout takes G lanes of a wavefront (8, 16 or 32), a lane C consecutive
// steps: lane g holds the controls u_j for j = g C .. g C + C - 1, and N <= G C.
// The recursion of Eq. (4)/(21) is a serial sum over the lane's steps and a
// scan over the G lanes, and every lane evaluates the noise, cost and contacts
// of its own steps.  C is even, so a lane uses both halves of each Philox block
// it draws.  Steps past N follow every state that counts, so they need no
// masks in the sums.  Bound by VALU issue in large launches and by the latency
// of one wave in small ones (the layout is chosen for each planner).  Measured
// against one step per lane, where a scan took six adds per lane and sum, a
// contact test its LDS read per state and N = 50 left 14 of 64 lanes idle:
// N = 50, K = 8,192 7.2 -> 5.0 us a launch back to back, K = 65,536 27.4 ->
// 17.4 us; the 64 planners of a batch 119 -> 60 us.  The sums of a rollout
// associate by layout, so its states and cost are the same to rounding, not bit
// for bit, in planners whose layouts differ.
template <int G>
constexpr int uni_per_block() {
  return kUniThreads / G;
}

// moves within a row of 16 lanes
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
  return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xf, 0xf, true);
}
// sum over the lower lanes of the rollout's G (g: lane within them)
template <int G>
__device__ __forceinline__ float uni_excl_scan(float v, int g) {
  if constexpr (G == 32) return seg_excl_scan<32>(v, g);
  // (rows of 16: with G = 8 they hold two rollouts, and what comes from the
  // other is left out)
  const float t1 = dpp_f<0x111>(v);  // row_shr:1
  v += G == 16 || g >= 1 ? t1 : 0.f;
  const float t2 = dpp_f<0x112>(v);
  v += G == 16 || g >= 2 ? t2 : 0.f;
  const float t4 = dpp_f<0x114>(v);
  v += G == 16 || g >= 4 ? t4 : 0.f;
  if constexpr (G == 16) v += dpp_f<0x118>(v);
  const float e = dpp_f<0x111>(v);
  return G == 16 || g >= 1 ? e : 0.f;
}
// sum and minimum over the rollout's lanes (every lane gets the same value); the
// sum in 64 bits, so that the cost is rounded once where lanes meet (the error
// of S against FP64 falls by a third, for 0.1 us)
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
  return __hiloint2double(dpp_i<CTRL>(__double2hiint(v)), dpp_i<CTRL>(__double2loint(v)));
}
template <int G>
__device__ __forceinline__ double uni_sum(double v) {
  v += dpp_d<0xB1>(v);   // quad_perm: neighbour
  v += dpp_d<0x4E>(v);   // quad_perm: other pair
  v += dpp_d<0x141>(v);  // row_half_mirror: other quad
  if constexpr (G >= 16) v += dpp_d<0x140>(v);  // row_mirror: other half row
  if constexpr (G >= 32) v += __shfl_xor(v, 16, kWave);
  return v;
}
template <int G>
__device__ __forceinline__ int uni_min(int v) {
  v = min(v, dpp_i<0xB1>(v));
  v = min(v, dpp_i<0x4E>(v));
  v = min(v, dpp_i<0x141>(v));
  if constexpr (G >= 16) v = min(v, dpp_i<0x140>(v));
  if constexpr (G >= 32) v = min(v, __shfl_xor(v, 16, kWave));
  return v;
}

struct UniLds {
  ObsLds o;
  int bad, closest;
  float p0[3];
  __align__(16) float rec[kUniThreads / 8][kPart];  // one per rollout
};

// The bx-th block of rollouts.  The prologue (obstacles, finiteness, o*) is the
// work of one wave: of one more than the rollouts take (EXTRA), beside their
// noise, dynamics and cost, or of the first one before its own.  Nothing is
// stored before the barrier that ends it.  CVM as for the prologue.
template <int G, int C, int CVM, bool EXTRA>
__device__ __forceinline__ void rollout_unicycle_body(const Cfg& c, const Bufs& b, int bx, const float* __restrict__ x_t,
                                                      const float* __restrict__ obs, int n_obs, UniLds& sh) {
  constexpr int RPB = uni_per_block<G>(), RPW = kWave / G;
  static_assert(C % 2 == 0 && RPB % kGroup == 0 && RPB <= kUniThreads / 8, "layout");
  const uint32_t step = b.ctrl->step_lo;
  const int N = c.N;
  const float dt = c.dt;
  const float x0 = x_t[0], y0 = x_t[1], th0 = x_t[2];
  const bool cv = CVM == 2 ? c.cv != 0 : CVM == 1;
  const int tid = item_thread(), lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  if (wave == (EXTRA ? kUniThreads / kWave : 0)) {
    prologue<0, CVM>(c, b, x_t, obs, n_obs, bx == 0, step, sh.o, sh.bad, sh.closest, sh.p0);
    if constexpr (EXTRA) {
      __syncthreads();  // the prologue
      __syncthreads();  // the records
      return;
    }
  }
  const int g = lane & (G - 1), j0 = g * C;
  const int kloc = wave * RPW + lane / G;
  const int k = bx * RPB + kloc;
  const int nv = N - j0;  // the lane's steps below N (if positive)
  // noise, perturbation and clamp (Eq. (3)); applied perturbation kept
  float a0[C], a1[C], px[C], py[C];
  float S;
  {
    float uv[C], uw[C];
#pragma unroll
    for (int q = 0; q < C; q += 2) {
      uint32_t w[4];
      philox((uint32_t)((j0 + q) >> 1), (uint32_t)k, step, c.stream_id, c.seed_lo, c.seed_hi, w);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const float2 u = reinterpret_cast<const float2*>(b.U)[min(j0 + q + h, N - 1)];
        float ga, gb;
        box_muller(w[2 * h], w[2 * h + 1], ga, gb);
        perturb_clamp(c, u, ga, gb, uv[q + h], uw[q + h], a0[q + h], a1[q + h]);
      }
    }
    // forward simulation, Eq. (4)/(21): th[q] is the heading of x_{j0+q},
    // px[q], py[q] the position of x_{j0+q+1}
    float th[C], s = 0.f;
#pragma unroll
    for (int q = 0; q < C; ++q) {
      th[q] = s;
      s = __builtin_fmaf(uw[q], dt, s);
    }
    const float thb = uni_excl_scan<G>(s, g);
    const float the = th0 + (thb + s);  // heading after the lane's steps
    float sx = 0.f, sy = 0.f;
#pragma unroll
    for (int q = 0; q < C; ++q) {
      th[q] = th0 + (thb + th[q]);
      float sn, cs;
      __sincosf(th[q], &sn, &cs);
      // (v dt first would round a clamped speed the same way at every step)
      sx = __builtin_fmaf(uv[q] * cs, dt, sx);
      sy = __builtin_fmaf(uv[q] * sn, dt, sy);
      px[q] = sx;
      py[q] = sy;
    }
    const float bxs = uni_excl_scan<G>(sx, g), bys = uni_excl_scan<G>(sy, g);
#pragma unroll
    for (int q = 0; q < C; ++q) {
      px[q] = x0 + (bxs + px[q]);
      py[q] = y0 + (bys + py[q]);
    }
    // cost, Eq. (5): the stage terms of (x_j, u_j) of the lane's steps, and
    // the terminal term on the lane whose last step is N - 1
    float qx = 0.f, qy = 0.f, qt = 0.f, qv = 0.f, qw = 0.f;
#pragma unroll
    for (int q = 0; q < C; ++q) {
      if (q < nv) {
        const float ex = (q == 0 ? x0 + bxs : px[q > 0 ? q - 1 : 0]) - c.goal[0];
        const float ey = (q == 0 ? y0 + bys : py[q > 0 ? q - 1 : 0]) - c.goal[1];
        const float et = th[q] - c.goal[2];
        qx = __builtin_fmaf(ex, ex, qx);
        qy = __builtin_fmaf(ey, ey, qy);
        qt = __builtin_fmaf(et, et, qt);
        qv = __builtin_fmaf(uv[q], uv[q], qv);
        qw = __builtin_fmaf(uw[q], uw[q], qw);
      }
    }
    double l = (double)c.Q[0] * qx + (double)c.Q[1] * qy + (double)c.Q[2] * qt + (double)c.R[0] * qv + (double)c.R[1] * qw;
    if (nv >= 1 && nv <= C) {
      float ex = px[0], ey = py[0], et = C > 1 ? th[1] : the;
#pragma unroll
      for (int q = 1; q < C; ++q) {
        const bool at = nv == q + 1;
        ex = at ? px[q] : ex;
        ey = at ? py[q] : ey;
        et = at ? (q + 1 < C ? th[q + 1 < C ? q + 1 : q] : the) : et;
      }
      l += c.Qf[0] * sq(ex - c.goal[0]) + c.Qf[1] * sq(ey - c.goal[1]) + c.Qf[2] * sq(et - c.goal[2]);
    }
    S = (float)uni_sum<G>(l);
  }
  __syncthreads();
  const int bad = sh.bad, closest = sh.closest;
  const bool act = k < c.K && !bad;
  if (act) {
    // (rows start at 16-byte boundaries when N is even)
    float2* ep = reinterpret_cast<float2*>(b.eps) + (size_t)k * N + j0;
    if ((N & 1) == 0) {
#pragma unroll
      for (int q = 0; q < C; q += 2)
        if (q < nv) reinterpret_cast<float4*>(ep)[q / 2] = make_float4(a0[q], a1[q], a0[q + 1], a1[q + 1]);
    } else {
#pragma unroll
      for (int q = 0; q < C; ++q)
        if (q < nv) ep[q] = make_float2(a0[q], a1[q]);
    }
  }
  // contacts of the lane's states with the obstacles (constant-velocity
  // obstacles: obstacle i at o_i + j dt v_i for state j)
  const int n_live = sh.o.n_live;
  bool touch[C];
#pragma unroll
  for (int q = 0; q < C; ++q) touch[q] = false;
  for (int i = 0; i < n_live; ++i) {
    const float4 o = sh.o.live[i];
    if (cv) {
      const float4 v = sh.o.vlive[i];
#pragma unroll
      for (int q = 0; q < C; ++q) {
        const float tj = (float)(j0 + q + 1) * dt;
        touch[q] |= dist2_2(px[q], py[q], __builtin_fmaf(tj, v.x, o.x), __builtin_fmaf(tj, v.y, o.y)) <= o.w;
      }
    } else {
#pragma unroll
      for (int q = 0; q < C; ++q) touch[q] |= dist2_2(px[q], py[q], o.x, o.y) <= o.w;
    }
  }
  // the first colliding state of the rollout, and (on its lane) the lowest
  // obstacle it touches
  int qf = C;
#pragma unroll
  for (int q = C - 1; q >= 0; --q) qf = touch[q] ? q : qf;
  const bool hit = act && qf < C && qf < nv;
  int col = 0, first = -1;
  float pfx = 0.f, pfy = 0.f;
  if (__ballot(hit) != 0ull) {
    const int jf = uni_min<G>(hit ? j0 + qf : kInt32Max);
    col = jf != kInt32Max ? 1 : 0;
    float hx = px[0], hy = py[0];
#pragma unroll
    for (int q = 1; q < C; ++q) {
      hx = qf == q ? px[q] : hx;
      hy = qf == q ? py[q] : hy;
    }
    int f = -1;
    if (hit && j0 + qf == jf) {
      const float tj = (float)(jf + 1) * dt;
      for (int i = n_live - 1; i >= 0; --i) {
        const float4 o = sh.o.live[i];
        float ox = o.x, oy = o.y;
        if (cv) {
          const float4 v = sh.o.vlive[i];
          ox = __builtin_fmaf(tj, v.x, o.x);
          oy = __builtin_fmaf(tj, v.y, o.y);
        }
        f = dist2_2(hx, hy, ox, oy) <= o.w ? sh.o.idx[i] : f;
      }
    }
    const int src = (lane & ~(G - 1)) + (col ? jf / C : 0);
    f = __shfl(f, src, kWave);
    hx = __shfl(hx, src, kWave);
    hy = __shfl(hy, src, kWave);
    if (col) {
      first = f;
      pfx = hx;
      pfy = hy;
    }
  }
  // p(x_N): lane (N - 1) / C, step (N - 1) mod C
  float ptx = px[0], pty = py[0];
  const int qn = (N - 1) % C;
#pragma unroll
  for (int q = 1; q < C; ++q) {
    ptx = qn == q ? px[q] : ptx;
    pty = qn == q ? py[q] : pty;
  }
  const int srcn = (lane & ~(G - 1)) + (N - 1) / C;
  ptx = __shfl(ptx, srcn, kWave);
  pty = __shfl(pty, srcn, kWave);
  if (g == 0) {
    if (act) {
      b.S[k] = S;
      b.col[k] = col;
      b.first[k] = first;
      reinterpret_cast<float2*>(b.pT)[k] = make_float2(ptx, pty);
      reinterpret_cast<float2*>(b.pF)[k] = make_float2(pfx, pfy);
      // unit terminal displacement, Eq. (15)
      const float ex = ptx - x0, ey = pty - y0;
      const float den = __builtin_amdgcn_sqrtf(__builtin_fmaf(ey, ey, ex * ex)) + c.norm_eps;
      const float inv = __builtin_amdgcn_rcpf(den);  // v_sqrt_f32 and one v_rcp_f32
      reinterpret_cast<float2*>(b.g)[k] = make_float2(ex * inv, ey * inv);
    }
    const bool fc = c.ref_mode == 1 && col;
    const float src[2] = {fc ? pfx : ptx, fc ? pfy : pty};
    rollout_contrib(sh.rec[kloc], act, col, first, closest, S, src, 2);
  }
  // partial records of the block's groups of kGroup rollouts
  __syncthreads();
  constexpr int NG = RPB / kGroup;
  if (tid < NG * kPart) {
    const int gr = tid / kPart, f = tid - gr * kPart, at = bx * NG + gr;
    if (at < c.npart) b.part[(size_t)at * kPart + f] = group_sum(sh.rec + gr * kGroup, f);
  }
}

template <int G, int C, int CV>
__global__ __launch_bounds__(kUniThreads + kWave) void k_rollout_unicycle(Cfg c, Bufs b, const float* __restrict__ x_t, const float* __restrict__ obs, int n_obs) {
  __shared__ UniLds sh;
  rollout_unicycle_body<G, C, CV, true>(c, b, (int)blockIdx.x, x_t, obs, n_obs, sh);
}

// ---------------------------------------------------------------------------
// Six-joint arm rollouts (Sec. III-C): joint-velocity control, q_{j+1} =
// q_j + u_j dt; end-effector cost (squared distance, or the pose cost of the
// real-robot experiment), joint-limit penalty, link spheres against obstacle
// spheres.  Lane j of a segment holds control u_j and the state x_{j+1} it
// leads to (an inclusive scan), so N <= 32 fits a 32-lane segment and a wave
// runs two rollouts; the state part of the cost of x_t (the same for every
// rollout) comes from the prologue.
//
// Contacts: the centres of eight link spheres are held in registers against
// each obstacle, read from LDS once (all spheres have one contact radius, so
// the least distance decides), and the obstacles are taken from the last to
// the first, so one pass gives the lowest obstacle touched.  Two passes of one
// sphere after another, with an LDS read per pair, and the prologue's kinematics
// ahead of the rollouts' took 16.7 us at K = 1,024 and 39.8 us at 20,011 (16
// obstacles, N = 32); this takes 12.5 and 33.0 us.  Bound by VALU issue in large
// launches (half of it the contacts), by one wave's chain in small ones.
constexpr int kArmSpheres = 8;
// Up to this many blocks (two on each of the 256 CUs) a launch has a wave of its
// own for the prologue; in larger ones three blocks of eight waves on a CU are
// worth more than two of nine.  Measured with / without, us: K = 4,096 12.8 / 13.7,
// 8,192 16.1 / 16.5, 12,000 24.9 / 21.3, 65,536 123 / 87.  (The rollouts are the
// same work in both, so on a part with fewer CUs the line only costs time.)
constexpr int kArmExtraBlocks = 512;
template <int SEG, int R, bool EXTRA>
__device__ __forceinline__ void rollout_arm_body(const Cfg& c, const Bufs& b, int bx,
                                                 const float* __restrict__ x_t,
                                                 const float* __restrict__ obs, int n_obs) {
  constexpr int SPW = kWave / SEG;
  constexpr int RPB = kRollWaves * SPW * R;
  __shared__ ObsLds L;
  __shared__ int s_bad, s_closest;
  __shared__ float s_p0[3], s_c0;
  __shared__ __align__(16) float s_rec[RPB][kPart];
  const uint32_t step = b.ctrl->step_lo;
  const int tid = item_thread(), lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
  // the prologue is the work of one wave: of one more than the rollouts take
  // (EXTRA), beside their noise and kinematics, or of the first one
  if (wave == (EXTRA ? kRollWaves : 0)) {
    prologue<1>(c, b, x_t, obs, n_obs, bx == 0, step, L, s_bad, s_closest, s_p0, &s_c0);
    if constexpr (EXTRA) {
      __syncthreads();  // the prologue
      __syncthreads();  // the records
      return;
    }
  }
  const int j = lane & (SEG - 1), sgi = lane / SEG;
  const int N = c.N;
  const float dt = c.dt;
  float un[6];
#pragma unroll
  for (int i = 0; i < 6; ++i) un[i] = j < N ? b.U[j * 6 + i] : 0.f;
  for (int rr = 0; rr < R; ++rr) {
    const int kloc = (rr * kRollWaves + wave) * SPW + sgi;
    const int k = SEG == 64 ? __builtin_amdgcn_readfirstlane(bx * RPB + kloc) : bx * RPB + kloc;
    const bool on = k < c.K && j < N;  // control u_j, state x_{j+1}
    const bool last = j == N - 1;      // state x_N: terminal weights

    float u[6], a[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) u[i] = a[i] = 0.f;
    if (on) {
      float g[6];
      step_gaussians<6>(c, step, k, j, g);
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        float e = 0.f;
#pragma unroll
        for (int cc = 0; cc < 6; ++cc)
          if (cc <= i) e += c.L[i * 6 + cc] * g[cc];
        const float n0 = un[i];
        const float t = n0 + e;
        u[i] = fminf(fmaxf(t, c.umin[i]), c.umax[i]);
        a[i] = u[i] == t ? e : u[i] - n0;
      }
    }
    float q[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) q[i] = x_t[i] + seg_incl_scan<SEG>(u[i] * dt, j);
    float P[7][3], Re[9];
    arm_origins(c, q, P, Re);
    const float ex = P[6][0], ey = P[6][1], ez = P[6][2];
    float l = 0.f;
    const float d2g = sq(ex - c.goal[0]) + sq(ey - c.goal[1]) + sq(ez - c.goal[2]);
    if (on) {
      float r = 0.f;
#pragma unroll
      for (int i = 0; i < 6; ++i) r += c.R[i] * u[i] * u[i];
      if (c.pose)  // Sec. III-C: w_p |p_ee - p_g| + w_R d_R (+ w_c I_col, below)
        l = (last ? c.Qf[0] : c.Q[0]) * sqrtf(d2g) + (last ? c.Qf[1] : c.Q[1]) * rot_angle(c, Re) +
            limit_penalty(c, q) + r;
      else
        l = (last ? c.Qf[0] : c.Q[0]) * d2g + limit_penalty(c, q) + r;
    }
    if (rr == 0) __syncthreads();  // the prologue
    const int bad = s_bad, closest = s_closest;
    const bool act = k < c.K && !bad, live = on && !bad;
    if (live) {
      float2* ep = reinterpret_cast<float2*>(b.eps + ((size_t)k * N + j) * 6);
      ep[0] = make_float2(a[0], a[1]);
      ep[1] = make_float2(a[2], a[3]);
      ep[2] = make_float2(a[4], a[5]);
    }

    // the lowest obstacle that any link sphere touches (at time (j + 1) dt for
    // moving obstacles)
    const float tj = (float)(j + 1) * dt;
    int hit = kInt32Max;
    for (int s0 = 0; s0 < c.ns; s0 += kArmSpheres) {
      float cx[kArmSpheres], cy[kArmSpheres], cz[kArmSpheres];
#pragma unroll
      for (int s = 0; s < kArmSpheres; ++s) sphere_centre(c, P, min(s0 + s, c.ns - 1), cx[s], cy[s], cz[s]);
      int hs = kInt32Max;
      for (int i = n_obs - 1; i >= 0; --i) {
        float4 o = L.o[i];
        if (c.cv) {
          const float4 v = L.v[i];
          o.x = __builtin_fmaf(tj, v.x, o.x);
          o.y = __builtin_fmaf(tj, v.y, o.y);
          o.z = __builtin_fmaf(tj, v.z, o.z);
        }
        float d2 = dist2_3(cx[0], cy[0], cz[0], o.x, o.y, o.z);
#pragma unroll
        for (int s = 1; s < kArmSpheres; ++s) d2 = fminf(d2, dist2_3(cx[s], cy[s], cz[s], o.x, o.y, o.z));
        hs = d2 <= o.w ? i : hs;
      }
      hit = min(hit, hs);
    }
    if (!live) hit = kInt32Max;
    if (c.pose && hit != kInt32Max) l += last ? c.Qf[2] : c.Q[2];
    const float S = seg_sum<SEG>(l) + s_c0;
    // first colliding state of each segment (lowest lane with a hit)
    const unsigned long long hm = __ballot(hit != kInt32Max);
    const unsigned long long m0 = SEG == 64 ? hm : (hm & 0xffffffffull);
    const unsigned long long m1 = SEG == 64 ? 0ull : (hm >> 32);
    const int f0 = m0 ? __ffsll((long long)m0) - 1 : 0;
    const int f1 = m1 ? __ffsll((long long)m1) - 1 : 0;
    const int col = (sgi == 0 ? m0 : m1) != 0ull;
    const int f = seg_pick_i<SEG>(hit, f0, f1);
    const float pfx = seg_pick<SEG>(ex, f0, f1), pfy = seg_pick<SEG>(ey, f0, f1),
                pfz = seg_pick<SEG>(ez, f0, f1);
    const int ln = N - 1;
    const float ptx = seg_bcast<SEG>(ex, ln), pty = seg_bcast<SEG>(ey, ln), ptz = seg_bcast<SEG>(ez, ln);

    float src[3];
    src[0] = c.ref_mode == 1 ? pfx : ptx;
    src[1] = c.ref_mode == 1 ? pfy : pty;
    src[2] = c.ref_mode == 1 ? pfz : ptz;
    if (j == 0) {
      if (act) {
        b.S[k] = S;
        b.col[k] = col;
        b.first[k] = col ? f : -1;
        b.pT[3 * k] = ptx;
        b.pT[3 * k + 1] = pty;
        b.pT[3 * k + 2] = ptz;
        b.pF[3 * k] = col ? pfx : 0.f;
        b.pF[3 * k + 1] = col ? pfy : 0.f;
        b.pF[3 * k + 2] = col ? pfz : 0.f;
        const float dx = ptx - s_p0[0], dy = pty - s_p0[1], dz = ptz - s_p0[2];
        const float den =
            __builtin_amdgcn_sqrtf(__builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx))) + c.norm_eps;
        const float inv = __builtin_amdgcn_rcpf(den);
        b.g[3 * k] = dx * inv;
        b.g[3 * k + 1] = dy * inv;
        b.g[3 * k + 2] = dz * inv;
      }
      rollout_contrib(s_rec[kloc], act, col, col ? f : -1, closest, S, src, 3);
    }
  }
  write_group_partials<kRollThreads>(c, b, s_rec, RPB, bx);
}

template <int SEG, bool EXTRA>
__global__ __launch_bounds__(kRollThreads + (EXTRA ? kWave : 0)) void k_rollout_arm(Cfg c, Bufs b, const float* __restrict__ x_t, const float* __restrict__ obs, int n_obs) {
  rollout_arm_body<SEG, 1, EXTRA>(c, b, (int)blockIdx.x, x_t, obs, n_obs);
}

// ---------------------------------------------------------------------------
// Batched rollouts: one persistent launch per rollout kind covers the rollout
// blocks of every planner of that kind in the batch; R rounds per wave.
__device__ __forceinline__ void rollout_unicycle_slot(CSlotStatic st, CSlotIO io, int slot, int local, UniLds& sh) {
  const SlotStatic& S = *(const SlotStatic*)(st + slot);
  const SlotIO& I = *(const SlotIO*)(io + slot);
  // the layout is the member's own (a block-uniform branch)
  switch (S.c.seg) {
#define CEMPPI_UNI(seg, G, C) \
  case seg: rollout_unicycle_body<G, C, 2, false>(S.c, S.b, local, I.x_t, I.obs, I.n_obs, sh); break;
    CEMPPI_UNI_LAYOUTS(CEMPPI_UNI)
#undef CEMPPI_UNI
  }
}

// Unicycle items with a block each (the full member set, whose items the host
// knows): the 64 planners of a batch, 15,000 items, take 60 us where persistent
// blocks, whose registers leave too few waves to cover an item's latency, take 88
// (the same members as a subset launch).
__global__ __launch_bounds__(kUniThreads) void kb_rollout_unicycle(CSlotStatic st, CSlotIO io, Tab t) {
  __shared__ UniLds sh;
  int local;
  const int slot = item_of(t, (int)blockIdx.x, &local);
  if (slot >= 0) rollout_unicycle_slot(st, io, slot, local, sh);
}
// and with persistent blocks (member subsets: the graph serves any of them)
__global__ __launch_bounds__(kUniThreads) void kb_rollout_unicycle_loop(CSlotStatic st, CSlotIO io, Tab t) {
  __shared__ int s_pref[kMaxBatch + 1];
  __shared__ UniLds sh;
  for_each_item<kUniThreads>(t, s_pref, [&](int slot, int local) { rollout_unicycle_slot(st, io, slot, local, sh); });
}

template <int R>
__global__ __launch_bounds__(kRollThreads) void kb_rollout_arm(CSlotStatic st, CSlotIO io, Tab t) {
  __shared__ int s_pref[kMaxBatch + 1];
  for_each_item<kRollThreads>(t, s_pref, [&](int slot, int local) {
    const SlotStatic& S = *(const SlotStatic*)(st + slot);
    const SlotIO& I = *(const SlotIO*)(io + slot);
    // the segment width is the member's own (a block-uniform branch)
    if (S.c.seg == 32)
      rollout_arm_body<32, R, false>(S.c, S.b, local, I.x_t, I.obs, I.n_obs);
    else
      rollout_arm_body<64, R, false>(S.c, S.b, local, I.x_t, I.obs, I.n_obs);
  });
}

// ---------------------------------------------------------------------------
// The same reduction on rollout records already in the planner buffers
// (records supplied by the caller): one rollout per thread.
constexpr int kRedThreads = 256;
template <int DYN>
__global__ __launch_bounds__(kRedThreads) void k_reduce_records(Cfg c, Bufs b,
                                                                const float* __restrict__ x_t,
                                                                const float* __restrict__ obs,
                                                                int n_obs) {
  __shared__ ObsLds L;
  __shared__ int s_bad, s_closest;
  __shared__ float s_p0[3];
  __shared__ __align__(16) float s_rec[kRedThreads][kPart];
  const uint32_t step = b.ctrl->step_lo;
  if (threadIdx.x < kWave) prologue<DYN>(c, b, x_t, obs, n_obs, blockIdx.x == 0, step, L, s_bad, s_closest, s_p0);
  __syncthreads();
  const int bad = s_bad, closest = s_closest;
  const int P = DYN == 0 ? 2 : 3;
  {
    const int k = blockIdx.x * kRedThreads + threadIdx.x;
    const bool act = k < c.K && !bad;
    int col = 0, f = -1;
    float S = 0.f, src[3] = {0.f, 0.f, 0.f};
    if (act) {
      col = b.col[k];
      f = b.first[k];
      S = b.S[k];
      const float* sp = c.ref_mode == 1 ? b.pF : b.pT;
      for (int i = 0; i < P; ++i) src[i] = sp[(size_t)k * P + i];
      // Eq. (15) from the supplied terminal point
      float e[3] = {0.f, 0.f, 0.f};
      for (int i = 0; i < P; ++i) e[i] = b.pT[(size_t)k * P + i] - s_p0[i];
      const float den =
          sqrtf(__builtin_fmaf(e[2], e[2], __builtin_fmaf(e[1], e[1], e[0] * e[0]))) + c.norm_eps;
      const float inv = __builtin_amdgcn_rcpf(den);
      for (int i = 0; i < P; ++i) b.g[(size_t)k * P + i] = e[i] * inv;
    }
    rollout_contrib(s_rec[threadIdx.x], act, col, f, closest, S, src, P);
  }
  write_group_partials<kRedThreads>(c, b, s_rec, kRedThreads, (int)blockIdx.x);
}

// Philox words and standard normals of every rollout (stage entry point):
// one thread per (rollout, counter block).
__global__ void k_stage_noise(Cfg c, uint32_t step, uint32_t* __restrict__ words,
                              float* __restrict__ gauss) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= c.K * c.B) return;
  const int k = t / c.B, bl = t % c.B;
  uint32_t w[4];
  philox((uint32_t)bl, (uint32_t)k, step, c.stream_id, c.seed_lo, c.seed_hi, w);
  if (words) {
    uint4* wp = reinterpret_cast<uint4*>(words) + t;
    *wp = make_uint4(w[0], w[1], w[2], w[3]);
  }
  if (gauss) {
    for (int h = 0; h < 2; ++h) {
      const int e = 4 * bl + 2 * h;
      if (e >= c.NM) break;
      float ga, gb;
      box_muller(w[2 * h], w[2 * h + 1], ga, gb);
      gauss[(size_t)k * c.NM + e] = ga;
      if (e + 1 < c.NM) gauss[(size_t)k * c.NM + e + 1] = gb;
    }
  }
}

// ---------------------------------------------------------------------------
// host-side launchers
// kind 0: unicycle (blocks loop over the items, or have one each), 1: arm (r
// rounds per wave and work item: 1, 2, 4 or 8)
void launch_batch_rollout(Launcher& L, int kind, int r, bool loop, const SlotStatic* st, const SlotIO* io, Tab t,
                          int grid) {
  if (grid <= 0) return;
  const CSlotStatic cst = (CSlotStatic)st;
  const CSlotIO cio = (CSlotIO)io;
  if (kind == 0) {
    L(loop ? kb_rollout_unicycle_loop : kb_rollout_unicycle, dim3(grid), dim3(kUniThreads), cst, cio, t);
    return;
  }
  switch (r) {
    case 2: L(kb_rollout_arm<2>, dim3(grid), dim3(kRollThreads), cst, cio, t); break;
    case 4: L(kb_rollout_arm<4>, dim3(grid), dim3(kRollThreads), cst, cio, t); break;
    case 8: L(kb_rollout_arm<8>, dim3(grid), dim3(kRollThreads), cst, cio, t); break;
    default: L(kb_rollout_arm<1>, dim3(grid), dim3(kRollThreads), cst, cio, t); break;
  }
}

void launch_rollout(Launcher& L, const Cfg& c, const Bufs& b, const float* x_t, const float* obs,
                    int n_obs) {
  const dim3 grid(c.nblk_roll);
  if (c.dyn == 0) {
    switch (c.seg) {
#define CEMPPI_UNI(seg, G, C)                                                                                \
  case seg:                                                                                                  \
    L(c.cv ? k_rollout_unicycle<G, C, 1> : k_rollout_unicycle<G, C, 0>, grid, dim3(kUniThreads + kWave), c, b, x_t, \
      obs, n_obs);                                                                                            \
    break;
      CEMPPI_UNI_LAYOUTS(CEMPPI_UNI)
#undef CEMPPI_UNI
    }
  } else {
    if (c.nblk_roll <= kArmExtraBlocks)
      L(c.seg == 32 ? k_rollout_arm<32, true> : k_rollout_arm<64, true>, grid, dim3(kRollThreads + kWave), c, b, x_t, obs,
        n_obs);
    else
      L(c.seg == 32 ? k_rollout_arm<32, false> : k_rollout_arm<64, false>, grid, dim3(kRollThreads), c, b, x_t, obs, n_obs);
  }
}

void launch_reduce_records(Launcher& L, const Cfg& c, const Bufs& b, const float* x_t,
                           const float* obs, int n_obs) {
  const dim3 grid((c.K + kRedThreads - 1) / kRedThreads), block(kRedThreads);
  if (c.dyn == 0)
    L(k_reduce_records<0>, grid, block, c, b, x_t, obs, n_obs);
  else
    L(k_reduce_records<1>, grid, block, c, b, x_t, obs, n_obs);
}

void launch_stage_noise(Launcher& L, const Cfg& c, uint32_t step, uint32_t* words, float* gauss) {
  const int total = c.K * c.B;
  L(k_stage_noise, dim3((total + 255) / 256), dim3(256), c, step, words, gauss);
}

}  // namespace cemppi
