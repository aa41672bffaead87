// Ray tracing with sixteen lanes per ray (a wave traces four rays), for gfx950. Included by
// trace.hip, whose TraceArgs it takes; sphere instances only.
//
// What bounds it: with sixteen waves on a CU (10 KB of LDS and 128 registers each) the vector
// units' issue. By the counters they are active in all of the launch's cycles on a 100k-Gaussian
// 800x800 frame (2,470 vector instructions a ray) and on 524,287 incoherent rays in 1M Gaussians
// (6,690), and in 82% of them in a served burst, with twelve waves. Measured against one lane per
// ray (k_trace<16>): 64x64 rays in 1,000 Gaussians 1,390 to 31 us, 2,777 rays in 50k 2,630 to
// 110 to 140 us by the scene drawn, the 800x800 frame 5.14 to 2.74 ms, the 524,287 rays 21.2 to
// 6.96 ms, a step of 2M incoherent rays and a 1920x1080 frame in 3M Gaussians, its build
// included, 132.7 to 67.5 ms.
//
// A ray traced by one lane is one serial chain of fetches, some 300 for a ray of a 100k
// scene and tens of thousands for one that starts in a dense cluster; whatever the number
// of rays, a launch lasts as long as its longest chain. Here the group takes up to sixteen
// nodes (or leaves) of its ray at a time, so a chain is about sixteen times shorter and
// each step has sixteen fetches in flight for the ray.
//
// Per ray: two stacks of (reference, entry distance), one of internal nodes and one of
// leaves, nearest on top, and a list of hits (key, 1 - alpha), all in LDS. A wave alternates
// whole steps:
//   node step   each group pops up to 16 nodes, one per lane; the children entered go onto
//               the stacks in the order of their lanes, the nearest child on top;
//   leaf step   each group pops up to 16 leaves, one per lane; hits go to the list;
//   finish step a group whose stacks are empty sorts its list and blends it front to back;
//               one whose list is filling sorts it, blends the hits nearer than everything
//               on its stacks and cuts the rest.
// The cut keeps the hits up to the one that ends the ray (transmittance below T_min), or
// the nearest kGroupKeep, and lowers t_max to the last one kept: later nodes, leaves and
// hits beyond it are dropped. If a list so limited is blended and the ray goes on, the next
// round starts at the root beyond the last blended hit, as in restart mode.
// The hits blended and their order are those of k_trace (all keys come from the same
// arithmetic), and so is every output bit.
#pragma once

#include <type_traits>

#include "trace_common.h"

namespace grtx {
namespace {

constexpr int kGroup = 16;       // lanes per ray: a DPP row
constexpr int kGroupsPerWave = 64 / kGroup;
// Hit list entries per ray: 64 and 96 were slower on most cases (64 restarts 11% of the rays of
// a 1M scene for want of room; 96 leaves room for fourteen waves on a CU instead of sixteen).
constexpr int kGroupHits = 80;
constexpr int kGroupKeep = kGroupHits - kGroup;
constexpr int kGroupLook = 56;  // hits at which a list is first sorted and cut
// The node stack's top is a ring of kGroupRing entries in LDS; its bottom, where a step's
// children might not fit in the ring, moves to the group's rows in device memory, kGroupMove
// entries at a time (n_low of them are there), and comes back when the ring is empty. Beyond
// kGroupWide entries a node step pops one node, and from there the stack grows as a
// depth-first traversal's does, by at most three entries per level.
// (A ring that throttled the steps instead, 80 entries with nothing moved out, left 17 of 64
// lanes with a node on the 3M scene: 195 ms for the launch that takes 76.)
constexpr int kGroupRing = 128;
constexpr int kGroupMove = 3 * kGroup;
constexpr int kGroupWide = 640;
constexpr int kGroupSpill = 1024;
static_assert(kGroupWide + 3 * kGroup + kMaxStack <= kGroupSpill, "the rows hold any stack");
constexpr int kGroupLeaves = 64;
// Leaves waiting (over the wave's groups) that call for a leaf step (24 to 48 measured alike),
// and steps a group ready for its finish step waits for a second one (6: 2% slower; for two more:
// 2% faster at 100k, 3% slower on 1M).
constexpr int kGroupLeafLanes = 32;
constexpr int kGroupWait = 24;
// A launch without a queue has one ray per group and waves to spare, so what its steps cost
// counts by the wave's own chain: a finish step is better shared by all four groups, and none
// waits long for it. 2,777 rays in 50k Gaussians: 142 us with the waits above, 113 with these
// (4 steps: 123, 12: 139; at two groups, 4 steps: 125); 64x64 in 1,000: 38.4, 31.0.
constexpr int kOnceReady = 4;
constexpr int kOnceWait = 8;

struct GroupLds {
  uint64_t key[kGroupHits];
  float rest[kGroupHits];                 // 1 - alpha
  // the node stack's ring, then the leaf stack, then what is written for a child not entered
  // (eight entries, so that the groups' start in different banks)
  uint2 item[kGroupRing + kGroupLeaves + 8];
};

// LDS traffic between lanes of one wave needs no barrier (a wave's LDS operations complete
// in order), only the compiler held to the order written.
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

template <int CTRL>
__device__ __forceinline__ int row_op(int old, int v, bool zero) {
  return zero ? __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, true)
              : __builtin_amdgcn_update_dpp(old, v, CTRL, 0xF, 0xF, false);
}
constexpr int kRowShr = 0x110;      // + n: lane l takes lane l - n of its row
constexpr int kRowRor = 0x120;      // + n: rotate the row by n
constexpr int kRowBcast = 0x150;    // + n: every lane takes lane n of its row
template <int N>
__device__ __forceinline__ float row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kRowBcast + N, 0xF, 0xF, true));
}
// Inclusive sum over the lanes of a row.
__device__ __forceinline__ int row_scan(int x) {
  x += row_op<kRowShr + 1>(0, x, true);
  x += row_op<kRowShr + 2>(0, x, true);
  x += row_op<kRowShr + 4>(0, x, true);
  x += row_op<kRowShr + 8>(0, x, true);
  return x;
}
// Inclusive product over the lanes of a row.
__device__ __forceinline__ float row_product(float x) {
  auto shr = [](float v, auto n) __attribute__((always_inline)) {
    return __int_as_float(row_op<kRowShr + decltype(n)::value>(__float_as_int(1.f), __float_as_int(v), false));
  };
  x *= shr(x, std::integral_constant<int, 1>());
  x *= shr(x, std::integral_constant<int, 2>());
  x *= shr(x, std::integral_constant<int, 4>());
  x *= shr(x, std::integral_constant<int, 8>());
  return x;
}

// Minimum over the lanes of a row.
__device__ __forceinline__ float row_min(float x) {
  auto ror = [](float v, auto n) __attribute__((always_inline)) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), kRowRor + decltype(n)::value, 0xF, 0xF, true));
  };
  x = fminf(x, ror(x, std::integral_constant<int, 1>()));
  x = fminf(x, ror(x, std::integral_constant<int, 2>()));
  x = fminf(x, ror(x, std::integral_constant<int, 4>()));
  x = fminf(x, ror(x, std::integral_constant<int, 8>()));
  return x;
}
// Order two keys (compared as doubles: one instruction each, where integers take five).
__device__ __forceinline__ void order2(uint64_t& a, uint64_t& b) {
  const double x = __longlong_as_double((long long)a), y = __longlong_as_double((long long)b);
  double lo, hi;
  asm("v_min_f64 %0, %1, %2" : "=v"(lo) : "v"(x), "v"(y));
  asm("v_max_f64 %0, %1, %2" : "=v"(hi) : "v"(x), "v"(y));
  a = (uint64_t)__double_as_longlong(lo);
  b = (uint64_t)__double_as_longlong(hi);
}

template <int J0, int J1, class F>
__device__ __forceinline__ void unroll(F&& f) {
  if constexpr (J0 < J1) {
    f(std::integral_constant<int, J0>());
    unroll<J0 + 1, J1>(f);
  }
}

// acc[j] = fma(w, v[j], acc[j]) for the hits of lanes 0 to 15 of each group in turn, all lanes of
// a group computing the same sums. (Written out: five instructions per hit and one register,
// where the compiler moves every broadcast into a register of its own first. The leading wait
// covers the two wait states between a register's write and its use across lanes.)
__device__ __forceinline__ void blend_row(float w, float c0, float c1, float c2, float t, float& C0, float& C1, float& C2,
                                          float& D) {
  float wj;
#define GRTX_BLEND(J)                                                          \
  "v_mov_b32_dpp %4, %5 row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"    \
  "v_fmac_f32_dpp %0, %6, %4 row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f32_dpp %1, %7, %4 row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f32_dpp %2, %8, %4 row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t" \
  "v_fmac_f32_dpp %3, %9, %4 row_newbcast:" #J " row_mask:0xf bank_mask:0xf\n\t"
  asm("s_nop 1\n\t" GRTX_BLEND(0) GRTX_BLEND(1) GRTX_BLEND(2) GRTX_BLEND(3) GRTX_BLEND(4) GRTX_BLEND(5) GRTX_BLEND(6)
          GRTX_BLEND(7) GRTX_BLEND(8) GRTX_BLEND(9) GRTX_BLEND(10) GRTX_BLEND(11) GRTX_BLEND(12) GRTX_BLEND(13)
              GRTX_BLEND(14) GRTX_BLEND(15)
      : "+v"(C0), "+v"(C1), "+v"(C2), "+v"(D), "=&v"(wj)
      : "v"(w), "v"(c0), "v"(c1), "v"(c2), "v"(t));
#undef GRTX_BLEND
}
// Transmittance before each lane's hit: T at lane 0, then each lane's predecessor's times that
// one's factor (`rest`, already moved up one lane); fifteen steps pass it from lane to lane.
__device__ __forceinline__ float pass_on(float T, float rest) {
  float before = T;
#define GRTX_PASS "s_nop 1\n\tv_mul_f32_dpp %0, %0, %1 row_shr:1 row_mask:0xf bank_mask:0xf\n\t"
  asm(GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS
          GRTX_PASS GRTX_PASS GRTX_PASS GRTX_PASS
      : "+v"(before)
      : "v"(rest));
#undef GRTX_PASS
  return before;
}

// (reads what was stored as uint2)
typedef uint64_t __attribute__((may_alias)) any_u64;
// The rows in device memory for the deep end of the group's node stack.
__device__ __forceinline__ uint2* group_spill(KernArgs& A, int lane) {
  return A.pool + ((int64_t)blockIdx.x * kGroupsPerWave + lane / kGroup) * kGroupSpill;
}

// A value the compiler cannot see through: what is computed from it stays where it is used
// instead of being held in registers from outside the loop.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Work items a served wave claims at a time (8: 1% slower over a burst of eight requests).
constexpr uint32_t kServeBatch = 16;

// DEG: the SH degree. SERVE: the serving kernel. Work comes from the serving queue instead of
// the ray arrays: each ray is generated from its request's camera, its outputs go to the
// request's buffers, and the wave that completes a request raises its flag in host memory.
// Idle waves wait for new requests and leave once the queue closes.
template <int DEG, bool SERVE>
__global__ void __launch_bounds__(64)
    __attribute__((amdgpu_waves_per_eu(4, 8))) k_trace_group(TraceArgs Args) {
  __shared__ GroupLds s_group[kGroupsPerWave];
  __shared__ ServeDesc s_desc;  // serving: the wave's copy of the request its items belong to
  __shared__ uint32_t s_myj;
  const int lane0 = threadIdx.x & 63;
  GroupLds& G = s_group[lane0 / kGroup];

  // Everything below that belongs to the ray holds the same value in all lanes of its group.
  bool live = false;
  int ray = -1;
  float ox = 0, oy = 0, oz = 0, dx = 0, dy = 0, dz = 0, ix = 0, iy = 0, iz = 0;
  float oix = 0, oiy = 0, oiz = 0;
  float tfar = INFINITY;
  uint64_t tmin = 0;              // key of the last blended hit
  uint64_t tmax = kEmptyKey;      // keys beyond it are not needed this round
  bool limited = false;           // t_max was lowered: hits beyond it may exist
  int n_node = 0, n_leaf = 0, n_hit = 0;
  int n_low = 0;                  // bottom entries of the node stack in device memory
  float low_t = INFINITY;         // ... and no more than their smallest entry distance
  int n_sorted = 0;               // the list's first hits that are in order
  int look = kGroupLook;          // the list is sorted and cut once it holds more hits
  float C0 = 0, C1 = 0, C2 = 0, Dp = 0, T = 1;
  int nblend = 0;
  // the wave's work items [q_next, q_end), taken from the launch's counter in batches
  unsigned q_next = 0, q_end = 0;
  bool exhausted = false;
  int waited = 0;  // steps since a group became ready for its finish step

  bool start = false;  // the ray begins, or goes on, at the root
  bool fresh = true;   // (wave) a group may be without a ray
  // serving: the ray's scene, output address and pixel count; of the wave, the request number of
  // its items, the rays finished of one request but not yet counted there, and since when it idles
  int sid = 0;
  float* out_at = nullptr;
  uint32_t out_n = 0;
  uint32_t sv_seq = 0, fin_slot = 0, fin_n = 0, fin_count = 0;
  uint64_t idle_since = 0;
  if constexpr (SERVE) {
    if (lane0 == 0) {
      s_desc.seq = ~0u;
      s_myj = kServeNoRequest;
    }
  }
  // Adds the finished rays to their request's count; the wave whose rays complete it resets
  // the count and raises the request's flag.
  auto count_finished = [&](KernArgs& A) __attribute__((always_inline)) {
    if (fin_count == 0) return;
    wait_writes();
    if (lane0 == 0 && atomicAdd(&A.sv_dev->slot[fin_slot].done, fin_count) + fin_count == fin_n) {
      atomicExch(&A.sv_dev->slot[fin_slot].done, 0u);
      wait_writes();
      __hip_atomic_store(&A.sv_host->done[fin_slot], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    fin_count = 0;
  };

  while (true) {
    KernArgs& A = kernel_args();
    const int lane = opaque(lane0);
    const int gl = lane & (kGroup - 1);        // lane within the group
    const int row0 = lane & ~(kGroup - 1);     // the group's first lane
    // ------------------------------------------------------------ rays for idle groups
    if (fresh) {
      const uint64_t idle = __ballot(!live && gl == 0);
      bool nowork = false;
      if constexpr (SERVE) {
        if (idle && !exhausted) {
          if (q_next >= q_end) {
            count_finished(A);
            uint32_t take = 0, j = 0, o = 0, closed = 0;
            if (lane == 0)
              take = serve_claim(A.sv_dev, A.sv_host, kServeBatch, A.sv_poll_ticks, &s_myj, &s_desc, &j, &o, &closed);
            take = (uint32_t)__builtin_amdgcn_readfirstlane((int)take);
            sv_seq = (uint32_t)__builtin_amdgcn_readfirstlane((int)j);
            q_next = (uint32_t)__builtin_amdgcn_readfirstlane((int)o);
            q_end = q_next + take;
            nowork = take == 0;
            if (__builtin_amdgcn_readfirstlane((int)closed)) exhausted = true;
            wave_order();
          }
          const uint32_t w = q_next + (uint32_t)__popcll(idle & ((1ull << row0) - 1ull));
          if (!live && w < q_end) {
            const ServeDesc& d = s_desc;
            const uint32_t* order = reinterpret_cast<const uint32_t*>(d.order);
            const uint32_t tile = order ? order[w >> 6] : w >> 6;
            const uint32_t ty = tile / (uint32_t)d.tiles_x, tx = tile - ty * (uint32_t)d.tiles_x;
            const int px = (int)(tx * 8 + (w & 7)), py = (int)(ty * 8 + ((w >> 3) & 7));
            if (px < d.width && py < d.height) {
              live = start = true;
              ray = (int)(((sv_seq % kServeRing) << kServePixelBits) | ((uint32_t)py * (uint32_t)d.width + (uint32_t)px));
              out_at = reinterpret_cast<float*>(d.out);
              out_n = d.n_pixels;
              sid = d.scene;
              ox = d.eye[0]; oy = d.eye[1]; oz = d.eye[2];
              pinhole_dir(d.fwd[0], d.fwd[1], d.fwd[2], d.right[0], d.right[1], d.right[2], d.up[0], d.up[1], d.up[2],
                          px, py, d.width, d.height, &dx, &dy, &dz);
              ix = safe_inv(dx); iy = safe_inv(dy); iz = safe_inv(dz);
              oix = ox * ix; oiy = oy * iy; oiz = oz * iz;
              T = 1.f;
              C0 = C1 = C2 = Dp = 0.f;
              nblend = 0;
              tmin = 0;
            }
          }
          q_next = min(q_end, q_next + (uint32_t)__popcll(idle));
        }
      } else if (idle && !exhausted) {
        if (q_next >= q_end) {
          const unsigned batch = (unsigned)A.group_batch;
          unsigned base = 0;
          if (A.counter) {
            if (lane == 0) base = atomicAdd(A.counter, batch);
            base = (unsigned)__builtin_amdgcn_readfirstlane((int)base);
          } else {
            // one item per group of the launch
            base = q_end == 0 ? blockIdx.x * batch : 0xFFFFFFFFu - batch;
          }
          q_next = base;
          q_end = base + batch;
          if ((int64_t)base >= A.n_work) exhausted = true;
          if ((int64_t)q_end > A.n_work) q_end = (unsigned)A.n_work;
        }
        if (!exhausted) {
          const unsigned w = q_next + (unsigned)__popcll(idle & ((1ull << row0) - 1ull));
          const int r = !live && w < q_end ? ray_of_item(A, w) : -1;
          q_next += (unsigned)__popcll(idle);
          if (r >= 0) {
            live = true;
            ray = r;
            const float* ro = A.ray_o + 3 * (int64_t)r;
            const float* rd = A.ray_d + 3 * (int64_t)r;
            ox = ro[0]; oy = ro[1]; oz = ro[2];
            dx = rd[0]; dy = rd[1]; dz = rd[2];
            ix = safe_inv(dx); iy = safe_inv(dy); iz = safe_inv(dz);
            oix = ox * ix; oiy = oy * iy; oiz = oz * iz;
            tfar = A.ray_tfar ? A.ray_tfar[r] : INFINITY;
            T = A.ray_trans ? A.ray_trans[r] : 1.f;
            C0 = C1 = C2 = Dp = 0.f;
            nblend = 0;
            tmin = 0;
            start = true;
          }
        }
      }
      if (__ballot(live) == 0) {
        if (SERVE) count_finished(A);
        if (exhausted) break;
        if (SERVE && nowork) {
          // nothing to trace: wait for new requests (checking about every 14 us at first,
          // every 110 us after 100 us), and once this wave has found no work for
          // idle_ticks, close the queue: every wave leaves when its rays are done, and the
          // host starts a new launch for later requests
          const uint64_t now = wall_clock();
          if (idle_since == 0) idle_since = now;
          if (now - idle_since > A.sv_idle_ticks) {
            if (lane == 0) atomicOr(reinterpret_cast<ull*>(&A.sv_dev->state), (ull)kServeClosing);
            break;
          }
          const int naps = now - idle_since > 25 * A.sv_poll_ticks ? 32 : 4;
#pragma unroll 1
          for (int z = 0; z < naps; ++z) __builtin_amdgcn_s_sleep(127);
        }
        continue;
      }
      idle_since = 0;
      // (an item outside the image leaves its group without a ray; a served wave whose claim found
      // nothing asks again at its next step, for a request may have come: asking every sixteen steps
      // made a burst of eight requests 1% slower)
      fresh = !exhausted && __ballot(!live) != 0;
      if (__ballot(start)) {
        // ---------------------------------------------------------- start at the root
        // The ray's first two levels in one step: lane 4 i + j tests child i of the root's record
        // and then child j of that child's, so a group has up to sixteen nodes at once instead of
        // after two steps with one and with four (the 800x800 frame of 100k Gaussians: 2.89 to
        // 2.78 ms).
        const float* rb = A.roots + 8 * sid;
        const float tlo = fmaxf(A.t_near, key_t(tmin));
        const Slab sb = slab(rb[0], rb[1], rb[2], rb[3], rb[4], rb[5], ox, oy, oz, ix, iy, iz);
        uint32_t ref = __float_as_uint(rb[6]);
        float te = sb.tn;
        bool in = start && sb.tn <= fminf(sb.tf, tfar) && fminf(sb.tf, tfar) >= tlo;
        bool lone = (ref & kLeafFlag) != 0;  // the item is one of the level above: the first lane's of its kind
        if (lone) in = in && gl == 0;
#pragma unroll
        for (int level = 0; level < 2; ++level) {
          if (in && !lone) {
            const int sh = level == 0 ? 8 * (gl >> 2) : 8 * (gl & 3);
            const float4* np = A.nodes + kNodeF4 * (int64_t)ref;
            const float4 q0 = np[0], q1 = np[1], q2 = np[2], q3 = np[3];
            const float Ax = q0.w * ix, Ay = q1.x * iy, Az = q1.y * iz;
            const float Bx = fmaf(q0.x, ix, -oix), By = fmaf(q0.y, iy, -oiy), Bz = fmaf(q0.z, iz, -oiz);
            auto plane = [&](float w, float a, float b) __attribute__((always_inline)) {
              return fmaf((float)((__float_as_uint(w) >> sh) & 0xFFu), a, b);
            };
            const float lx = plane(q2.z, Ax, Bx), ly = plane(q2.w, Ay, By), lz = plane(q3.x, Az, Bz);
            const float hx = plane(q3.y, Ax, Bx), hy = plane(q3.z, Ay, By), hz = plane(q3.w, Az, Bz);
            const float tn = fmaxf(fmaxf(ix < 0.f ? hx : lx, iy < 0.f ? hy : ly), iz < 0.f ? hz : lz);
            const float tf = fminf(fminf(fminf(ix < 0.f ? lx : hx, iy < 0.f ? ly : hy), iz < 0.f ? lz : hz), tfar);
            const int pick = sh >> 3;
            ref = __float_as_uint(pick == 0 ? q1.z : pick == 1 ? q1.w : pick == 2 ? q2.x : q2.y);
            te = fmaxf(tn, te);
            in = ref != kNoChild && fmaxf(tn, tlo) <= tf && te < INFINITY;
            if (level == 0 && (ref & kLeafFlag)) {
              lone = true;
              in = in && (gl & 3) == 0;
            }
          }
        }
        // their places on the stacks, nearest on top: ranks by entry (the lane in the low bits keeps
        // them apart), then the ranks taken as bits of one mask per group
        const float by = __uint_as_float(((in ? __float_as_uint(te) : 0x7F7FFFFFu) & ~15u) | (unsigned)gl);
        int rank = 0;
        unroll<1, kGroup>([&](auto n) __attribute__((always_inline)) {
          rank += __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(by), kRowRor + decltype(n)::value, 0xF, 0xF, true)) < by;
        });
        const bool is_leaf = (ref & kLeafFlag) != 0;
        int mask = in ? 1 << (rank + (is_leaf ? 16 : 0)) : 0;
        unroll<0, 4>([&](auto n) __attribute__((always_inline)) {
          mask |= __builtin_amdgcn_mov_dpp(mask, kRowRor + (1 << decltype(n)::value), 0xF, 0xF, true);
        });
        if (in) {
          const int above = is_leaf ? (int)((unsigned)mask >> 16) : mask & 0xFFFF;
          G.item[(is_leaf ? kGroupRing : 0) + __popc((unsigned)above >> rank >> 1)] = make_uint2(ref, __float_as_uint(te));
        }
        if (start) {
          n_node = __popc((unsigned)mask & 0xFFFFu);
          n_leaf = __popc((unsigned)mask >> 16);
          n_hit = n_sorted = 0;
          n_low = 0;
          low_t = INFINITY;
          look = kGroupLook;
          tmax = kEmptyKey;
          limited = false;
          start = false;
        }
      }
    }
    wave_order();

    // ------------------------------------------------------------ what each group can do
    // nodes: those whose leaves have room, one where the stack is very long; leaves: while the
    // list has room for a hit of each
    const int in_ring = n_node - n_low;
    const int wide = n_node > kGroupWide ? 1 : kGroup;
    const int p = live ? min(min(wide, n_node), (kGroupLeaves - n_leaf) >> 2) : 0;
    const int q = live && n_hit <= kGroupKeep ? min(kGroup, n_leaf) : 0;
    const bool ready = live && (n_hit > look || (n_node | n_leaf) == 0);
    const int nodes = __popcll(__ballot(gl < p)), leaves = __popcll(__ballot(gl < q));
    const uint64_t readies = __ballot(ready);
    const float tmax_t = key_t(tmax);
    waited = readies ? waited + 1 : 0;
    const bool once = !SERVE && !A.counter;
    if (__popcll(readies) >= (once ? kOnceReady : 2) * kGroup || (nodes | leaves) == 0 ||
        waited > (once ? kOnceWait : kGroupWait)) {
      // ---------------------------------------------------------- finish step
      waited = 0;
      fresh = true;
      constexpr int kOwn = kGroupHits / kGroup;
      // the longest list, the longest sorted start and the most unsorted hits of a ready group
      auto most = [&](int m) __attribute__((always_inline)) {
        m = max(m, __shfl_xor(m, 16));
        return __builtin_amdgcn_readfirstlane(max(m, __shfl_xor(m, 32)));
      };
      const int s0 = n_sorted, m = ready ? n_hit - s0 : 0;
      const int n_max = most(ready ? n_hit : 0), s_max = most(ready ? s0 : 0), m_max = most(m);
      if (s_max == 0 || m_max > 2 * kGroup) {
      // each lane's entries gl, gl + 16, ... and their ranks among the group's; the places
      // past the list's end hold the empty key
      uint64_t key[kOwn];
      int rank[kOwn];
#pragma unroll
      for (int j = 0; j < kOwn; ++j) {
        const int e = gl + j * kGroup;
        key[j] = e < n_hit ? G.key[e] : kEmptyKey;
        rank[j] = 0;
        if (ready && e >= n_hit) G.key[e] = kEmptyKey;
      }
      wave_order();
      if (ready) {
        // Keys compare as doubles just as they do as integers (no sign, the exponent field
        // never all ones), and the hardware compares doubles in one instruction.
        auto count = [&](auto rows) __attribute__((always_inline)) {
          for (int i = 0; i < n_max; i += 2) {
            const double a = __longlong_as_double((long long)G.key[i]), b = __longlong_as_double((long long)G.key[i + 1]);
#pragma unroll
            for (int j = 0; j < decltype(rows)::value; ++j) {
              const double k = __longlong_as_double((long long)key[j]);
              rank[j] += a < k ? 1 : 0;
              rank[j] += b < k ? 1 : 0;
            }
          }
        };
        if (n_max <= kGroup) count(std::integral_constant<int, 1>());
        else if (n_max <= 2 * kGroup) count(std::integral_constant<int, 2>());
        else if (n_max <= 3 * kGroup) count(std::integral_constant<int, 3>());
        else if (n_max <= 4 * kGroup) count(std::integral_constant<int, 4>());
        else count(std::integral_constant<int, kOwn>());
      }
      {
        float rest[kOwn];
#pragma unroll
        for (int j = 0; j < kOwn; ++j) rest[j] = G.rest[gl + j * kGroup];
        wave_order();
#pragma unroll
        for (int j = 0; j < kOwn; ++j)
          if (ready && gl + j * kGroup < n_hit) {
            G.key[rank[j]] = key[j];
            G.rest[rank[j]] = rest[j];
          }
        wave_order();
      }
      } else {
        // A list that was cut starts with its sorted hits: only the new ones are ranked among
        // each other; a search in the sorted part gives their places there, and the sorted hits
        // move up into the places between. (Ranked as a whole, 80 entries take some 800
        // instructions, so some
        // 350. 524,287 rays in 1M Gaussians 7,360 to 6,960 us, the 3M step 71.1 to 67.7 ms, the
        // 800x800 frame of 100k 2,760 to 2,740 us. Lists with more than 32 new hits, as where
        // another group sorts for the first time, are ranked whole: merged too, the registers
        // that takes cost the frame 4%.)
        auto merge = [&](auto rows) __attribute__((always_inline)) {
          constexpr int R = decltype(rows)::value;
          uint64_t nk[R];
          float nr[R];
          int f[R];
          int taken0 = 0, taken1 = 0, taken2 = 0;  // bit p: a new hit's place
#pragma unroll
          for (int r = 0; r < R; ++r) {
            const int e = gl + r * kGroup;
            nk[r] = e < m ? G.key[s0 + e] : kEmptyKey;
            nr[r] = e < m ? G.rest[s0 + e] : 0.f;
            f[r] = 0;
          }
          for (int i = 0; i < m_max; i += 2)
            if (i < m) {
              const uint64_t next = G.key[min(s0 + i + 1, kGroupHits - 1)];
              const double a = __longlong_as_double((long long)G.key[s0 + i]);
              const double b = __longlong_as_double((long long)(i + 1 < m ? next : kEmptyKey));
#pragma unroll
              for (int r = 0; r < R; ++r) {
                const double k = __longlong_as_double((long long)nk[r]);
                f[r] += a < k ? 1 : 0;
                f[r] += b < k ? 1 : 0;
              }
            }
#pragma unroll
          for (int r = 0; r < R; ++r) {
            int at = 0;
            for (int step = 64; step > 0; step >>= 1) {
              if (step > s_max) continue;
              const int q = at + step;
              if (q <= s0 && __longlong_as_double((long long)G.key[min(q, kGroupHits) - 1]) < __longlong_as_double((long long)nk[r]))
                at = q;
            }
            f[r] += at;
            const int bit = gl + r * kGroup < m ? 1 << (f[r] & 31) : 0;
            taken0 |= f[r] < 32 ? bit : 0;
            taken1 |= (f[r] & 32) ? bit : 0;
            taken2 |= f[r] >= 64 ? bit : 0;
          }
          unroll<0, 4>([&](auto n) __attribute__((always_inline)) {
            taken0 |= __builtin_amdgcn_mov_dpp(taken0, kRowRor + (1 << decltype(n)::value), 0xF, 0xF, true);
            taken1 |= __builtin_amdgcn_mov_dpp(taken1, kRowRor + (1 << decltype(n)::value), 0xF, 0xF, true);
            taken2 |= __builtin_amdgcn_mov_dpp(taken2, kRowRor + (1 << decltype(n)::value), 0xF, 0xF, true);
          });
          uint64_t key[kOwn];
          float rest[kOwn];
          bool moved[kOwn];
#pragma unroll
          for (int j = 0; j < kOwn; ++j) {
            const int p = gl + j * kGroup;
            const unsigned w = (unsigned)(j < 2 ? taken0 : j < 4 ? taken1 : taken2);
            const int bit = gl + (j & 1) * kGroup;
            const int below = __popc(w & ((1u << bit) - 1u)) + (j >= 2 ? __popc((unsigned)taken0) : 0) +
                              (j >= 4 ? __popc((unsigned)taken1) : 0);
            moved[j] = ready && p < n_hit && !((w >> bit) & 1u);
            key[j] = G.key[moved[j] ? p - below : 0];
            rest[j] = G.rest[moved[j] ? p - below : 0];
          }
          wave_order();
#pragma unroll
          for (int j = 0; j < kOwn; ++j)
            if (moved[j]) {
              G.key[gl + j * kGroup] = key[j];
              G.rest[gl + j * kGroup] = rest[j];
            }
#pragma unroll
          for (int r = 0; r < R; ++r)
            if (gl + r * kGroup < m) {
              G.key[f[r]] = nk[r];
              G.rest[f[r]] = nr[r];
            }
        };
        if (m_max <= kGroup) merge(std::integral_constant<int, 1>());
        else merge(std::integral_constant<int, 2>());
        wave_order();
      }
      // Hits nearer than everything on the stacks can be blended; where the stacks are empty
      // that is the whole list.
      const bool open = ready && (n_node | n_leaf) != 0;  // (the list is full)
      int n_fin = ready ? n_hit : 0;
      if (__ballot(open)) {
        float front = low_t;
        const int n_open = open ? n_node - n_low : 0;
        for (int i = gl; __ballot(i < n_open) != 0; i += kGroup)
          if (i < n_open) front = fminf(front, __uint_as_float(G.item[(n_low + i) & (kGroupRing - 1)].y));
#pragma unroll
        for (int j = 0; j < kGroupLeaves; j += kGroup)
          if (open && gl + j < n_leaf) front = fminf(front, __uint_as_float(G.item[kGroupRing + gl + j].y));
        front = row_min(front);
        int before = 0;
#pragma unroll
        for (int j = 0; j < kOwn; ++j) {
          const int e = gl + j * kGroup;
          before += __popc((unsigned)(__ballot(open && e < n_hit && key_t(G.key[e]) < front) >> row0) & 0xFFFFu);
        }
        if (open) n_fin = before;
      }
      bool ert = false;
      {
        float Y[16];
        sh_basis_of(dx, dy, dz, DEG, Y);
#pragma unroll 1
        for (int c0 = 0; __ballot(!ert && c0 < n_fin) != 0; c0 += kGroup) {
          const int e = c0 + gl;
          const bool mine = !ert && e < n_fin;
          HitAlpha h{0.f, 1.f, 0.f};
          uint32_t gid = 0;
          float c[3] = {0.f, 0.f, 0.f};
          if (mine) {
            const float4* ip = A.inst + 4 * (int64_t)(uint32_t)G.key[e];
            const float4 r0 = ip[0], r1 = ip[1], r2 = ip[2], r3 = ip[3];
            gid = __float_as_uint(r3.z);
            h = hit_alpha(sphere_terms(r0, r1, r2, ox, oy, oz, dx, dy, dz), r3);
            sh_colour(A.sh, gid, DEG, Y, c);
#pragma unroll
            for (int ch = 0; ch < 3; ++ch) c[ch] = fmaxf(c[ch], 0.f);
          }
          const float before =
              pass_on(T, __int_as_float(row_op<kRowShr + 1>(__float_as_int(1.f), __float_as_int(h.rest), false)));
          const float after = before * h.rest;
          // the ray ends after the first hit that brings it below T_min
          const unsigned end = (unsigned)(__ballot(mine && after < A.T_min) >> row0) & 0xFFFFu;
          const int last = end ? __ffs((int)end) - 1 : kGroup - 1;
          const bool blend = mine && gl <= last;
          const int n_blend = __popc((unsigned)(__ballot(blend) >> row0) & 0xFFFFu);
          const float w = blend ? before * h.alpha : 0.f;
          const float b0 = blend ? c[0] : 0.f, b1 = blend ? c[1] : 0.f, b2 = blend ? c[2] : 0.f;
          blend_row(w, b0, b1, b2, blend ? -h.neg_t : 0.f, C0, C1, C2, Dp);
          const float t_end = __shfl(after, row0 + last);
          if (!ert && c0 < n_fin) {
            T = t_end;
            if (blend && A.hit_ids && nblend + gl < A.hit_cap)
              A.hit_ids[(int64_t)ray * A.hit_cap + nblend + gl] = (int32_t)gid;
            nblend += n_blend;
            ert = end != 0;
          }
        }
      }
      if (n_fin > 0) tmin = G.key[n_fin - 1];
      const bool cut = open && !ert;
      if (__ballot(cut)) {
        // the rest of the list moves to its start ...
        uint64_t mkey[kOwn];
        float mrest[kOwn];
#pragma unroll
        for (int j = 0; j < kOwn; ++j) {
          const int e = gl + j * kGroup + n_fin;
          mkey[j] = G.key[e < kGroupHits ? e : 0];
          mrest[j] = G.rest[e < kGroupHits ? e : 0];
        }
        wave_order();
        const int rest_n = n_hit - n_fin;
        float t = T;
        int keep = rest_n < kGroupKeep ? rest_n : kGroupKeep;
        bool found = false;
#pragma unroll
        for (int j = 0; j < kOwn; ++j) {
          const int e = gl + j * kGroup;
          const bool in = cut && e < rest_n;
          if (in) {
            G.key[e] = mkey[j];
            G.rest[e] = mrest[j];
          }
          // ... up to the hit that brings the transmittance safely below T_min
          const float after = t * row_product(in ? mrest[j] : 1.f);
          const unsigned ends = (unsigned)(__ballot(in && after < 0.999f * A.T_min) >> row0) & 0xFFFFu;
          if (!found && ends) {
            keep = min(keep, j * kGroup + __ffs((int)ends));
            found = true;
          }
          t = row_bcast<kGroup - 1>(after);
        }
        wave_order();
        if (cut) {
          n_hit = n_sorted = keep;
          look = min(kGroupKeep, keep + kGroup);
          if (found || keep < rest_n) {
            tmax = G.key[keep - 1];
            limited = true;
          }
        }
      }
      if (ready && !cut) {
        const bool done = ert || !limited;
        bool cont = false;
        if (!SERVE && done && A.ray_kind && tfar != INFINITY && T >= A.T_min) {
          const int kd = A.ray_kind[ray];
          cont = kd == GRTX_OBJECT_MIRROR || kd == GRTX_OBJECT_GLASS;
        }
        if (cont) {
          // on along the reflected or refracted ray (see k_trace)
          const float* no = A.ray_next_o + 3 * (int64_t)ray;
          const float* nd = A.ray_next_d + 3 * (int64_t)ray;
          ox = no[0]; oy = no[1]; oz = no[2];
          dx = nd[0]; dy = nd[1]; dz = nd[2];
          ix = safe_inv(dx); iy = safe_inv(dy); iz = safe_inv(dz);
          oix = ox * ix; oiy = oy * iy; oiz = oz * iz;
          Dp = fmaf(A.ray_path[ray], T, Dp);
          tfar = INFINITY;
          tmin = 0;
          start = true;
        } else if (SERVE && done) {
          // written through to device scope
          if (gl == 0) {
            const uint32_t pix = (uint32_t)ray & ((1u << kServePixelBits) - 1u);
            st_dev(out_at + 3 * (int64_t)pix + 0, fmaf(T, A.bg0, C0));
            st_dev(out_at + 3 * (int64_t)pix + 1, fmaf(T, A.bg1, C1));
            st_dev(out_at + 3 * (int64_t)pix + 2, fmaf(T, A.bg2, C2));
            st_dev(out_at + 3 * (int64_t)out_n + pix, Dp);
            st_dev(out_at + 4 * (int64_t)out_n + pix, 1.f - T);
          }
          live = false;
        } else if (done) {
          if (gl == 0) {
            const float bgT = tfar == INFINITY ? T : 0.f;
            A.rgb[3 * (int64_t)ray + 0] = fmaf(bgT, A.bg0, C0);
            A.rgb[3 * (int64_t)ray + 1] = fmaf(bgT, A.bg1, C1);
            A.rgb[3 * (int64_t)ray + 2] = fmaf(bgT, A.bg2, C2);
            float depth = Dp;
            if (A.ray_kind && tfar == INFINITY && A.ray_tfar[ray] != INFINITY) depth = fmaf(-A.ray_path[ray], T, depth);
            A.depth[ray] = depth;
            A.opac[ray] = 1.f - T;
            if (A.hit_counts) A.hit_counts[ray] = nblend;
          }
          live = false;
        } else {
          start = true;
        }
      }
      if constexpr (SERVE) {
        // the rays that finished here, by request
        uint64_t fin = __ballot(ready && !cut && !live && gl == 0);
        const uint32_t slot = (uint32_t)ray >> kServePixelBits;
        while (fin) {
          const int l0 = __ffsll((unsigned long long)fin) - 1;
          const uint32_t s0 = (uint32_t)__builtin_amdgcn_readlane((int)slot, l0);
          const uint64_t same = fin & __ballot(slot == s0);
          if (fin_count && fin_slot != s0) count_finished(A);
          fin_slot = s0;
          fin_n = (uint32_t)__builtin_amdgcn_readlane((int)out_n, l0);
          fin_count += (uint32_t)__popcll(same);
          fin &= ~same;
        }
        if (q_next >= q_end) count_finished(A);
      }
      wave_order();
    } else if (leaves >= kGroupLeafLanes || 2 * leaves >= nodes) {
      // ---------------------------------------------------------- leaf step
      const float tnear = A.t_near;
      n_leaf -= q;
      uint2 it = make_uint2(0u, 0x7FC00000u);
      if (gl < q) it = G.item[kGroupRing + n_leaf + q - 1 - gl];
      const float te = __uint_as_float(it.y);
      bool hit = false;
      uint64_t key = 0;
      float rest = 1.f;
      if (gl < q && te <= tmax_t) {
        const uint32_t leaf = it.x & ~kLeafFlag;
        const float4* ip = A.inst + 4 * (int64_t)leaf;
        const float4 r0 = ip[0], r1 = ip[1], r2 = ip[2], r3 = ip[3];
        const SphereHit h = sphere_terms(r0, r1, r2, ox, oy, oz, dx, dy, dz);
        const float t0 = sphere_entry(h);
        key = make_key(fmaxf(t0, te), leaf);
        hit = h.a > 0.f && h.c2 <= h.a && t0 > tnear && t0 < tfar && key > tmin && key <= tmax;
        rest = hit_alpha(h, r3).rest;
      }
      const unsigned hits = (unsigned)(__ballot(hit) >> row0) & 0xFFFFu;
      if (hit) {
        const int e = n_hit + __popc(hits & ((1u << gl) - 1u));
        G.key[e] = key;
        G.rest[e] = rest;
      }
      n_hit += __popc(hits);
    } else {
      // ---------------------------------------------------------- node step
      const float tnear = A.t_near;
      if (__ballot(p > 0 && (in_ring > kGroupRing - 3 * kGroup || in_ring < p))) {
        uint2* const spill = group_spill(A, lane);
        if (p > 0 && in_ring > kGroupRing - 3 * kGroup) {
          // the ring's oldest entries move out
#pragma unroll
          for (int j = 0; j < kGroupMove; j += kGroup) {
            const uint2 v = G.item[(n_low + j + gl) & (kGroupRing - 1)];
            spill[n_low + j + gl] = v;
            low_t = fminf(low_t, __uint_as_float(v.y));
          }
          n_low += kGroupMove;
          low_t = row_min(low_t);
        } else if (p > 0 && in_ring < p) {
          // the latest to move out come back
          n_low -= kGroupMove;
#pragma unroll
          for (int j = 0; j < kGroupMove; j += kGroup) {
            const uint64_t v = *reinterpret_cast<const any_u64*>(spill + n_low + j + gl);
            G.item[(n_low + j + gl) & (kGroupRing - 1)] = make_uint2((uint32_t)v, (uint32_t)(v >> 32));
          }
          if (n_low == 0) low_t = INFINITY;
        }
        wave_order();
      }
      const int popped = n_node - p;
      uint2 it = make_uint2(0u, 0x7FC00000u);
      if (gl < p) it = G.item[(n_node - 1 - gl) & (kGroupRing - 1)];
      const float cur_t = __uint_as_float(it.y);
      const float tcap = fminf(tfar, tmax_t);
      uint64_t child[4];  // entry distance << 32 | reference; infinitely far: not entered
#pragma unroll
      for (int j = 0; j < 4; ++j) child[j] = kEmptyKey;
      if (gl < p && cur_t <= tmax_t) {
        // slab distances from the 8-bit planes, as in k_trace
        const float4* np = A.nodes + kNodeF4 * (int64_t)it.x;
        const float4 q0 = np[0], q1 = np[1], q2 = np[2], q3 = np[3];
        const float tlo = fmaxf(tnear, key_t(tmin));
        const float Ax = q0.w * ix, Ay = q1.x * iy, Az = q1.y * iz;
        const float Bx = fmaf(q0.x, ix, -oix), By = fmaf(q0.y, iy, -oiy), Bz = fmaf(q0.z, iz, -oiz);
        const uint32_t wlx = __float_as_uint(q2.z), wly = __float_as_uint(q2.w), wlz = __float_as_uint(q3.x);
        const uint32_t whx = __float_as_uint(q3.y), why = __float_as_uint(q3.z), whz = __float_as_uint(q3.w);
        const uint32_t wnx = ix < 0.f ? whx : wlx, wfx = ix < 0.f ? wlx : whx;
        const uint32_t wny = iy < 0.f ? why : wly, wfy = iy < 0.f ? wly : why;
        const uint32_t wnz = iz < 0.f ? whz : wlz, wfz = iz < 0.f ? wlz : whz;
        const uint32_t c[4] = {__float_as_uint(q1.z), __float_as_uint(q1.w), __float_as_uint(q2.x), __float_as_uint(q2.y)};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float tnx = fmaf((float)((wnx >> (8 * j)) & 0xFFu), Ax, Bx);
          const float tfx = fmaf((float)((wfx >> (8 * j)) & 0xFFu), Ax, Bx);
          const float tny = fmaf((float)((wny >> (8 * j)) & 0xFFu), Ay, By);
          const float tfy = fmaf((float)((wfy >> (8 * j)) & 0xFFu), Ay, By);
          const float tnz = fmaf((float)((wnz >> (8 * j)) & 0xFFu), Az, Bz);
          const float tfz = fmaf((float)((wfz >> (8 * j)) & 0xFFu), Az, Bz);
          const float tn = fmaxf(fmaxf(tnx, tny), tnz);
          // (entered before it ends, before the surface and not beyond t_max; ended after tlo,
          // which is never beyond t_max)
          const float tf = fminf(fminf(fminf(tfx, tfy), tfz), tcap);
          const float te = fmaxf(tn, cur_t);
          child[j] = make_key(c[j] != kNoChild && fmaxf(tn, tlo) <= tf ? te : INFINITY, c[j]);
        }
        // near to far; as doubles the pairs compare by distance (never a NaN: the exponent
        // field of a double takes eleven bits, of which a float leaves the last three clear)
        order2(child[0], child[1]);
        order2(child[2], child[3]);
        order2(child[0], child[2]);
        order2(child[1], child[3]);
        order2(child[1], child[2]);
      }
      // places on the two stacks: lane 0 popped the nearest node, so its children go on top
      int kind[4], mine = 0;  // 1 per internal node, 0x10000 per leaf
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        kind[j] = key_t(child[j]) < INFINITY ? ((uint32_t)child[j] & kLeafFlag ? 0x10000 : 1) : 0;
        mine += kind[j];
      }
      const int incl = row_scan(mine);
      const int total = __builtin_amdgcn_mov_dpp(incl, kRowBcast + kGroup - 1, 0xF, 0xF, true);
      int at = (((kGroupRing + n_leaf) << 16) | popped) + total - incl;
      n_node = popped + (total & 0xFFFF);
      n_leaf += total >> 16;
#pragma unroll
      for (int j = 3; j >= 0; --j) {
        const int i = (uint32_t)child[j] & kLeafFlag ? at >> 16 : at & (kGroupRing - 1);
        G.item[kind[j] ? i : kGroupRing + kGroupLeaves] = make_uint2((uint32_t)child[j], (uint32_t)(child[j] >> 32));
        at += kind[j];
      }
    }
  }
}

}  // namespace
}  // namespace grtx
