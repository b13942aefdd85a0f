// Batched depth ray casting of the envs' deformed surfaces (supplementary: depth simulation --
// depth maps, instance segmentation masks and point clouds cast from the simulation state).
//
// Create: per distinct surface topology a bounding-volume hierarchy over its triangles, built once
// on the host from the given rest shape (median split of triangle centroids along the longest axis,
// at most kLeafTris triangles per leaf) and stored four children to a node.  Nodes are numbered so that
// each subtree of at most kGroupTris triangles, and the nodes above them, list their levels deepest first.
// Every frame: the node boxes are refitted to the current vertex positions (one workgroup per subtree,
// then one per env for the nodes above), which also lays out each leaf's triangles side by side; then one
// thread per pixel traverses its env's hierarchy, nearest child first (FP32 slab tests, Moller-Trumbore
// with a closed barycentric band so that rays along shared edges are caught) and tests the env's obstacles
// analytically (plane, box slabs, capsule).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "../../include/flash.h"
#include "flash_common.h"

namespace {

using flash::FlashError;

constexpr int kLeafTris = 4;
constexpr int kMaxDepth = 48;         // create rejects deeper (binary) hierarchies
constexpr int kGroupTris = 1024;      // triangles of a refit workgroup's subtree: 256 leaves, one per thread
constexpr int kMaxEntries = 256;      // subtrees a workgroup chooses from, one per thread
constexpr int kNone = INT32_MIN;      // no child, no node
constexpr int kTile = 16;             // pixels per side of one workgroup's tile
constexpr int kRefitBlock = 256;
constexpr float kEdgeBand = 1e-6f;    // barycentric band: FP32 solves of a ray on a shared edge

struct DevCam {
  float o[3], R[9], fx, fy, cx, cy;
  float inv[9];   // of R
  int cull;       // R is a rotation up to rounding: boxes may be projected onto the image
};
struct DevObs {
  float c[3], R[9], size[3];
  int kind, pad[3];
};

// Nodes of a refit workgroup, contiguous, by level: level l is [off[l], off[l + 1]).
struct Group {
  int n_levels;
  int off[kMaxDepth / 2 + 2];
};

struct Topo {
  int n_vertices = 0;
  std::vector<int32_t> tris;          // 3 per triangle, local ids, as given
  std::vector<int4> bin;              // binary tree: (left, right, first, count): count > 0 = leaf of tris first..
  std::vector<int32_t> order;         // triangles in leaf order (index into the given list)
  // 4 children per node: a node id, -1 - leaf, or kNone; the root is the last node
  std::vector<int4> child;
  std::vector<int32_t> leaf_tri;      // 3 per triangle, kLeafTris triangles per leaf, the last one repeated
  std::vector<Group> groups;          // the subtrees, then (if there are several) the nodes above them
  int n_subtrees = 0;
  std::vector<int32_t> entries;       // at most kMaxEntries child slots (4 node + child) that cover the surface
  int depth = 0, levels = 0;          // nodes on the longest path from the root, and below an entry
  // device
  int4* d_child = nullptr;
  int4* d_tri = nullptr;              // leaf_tri
  Group* d_groups = nullptr;
  int* d_entries = nullptr;
};

// one env's part of a render
struct EnvRef {
  const int4* child;
  const int4* tri;
  const Group* groups;
  const int* entries;
  long long node0;      // first of its nodes in the box array
  long long leaf0;      // first of its leaves in the triangle array
  int voff;             // first vertex column in x
  int n_nodes;
  int n_subtrees, n_groups;
  int n_entries;
};

// The triangles a body shows: membrane triangles as given, or the faces of a tet mesh that
// belong to exactly one tet (its boundary), in the tets' own vertex order.
std::vector<int32_t> surface_of(const flash_env_desc& d) {
  std::vector<int32_t> out;
  if (d.elem == FLASH_TRI) {
    out.assign(d.elements, d.elements + 3 * (size_t)d.n_elements);
    return out;
  }
  static const int F[4][3] = {{1, 2, 3}, {0, 3, 2}, {0, 1, 3}, {0, 2, 1}};
  std::map<std::array<int32_t, 3>, int> count;
  for (int t = 0; t < d.n_elements; ++t)
    for (const auto& f : F) {
      std::array<int32_t, 3> key = {d.elements[4 * t + f[0]], d.elements[4 * t + f[1]], d.elements[4 * t + f[2]]};
      std::sort(key.begin(), key.end());
      count[key] += 1;
    }
  for (int t = 0; t < d.n_elements; ++t)
    for (const auto& f : F) {
      std::array<int32_t, 3> key = {d.elements[4 * t + f[0]], d.elements[4 * t + f[1]], d.elements[4 * t + f[2]]};
      std::sort(key.begin(), key.end());
      if (count[key] == 1)
        for (int a = 0; a < 3; ++a) out.push_back(d.elements[4 * t + f[a]]);
    }
  return out;
}

// Subtree over triangles order[lo, hi) at depth `level`; returns its node id.
int build_node(Topo& T, const std::vector<float>& cen, int lo, int hi, int level) {
  if (level + 1 >= kMaxDepth) throw FlashError(FLASH_ERR_INVALID_ARG, "surface hierarchy too deep");
  const int id = (int)T.bin.size();
  T.bin.push_back(make_int4(-1, -1, lo, hi - lo));
  if (hi - lo <= kLeafTris) return id;
  float bl[3] = {INFINITY, INFINITY, INFINITY}, bh[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int i = lo; i < hi; ++i)
    for (int k = 0; k < 3; ++k) {
      bl[k] = std::min(bl[k], cen[3 * (size_t)T.order[i] + k]);
      bh[k] = std::max(bh[k], cen[3 * (size_t)T.order[i] + k]);
    }
  int ax = 0;
  for (int k = 1; k < 3; ++k)
    if (bh[k] - bl[k] > bh[ax] - bl[ax]) ax = k;
  const int mid = lo + (hi - lo) / 2;
  std::nth_element(T.order.begin() + lo, T.order.begin() + mid, T.order.begin() + hi, [&](int a, int b) {
    const float ca = cen[3 * (size_t)a + ax], cb = cen[3 * (size_t)b + ax];
    return ca < cb || (ca == cb && a < b);
  });
  const int left = build_node(T, cen, lo, mid, level + 1);
  const int right = build_node(T, cen, mid, hi, level + 1);
  T.bin[id] = make_int4(left, right, lo, -(hi - lo));
  return id;
}

// Four children per node from the binary tree: a node's children, inner ones replaced by theirs.
struct WideNode {
  int kids[4];    // indices into the list (>= 0), leaves (-1 - leaf) or kNone
  int tris;
};
int widen(Topo& T, int b, std::vector<WideNode>& out) {
  const int id = (int)out.size();
  out.push_back({{kNone, kNone, kNone, kNone}, std::abs(T.bin[b].w)});
  int kid[4], n = 0;
  if (T.bin[b].w > 0) kid[n++] = b;   // a surface of one leaf
  else
    for (int c : {T.bin[b].x, T.bin[b].y}) {
      if (T.bin[c].w > 0) kid[n++] = c;
      else { kid[n++] = T.bin[c].x; kid[n++] = T.bin[c].y; }
    }
  for (int i = 0; i < n; ++i) {
    const int4 c = T.bin[kid[i]];
    int code;
    if (c.w > 0) {
      code = -1 - (int)(T.leaf_tri.size() / (3 * kLeafTris));
      for (int t = 0; t < kLeafTris; ++t)
        for (int a = 0; a < 3; ++a) T.leaf_tri.push_back(T.tris[3 * (size_t)T.order[c.z + std::min(t, c.w - 1)] + a]);
    } else {
      code = widen(T, kid[i], out);
    }
    out[id].kids[i] = code;
  }
  return id;
}

// Numbers the nodes below `root` that `in` admits, deepest level first, as the next group.
template <class F>
void number_group(const std::vector<WideNode>& W, int root, F in, std::vector<int>& id, int& next, Topo& T) {
  std::vector<std::vector<int>> lev(1, {root});
  for (;;) {
    std::vector<int> below;
    for (int w : lev.back())
      for (int c : W[w].kids)
        if (c >= 0 && in(c)) below.push_back(c);
    if (below.empty()) break;
    lev.push_back(below);
  }
  Group g{};
  g.n_levels = (int)lev.size();
  for (int l = 0; l < g.n_levels; ++l) {
    g.off[l] = next;
    for (int w : lev[g.n_levels - 1 - l]) id[w] = next++;
  }
  g.off[g.n_levels] = next;
  T.groups.push_back(g);
}

void build_bvh(Topo& T, const double* rest) {
  const int m = (int)(T.tris.size() / 3);
  std::vector<float> cen(3 * (size_t)m);
  for (int t = 0; t < m; ++t)
    for (int k = 0; k < 3; ++k) {
      double s = 0.0;
      for (int a = 0; a < 3; ++a) s += rest[3 * (size_t)T.tris[3 * t + a] + k];
      cen[3 * (size_t)t + k] = (float)(s / 3.0);
    }
  T.order.resize(m);
  for (int t = 0; t < m; ++t) T.order[t] = t;
  T.bin.clear();
  T.leaf_tri.clear();
  build_node(T, cen, 0, m, 0);
  std::vector<WideNode> W;
  widen(T, 0, W);
  // groups: the subtrees of at most kGroupTris triangles, then the nodes above
  std::vector<int> id(W.size(), -1), roots;
  if (W[0].tris <= kGroupTris) roots.push_back(0);
  else
    for (const WideNode& w : W)
      if (w.tris > kGroupTris)
        for (int c : w.kids)
          if (c >= 0 && W[c].tris <= kGroupTris) roots.push_back(c);
  int next = 0;
  for (int r : roots) number_group(W, r, [](int) { return true; }, id, next, T);
  T.n_subtrees = (int)roots.size();
  if (W[0].tris > kGroupTris) number_group(W, 0, [&](int c) { return W[c].tris > kGroupTris; }, id, next, T);
  T.child.resize(W.size());
  for (size_t w = 0; w < W.size(); ++w) {
    int k[4];
    for (int i = 0; i < 4; ++i) k[i] = W[w].kids[i] >= 0 ? id[W[w].kids[i]] : W[w].kids[i];
    T.child[id[w]] = make_int4(k[0], k[1], k[2], k[3]);
  }
  // entries: whole levels from the root down while they number at most kMaxEntries
  T.levels = 0;
  for (int g = 0; g < T.n_subtrees; ++g) T.levels = std::max(T.levels, T.groups[g].n_levels);
  if ((int)T.groups.size() > T.n_subtrees) T.levels += T.groups.back().n_levels;
  T.depth = T.levels;
  const int* code = reinterpret_cast<const int*>(T.child.data());
  auto slots_of = [&](int node, std::vector<int32_t>& out) {
    for (int c = 0; c < 4; ++c)
      if (code[4 * node + c] != kNone) out.push_back(4 * node + c);
  };
  T.entries.clear();
  slots_of((int)T.child.size() - 1, T.entries);
  for (T.levels -= 1; T.levels > 0; --T.levels) {
    std::vector<int32_t> below;
    for (int s : T.entries) {
      if (code[s] >= 0) slots_of(code[s], below);
      else below.push_back(s);
    }
    if (below.size() > kMaxEntries) break;
    T.entries = below;
  }
}

// ---------------------------------------------------------------------------------------------
// device

__device__ __forceinline__ float3 vtx(const float* x, long long ld, int col) {
  return make_float3(x[col], x[ld + col], x[2 * ld + col]);
}

// Boxes of a node's children: 6 x 4 floats (lower x, y, z of the four, then upper), relative to the camera.
constexpr int kNodeFloats = 24;
// A leaf: per triangle (o - A, B - A, C - A), o the camera's position: 9 floats in 3 float4.
constexpr int kLeafVecs = 3 * kLeafTris;

// Node boxes of one group (blockIdx.x, or the env's last with `top`) of one env (blockIdx.y), one thread per
// child, deepest level first.  Leaves also write their triangles.  All of an env's rays start at its camera, so
// the differences to it are formed once here, with the rounding they have in the ray tests.  Bound by the
// vertex gathers.  A sheet of 64800 triangles: 13 us (one env) and 92 us (48), both launches; with one
// workgroup per env over all levels, which left 255 CUs idle with one env, 236 and 304 us.
__global__ void __launch_bounds__(kRefitBlock) k_refit(const float* __restrict__ x, long long ld,
                                                       const EnvRef* __restrict__ envs,
                                                       const DevCam* __restrict__ cams, int top, float* boxes,
                                                       float4* __restrict__ tris) {
  const EnvRef E = envs[blockIdx.y];
  const int g = top ? E.n_subtrees : (int)blockIdx.x;
  if (g >= (top ? E.n_groups : E.n_subtrees)) return;
  const Group& G = E.groups[g];
  float* bx = boxes + kNodeFloats * E.node0;
  float4* tr = tris + kLeafVecs * E.leaf0;
  const float3 o = make_float3(cams[blockIdx.y].o[0], cams[blockIdx.y].o[1], cams[blockIdx.y].o[2]);
  const int nl = G.n_levels;
  for (int l = 0; l < nl; ++l) {
    const int s0 = 4 * G.off[l], s1 = 4 * G.off[l + 1];
    for (int s = s0 + threadIdx.x; s < s1; s += kRefitBlock) {
      const int code = reinterpret_cast<const int*>(E.child)[s];
      float lo0 = INFINITY, lo1 = INFINITY, lo2 = INFINITY, hi0 = -INFINITY, hi1 = -INFINITY, hi2 = -INFINITY;
      if (code >= 0) {
        const float* b = bx + kNodeFloats * (size_t)code;
        for (int i = 0; i < 4; ++i) {
          lo0 = fminf(lo0, b[i]); lo1 = fminf(lo1, b[4 + i]); lo2 = fminf(lo2, b[8 + i]);
          hi0 = fmaxf(hi0, b[12 + i]); hi1 = fmaxf(hi1, b[16 + i]); hi2 = fmaxf(hi2, b[20 + i]);
        }
      } else if (code != kNone) {
        const int leaf = -1 - code;
        const int4 i0 = E.tri[3 * (size_t)leaf], i1 = E.tri[3 * (size_t)leaf + 1], i2 = E.tri[3 * (size_t)leaf + 2];
        const int id[3 * kLeafTris] = {i0.x, i0.y, i0.z, i0.w, i1.x, i1.y, i1.z, i1.w, i2.x, i2.y, i2.z, i2.w};
        float3 p[3 * kLeafTris];
#pragma unroll
        for (int k = 0; k < 3 * kLeafTris; ++k) p[k] = vtx(x, ld, E.voff + id[k]);   // all loads go out together
        float4* q = tr + kLeafVecs * (size_t)leaf;
#pragma unroll
        for (int t = 0; t < kLeafTris; ++t) {
#pragma unroll
          for (int a = 3 * t; a < 3 * t + 3; ++a) {
            lo0 = fminf(lo0, p[a].x); lo1 = fminf(lo1, p[a].y); lo2 = fminf(lo2, p[a].z);
            hi0 = fmaxf(hi0, p[a].x); hi1 = fmaxf(hi1, p[a].y); hi2 = fmaxf(hi2, p[a].z);
          }
          const float3 A = p[3 * t], B = p[3 * t + 1], C = p[3 * t + 2];
          q[3 * t] = make_float4(o.x - A.x, o.y - A.y, o.z - A.z, B.x - A.x);
          q[3 * t + 1] = make_float4(B.y - A.y, B.z - A.z, C.x - A.x, C.y - A.y);
          q[3 * t + 2] = make_float4(C.z - A.z, 0.0f, 0.0f, 0.0f);
        }
        lo0 -= o.x; lo1 -= o.y; lo2 -= o.z;
        hi0 -= o.x; hi1 -= o.y; hi2 -= o.z;
      }
      float* out = bx + 6 * (size_t)(s & ~3) + (s & 3);
      out[0] = lo0; out[4] = lo1; out[8] = lo2; out[12] = hi0; out[16] = hi1; out[20] = hi2;
    }
    __syncthreads();
  }
}

// entry of the ray into a box given relative to its origin (INFINITY: none before tmax)
__device__ __forceinline__ float slab_entry(float lx, float ly, float lz, float hx, float hy, float hz, float3 inv,
                                            float tmax) {
  float t0 = lx * inv.x, t1 = hx * inv.x;
  float tn = fminf(t0, t1), tf = fmaxf(t0, t1);
  t0 = ly * inv.y; t1 = hy * inv.y;
  tn = fmaxf(tn, fminf(t0, t1)); tf = fminf(tf, fmaxf(t0, t1));
  t0 = lz * inv.z; t1 = hz * inv.z;
  tn = fmaxf(tn, fminf(t0, t1)); tf = fminf(tf, fmaxf(t0, t1));
  tn = fmaxf(tn, 0.0f);
  return (tn <= tf && tn < tmax) ? tn : INFINITY;
}

// Products with their roundings fixed: rays along shared edges are decided by the last bits, and the order in
// which a compiler fuses a sum of products is its own choice.
__device__ __forceinline__ float dot3(float3 a, float3 b) {
  return __fmaf_rn(a.z, b.z, __fmaf_rn(a.x, b.x, a.y * b.y));
}
__device__ __forceinline__ float det2(float a, float b, float c, float d) { return __fmaf_rn(a, b, -(c * d)); }

// triangle o - s, o - s + e1, o - s + e2
__device__ __forceinline__ float tri_hit(float3 d, float3 s, float3 e1, float3 e2) {
  const float3 P = make_float3(det2(d.y, e2.z, d.z, e2.y), det2(d.z, e2.x, d.x, e2.z), det2(d.x, e2.y, d.y, e2.x));
  const float det = dot3(P, e1);
  if (det == 0.0f) return INFINITY;
  const float inv = 1.0f / det;
  const float ps = dot3(P, s);
  const float3 Q = make_float3(det2(s.y, e1.z, s.z, e1.y), det2(s.z, e1.x, s.x, e1.z), det2(s.x, e1.y, s.y, e1.x));
  const float b1 = ps * inv;
  const float b2 = dot3(d, Q) * inv;
  const float t = dot3(e2, Q) * inv;
  const bool hit = b1 >= -kEdgeBand && b2 >= -kEdgeBand && __fmaf_rn(ps, inv, b2) <= 1.0f + kEdgeBand && t > 0.0f;
  return hit ? t : INFINITY;
}

// nearest t > 0 of the ray with one obstacle (INFINITY: none)
__device__ float obstacle_hit(const DevObs& ob, float3 o, float3 d) {
  const float* R = ob.R;
  if (ob.kind == FLASH_PLANE) {
    const float n0 = R[1], n1 = R[4], n2 = R[7];
    const float dn = d.x * n0 + d.y * n1 + d.z * n2;
    if (dn == 0.0f) return INFINITY;
    const float t = ((ob.c[0] - o.x) * n0 + (ob.c[1] - o.y) * n1 + (ob.c[2] - o.z) * n2) / dn;
    return t > 0.0f ? t : INFINITY;
  }
  // ray in the obstacle frame: ol = R^T (o - c), dl = R^T d
  const float r0 = o.x - ob.c[0], r1 = o.y - ob.c[1], r2 = o.z - ob.c[2];
  float ol[3], dl[3];
  for (int k = 0; k < 3; ++k) {
    ol[k] = R[k] * r0 + R[3 + k] * r1 + R[6 + k] * r2;
    dl[k] = R[k] * d.x + R[3 + k] * d.y + R[6 + k] * d.z;
  }
  if (ob.kind == FLASH_BOX) {
    float tn = -INFINITY, tf = INFINITY;
    for (int k = 0; k < 3; ++k) {
      const float e = ob.size[k];
      if (dl[k] == 0.0f) {
        if (fabsf(ol[k]) > e) return INFINITY;
        continue;
      }
      const float inv = 1.0f / dl[k];
      const float t0 = (-e - ol[k]) * inv, t1 = (e - ol[k]) * inv;
      tn = fmaxf(tn, fminf(t0, t1));
      tf = fminf(tf, fmaxf(t0, t1));
    }
    if (tn > tf) return INFINITY;
    const float t = tn > 0.0f ? tn : tf;
    return t > 0.0f ? t : INFINITY;
  }
  // capsule: radius size[0] around the local x axis, half-length size[1]
  const float rad = ob.size[0], half = ob.size[1];
  float best = INFINITY;
  const float a = dl[1] * dl[1] + dl[2] * dl[2];
  if (a > 0.0f) {
    const float b = 2.0f * (ol[1] * dl[1] + ol[2] * dl[2]);
    const float cc = ol[1] * ol[1] + ol[2] * ol[2] - rad * rad;
    const float disc = b * b - 4.0f * a * cc;
    if (disc >= 0.0f) {
      const float sq = sqrtf(disc);
      for (int sgn = -1; sgn <= 1; sgn += 2) {
        const float t = (-b + (float)sgn * sq) / (2.0f * a);
        const float x0 = ol[0] + t * dl[0];
        if (t > 0.0f && fabsf(x0) <= half && t < best) best = t;
      }
    }
  }
  const float dd = dl[0] * dl[0] + dl[1] * dl[1] + dl[2] * dl[2];
  for (int end = -1; end <= 1; end += 2) {
    const float oc0 = ol[0] - (float)end * half, oc1 = ol[1], oc2 = ol[2];
    const float bb = dl[0] * oc0 + dl[1] * oc1 + dl[2] * oc2;
    const float c2 = oc0 * oc0 + oc1 * oc1 + oc2 * oc2 - rad * rad;
    const float disc = bb * bb - dd * c2;
    if (disc < 0.0f) continue;
    const float sq = sqrtf(disc);
    for (int sgn = -1; sgn <= 1; sgn += 2) {
      const float t = (-bb + (float)sgn * sq) / dd;
      if (t > 0.0f && t < best) best = t;
    }
  }
  return best;
}

// Whether some ray of the pixels [u0, u0 + kTile) x [v0, v0 + kTile) may enter a box given relative to the camera
// (conservative: only boxes whose projection, with its rounding, lies outside are dropped); *key: its least depth.
__device__ bool tile_may_see(const DevCam& cam, const float (&lo)[3], const float (&hi)[3], int u0, int v0, float* key) {
  float zmin = INFINITY, pmax = 0.0f, ulo = INFINITY, uhi = -INFINITY, vlo = INFINITY, vhi = -INFINITY;
  bool bad = false;
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    const float x = c & 1 ? hi[0] : lo[0], y = c & 2 ? hi[1] : lo[1], z = c & 4 ? hi[2] : lo[2];
    const float* I = cam.inv;
    const float X = I[0] * x + I[1] * y + I[2] * z, Y = I[3] * x + I[4] * y + I[5] * z,
                Z = I[6] * x + I[7] * y + I[8] * z;
    const float rz = __builtin_amdgcn_rcpf(Z);   // (one unit in the last place, inside the pad)
    const float u = cam.fx * (X * rz), v = cam.fy * (Y * rz);
    bad = bad || !(fabsf(u) < INFINITY) || !(fabsf(v) < INFINITY) || !(Z > 0.0f);
    zmin = fminf(zmin, Z);
    pmax = fmaxf(pmax, fmaxf(fabsf(x), fmaxf(fabsf(y), fabsf(z))));
    ulo = fminf(ulo, u); uhi = fmaxf(uhi, u);
    vlo = fminf(vlo, v); vhi = fmaxf(vhi, v);
  }
  *key = zmin;
  if (bad || !(zmin > 1e-3f * pmax)) return true;   // near or behind the camera's plane
  const float k = pmax / zmin;
  const float pad = 1.0f + 4e-6f * (fmaxf(cam.fx, cam.fy) * k * (1.0f + k) + fabsf(cam.cx) + fabsf(cam.cy));
  const float ul = (float)u0 + 0.5f - cam.cx, vl = (float)v0 + 0.5f - cam.cy;
  return !(uhi + pad < ul) && !(ulo - pad > ul + kTile) && !(vhi + pad < vl) && !(vlo - pad > vl + kTile);
}

// One workgroup renders one 16 x 16 tile of one env's image, 8 x 8 pixels per wave; stack: LDS ints, one
// column per thread.  What bounds it: vector instructions of the slab and triangle tests.  PICK: the workgroup
// first picks, with one test per thread, the subtrees (of up to kMaxEntries) whose boxes project onto the tile,
// nearest first; each ray starts at those, which spares it the upper half of the descent.  Four children per
// node halve the dependent loads of the rest; their boxes and a leaf's triangles are read 16 bytes at a
// time; lanes go on through inner nodes until the wave's all have a leaf, so that the triangle tests run
// together.  One 128 x 128 image of a 64800-triangle sheet: 32 us (81 us with binary nodes, triangles through
// their vertex ids and the stack in scratch); 48 of 640 x 480: 590 us, 711 from the root, 1445 us before.
template <bool PICK>
__global__ void __launch_bounds__(kTile * kTile) k_render(const float4* __restrict__ tris,
                                                          const EnvRef* __restrict__ envs,
                                                          const float* __restrict__ boxes, const DevCam* __restrict__ cams,
                                                          const DevObs* __restrict__ obs, const int* __restrict__ nobs,
                                                          int width, int height, int tiles_x, float* depth,
                                                          int* inst, float* pts) {
  extern __shared__ int stack_lds[];
  constexpr int NE = PICK ? kMaxEntries : 1;
  __shared__ float s_box[6][NE], s_key[NE];
  __shared__ int s_code[NE], s_order[NE];
  __shared__ int s_count[kTile * kTile / 64];
  const int e = blockIdx.y;
  const int tile = blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int u0 = (tile % tiles_x) * kTile, v0 = (tile / tiles_x) * kTile;
  const EnvRef E = envs[e];
  const DevCam& cam = cams[e];
  int n_entries = 0;
  if constexpr (PICK) {
    float lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0}, key = 0.0f;
    int code = kNone;
    bool keep = false;
    if ((int)threadIdx.x < E.n_entries) {
      const int s = E.entries[threadIdx.x];
      const float* b = boxes + kNodeFloats * (E.node0 + (s >> 2)) + (s & 3);
      for (int k = 0; k < 3; ++k) { lo[k] = b[4 * k]; hi[k] = b[12 + 4 * k]; }
      code = reinterpret_cast<const int*>(E.child)[s];
      keep = tile_may_see(cam, lo, hi, u0, v0, &key) | !cam.cull;
    }
    const unsigned long long m = __ballot(keep);
    if (lane == 0) s_count[wave] = __popcll(m);
    __syncthreads();
    int at = __popcll(m & ((1ull << lane) - 1ull));
    for (int w = 0; w < kTile * kTile / 64; ++w) {
      if (w < wave) at += s_count[w];
      n_entries += s_count[w];
    }
    if (keep) {
      for (int k = 0; k < 3; ++k) { s_box[k][at] = lo[k]; s_box[3 + k][at] = hi[k]; }
      s_code[at] = code;
      s_key[at] = key == key ? key : -INFINITY;
    }
    __syncthreads();
    if ((int)threadIdx.x < n_entries) {   // nearest first, ties in list order
      const float mine = s_key[threadIdx.x];
      int rank = 0;
      for (int q = 0; q < n_entries; ++q) rank += (s_key[q] < mine) | ((s_key[q] == mine) & (q < (int)threadIdx.x));
      s_order[rank] = threadIdx.x;
    }
    __syncthreads();
  }
  const int u = u0 + 8 * (wave & 1) + (lane & 7);
  const int v = v0 + 8 * (wave >> 1) + (lane >> 3);
  if (u >= width || v >= height) return;
  const float xn = ((float)u + 0.5f - cam.cx) / cam.fx;
  const float yn = ((float)v + 0.5f - cam.cy) / cam.fy;
  const float3 o = make_float3(cam.o[0], cam.o[1], cam.o[2]);
  const float3 d = make_float3(__fmaf_rn(cam.R[0], xn, cam.R[1] * yn) + cam.R[2],
                               __fmaf_rn(cam.R[3], xn, cam.R[4] * yn) + cam.R[5],
                               __fmaf_rn(cam.R[6], xn, cam.R[7] * yn) + cam.R[8]);
  const float3 inv = make_float3(1.0f / d.x, 1.0f / d.y, 1.0f / d.z);
  float tbest = INFINITY;
  int ibest = -1;
  if (PICK ? n_entries > 0 : E.n_nodes > 0) {
    const float4* bx = reinterpret_cast<const float4*>(boxes + kNodeFloats * E.node0);
    const float4* tr = tris + kLeafVecs * E.leaf0;
    int* stack = stack_lds + threadIdx.x;
    int sp = 0, next = 0;
    if (!PICK) stack[kTile * kTile * sp++] = E.n_nodes - 1;
    for (;;) {
      int cur = kNone;
      if (sp > 0) {
        cur = stack[kTile * kTile * --sp];
      } else {
        while (next < n_entries) {
          const int q = s_order[next++];
          if (slab_entry(s_box[0][q], s_box[1][q], s_box[2][q], s_box[3][q], s_box[4][q], s_box[5][q], inv, tbest) <
              INFINITY) {
            cur = s_code[q];
            break;
          }
        }
        if (cur == kNone) break;
      }
      while (cur >= 0) {
        const float4* b = bx + kNodeFloats / 4 * (size_t)cur;
        const float4 lx = b[0], ly = b[1], lz = b[2], hx = b[3], hy = b[4], hz = b[5];
        const int4 ch = E.child[cur];
        const float t0 = ch.x != kNone ? slab_entry(lx.x, ly.x, lz.x, hx.x, hy.x, hz.x, inv, tbest) : INFINITY;
        const float t1 = ch.y != kNone ? slab_entry(lx.y, ly.y, lz.y, hx.y, hy.y, hz.y, inv, tbest) : INFINITY;
        const float t2 = ch.z != kNone ? slab_entry(lx.z, ly.z, lz.z, hx.z, hy.z, hz.z, inv, tbest) : INFINITY;
        const float t3 = ch.w != kNone ? slab_entry(lx.w, ly.w, lz.w, hx.w, hy.w, hz.w, inv, tbest) : INFINITY;
        // the nearest child next, the others that the ray enters on the stack
        const bool a = t1 < t0, c = t3 < t2;
        const float ta = a ? t1 : t0, tc = c ? t3 : t2;
        const int na = a ? ch.y : ch.x, nc = c ? ch.w : ch.z;
        const int fa = a ? ch.x : ch.y, fc = c ? ch.z : ch.w;
        const float sa = a ? t0 : t1, sc = c ? t2 : t3;
        const bool near_c = tc < ta;
        if (sa < INFINITY) { stack[kTile * kTile * sp] = fa; ++sp; }
        if (sc < INFINITY) { stack[kTile * kTile * sp] = fc; ++sp; }
        const float far_t = near_c ? ta : tc;
        if (far_t < INFINITY) { stack[kTile * kTile * sp] = near_c ? na : nc; ++sp; }
        cur = near_c ? nc : na;
        if (!(fminf(ta, tc) < INFINITY)) cur = sp > 0 ? stack[kTile * kTile * --sp] : kNone;
      }
      if (cur == kNone) continue;
      float4 q[kLeafVecs];
#pragma unroll
      for (int k = 0; k < kLeafVecs; ++k) q[k] = tr[kLeafVecs * (size_t)(-1 - cur) + k];
#pragma unroll
      for (int t = 0; t < kLeafTris; ++t) {   // a short leaf repeats its last triangle
        const float4 a = q[3 * t], b = q[3 * t + 1];
        const float th = tri_hit(d, make_float3(a.x, a.y, a.z), make_float3(a.w, b.x, b.y),
                                 make_float3(b.z, b.w, q[3 * t + 2].x));
        if (th < tbest) { tbest = th; ibest = 0; }
      }
    }
  }
  const int no = nobs[e];
  for (int q = 0; q < no; ++q) {
    const float th = obstacle_hit(obs[(size_t)e * FLASH_MAX_OBSTACLES + q], o, d);
    if (th < tbest) { tbest = th; ibest = 1 + q; }
  }
  const size_t px = ((size_t)e * height + v) * width + u;
  const bool hit = ibest >= 0;
  if (depth) depth[px] = hit ? tbest : 0.0f;
  if (inst) inst[px] = ibest;
  if (pts) {
    pts[3 * px] = hit ? o.x + tbest * d.x : 0.0f;
    pts[3 * px + 1] = hit ? o.y + tbest * d.y : 0.0f;
    pts[3 * px + 2] = hit ? o.z + tbest * d.z : 0.0f;
  }
}

}  // namespace

struct flash_renderer {
  int n_envs = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  std::vector<Topo> topos;
  std::vector<EnvRef> envs;
  std::vector<int> voff;
  long long n_nodes = 0, n_leaves = 0;
  int max_subtrees = 0, max_levels = 0, max_depth = 0;
  bool any_top = false;               // some env has nodes above its subtrees
  std::vector<void*> owned;
  EnvRef* d_envs = nullptr;
  float* d_boxes = nullptr;
  float4* d_tris = nullptr;
  // a frame's cameras, obstacles and obstacle counts, one block on either side: one copy per frame
  DevCam* d_cams = nullptr;
  DevObs* d_obs = nullptr;
  int* d_nobs = nullptr;
  void* h_frame = nullptr;            // pinned
  size_t frame_bytes = 0;
  DevCam* h_cams = nullptr;
  DevObs* h_obs = nullptr;
  int* h_nobs = nullptr;

  ~flash_renderer() {
    if (stream) (void)hipStreamSynchronize(stream);
    for (void* p : owned) (void)hipFree(p);
    if (h_frame) (void)hipHostFree(h_frame);
    if (own_stream && stream) (void)hipStreamDestroy(stream);
  }
  template <class X>
  X* alloc(size_t n) {
    void* p = nullptr;
    HIPCHK(hipMalloc(&p, std::max<size_t>(n, 1) * sizeof(X)));
    owned.push_back(p);
    return static_cast<X*>(p);
  }
};

// Inverse of a camera's R; false where R is no rotation (to 1e-3) and boxes cannot be projected with it.
static bool rotation_inverse(const double* R, float* inv) {
  bool ok = true;
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      double g = 0.0;
      for (int k = 0; k < 3; ++k) g += R[3 * k + i] * R[3 * k + j];
      ok = ok && std::fabs(g - (i == j ? 1.0 : 0.0)) < 1e-3;
    }
  const double det = R[0] * (R[4] * R[8] - R[5] * R[7]) - R[1] * (R[3] * R[8] - R[5] * R[6]) +
                     R[2] * (R[3] * R[7] - R[4] * R[6]);
  for (int i = 0; i < 3; ++i)
    for (int j = 0; j < 3; ++j) {
      const int a = (j + 1) % 3, b = (j + 2) % 3, c = (i + 1) % 3, d = (i + 2) % 3;
      inv[3 * i + j] = ok ? (float)((R[3 * a + c] * R[3 * b + d] - R[3 * a + d] * R[3 * b + c]) / det) : 0.0f;
    }
  return ok;
}

extern "C" {

flash_status flash_renderer_create(const flash_env_desc* descs, int32_t n_envs, void* hip_stream,
                                   flash_renderer** out) {
  if (!out || !descs || n_envs <= 0) return flash::record_error(FLASH_ERR_INVALID_ARG, "null argument or n_envs <= 0");
  *out = nullptr;
  std::vector<std::vector<int32_t>> surf(n_envs);
  std::vector<int> n_vertices(n_envs), n_tris(n_envs);
  for (int e = 0; e < n_envs; ++e) {
    const flash_env_desc& d = descs[e];
    const int k = d.elem == FLASH_TET ? 4 : 3;
    if ((d.elem != FLASH_TET && d.elem != FLASH_TRI) || d.n_vertices <= 0 || d.n_elements <= 0 || !d.rest_x ||
        !d.elements)
      return flash::record_error(FLASH_ERR_INVALID_ARG, "invalid surface of env " + std::to_string(e));
    for (int64_t q = 0; q < (int64_t)k * d.n_elements; ++q)
      if (d.elements[q] < 0 || d.elements[q] >= d.n_vertices)
        return flash::record_error(FLASH_ERR_INVALID_ARG, "element vertex out of range in env " + std::to_string(e));
    surf[e] = surface_of(d);
    n_vertices[e] = d.n_vertices;
    n_tris[e] = (int)(surf[e].size() / 3);
  }
  flash_renderer* r = new flash_renderer();
  try {
    r->n_envs = n_envs;
    if (hip_stream) r->stream = static_cast<hipStream_t>(hip_stream);
    else { HIPCHK(hipStreamCreateWithFlags(&r->stream, hipStreamNonBlocking)); r->own_stream = true; }
    r->voff.assign(n_envs + 1, 0);
    for (int e = 0; e < n_envs; ++e) r->voff[e + 1] = r->voff[e] + n_vertices[e];
    // topologies: equal triangle lists over equal vertex counts share one hierarchy
    std::map<std::pair<int, int>, std::vector<int>> seen;
    std::vector<int> env_topo(n_envs);
    for (int e = 0; e < n_envs; ++e) {
      int id = -1;
      for (int t : seen[{n_vertices[e], n_tris[e]}]) {
        const Topo& T = r->topos[t];
        if (T.tris == surf[e]) { id = t; break; }
      }
      if (id < 0) {
        Topo T;
        T.n_vertices = n_vertices[e];
        T.tris = surf[e];
        if (n_tris[e] > 0) build_bvh(T, descs[e].rest_x);
        id = (int)r->topos.size();
        r->topos.push_back(std::move(T));
        seen[{n_vertices[e], n_tris[e]}].push_back(id);
      }
      env_topo[e] = id;
    }
    for (Topo& T : r->topos) {
      T.d_child = r->alloc<int4>(T.child.size());
      T.d_tri = r->alloc<int4>(T.leaf_tri.size() / 4);
      T.d_groups = r->alloc<Group>(T.groups.size());
      T.d_entries = r->alloc<int>(T.entries.size());
      if (!T.child.empty()) {
        HIPCHK(hipMemcpy(T.d_child, T.child.data(), T.child.size() * sizeof(int4), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(T.d_tri, T.leaf_tri.data(), T.leaf_tri.size() * sizeof(int), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(T.d_groups, T.groups.data(), T.groups.size() * sizeof(Group), hipMemcpyHostToDevice));
        HIPCHK(hipMemcpy(T.d_entries, T.entries.data(), T.entries.size() * sizeof(int), hipMemcpyHostToDevice));
      }
      r->max_subtrees = std::max(r->max_subtrees, T.n_subtrees);
      r->max_levels = std::max(r->max_levels, T.levels);
      r->max_depth = std::max(r->max_depth, T.depth);
      r->any_top |= (int)T.groups.size() > T.n_subtrees;
    }
    for (int e = 0; e < n_envs; ++e) {
      const Topo& T = r->topos[env_topo[e]];
      EnvRef E{};
      E.child = T.d_child;
      E.tri = T.d_tri;
      E.groups = T.d_groups;
      E.node0 = r->n_nodes;
      E.leaf0 = r->n_leaves;
      E.voff = r->voff[e];
      E.n_nodes = (int)T.child.size();
      E.n_subtrees = T.n_subtrees;
      E.n_groups = (int)T.groups.size();
      E.entries = T.d_entries;
      E.n_entries = (int)T.entries.size();
      r->n_nodes += E.n_nodes;
      r->n_leaves += (long long)T.leaf_tri.size() / (3 * kLeafTris);
      r->envs.push_back(E);
    }
    r->d_envs = r->alloc<EnvRef>(n_envs);
    HIPCHK(hipMemcpy(r->d_envs, r->envs.data(), n_envs * sizeof(EnvRef), hipMemcpyHostToDevice));
    r->d_boxes = r->alloc<float>((size_t)r->n_nodes * kNodeFloats);
    r->d_tris = r->alloc<float4>((size_t)r->n_leaves * kLeafVecs);
    const size_t obs_at = n_envs * sizeof(DevCam);
    const size_t nobs_at = obs_at + (size_t)n_envs * FLASH_MAX_OBSTACLES * sizeof(DevObs);
    r->frame_bytes = nobs_at + n_envs * sizeof(int);
    unsigned char* d = r->alloc<unsigned char>(r->frame_bytes);
    HIPCHK(hipHostMalloc(&r->h_frame, r->frame_bytes, hipHostMallocDefault));
    unsigned char* h = static_cast<unsigned char*>(r->h_frame);
    std::memset(h, 0, r->frame_bytes);
    r->d_cams = reinterpret_cast<DevCam*>(d);
    r->d_obs = reinterpret_cast<DevObs*>(d + obs_at);
    r->d_nobs = reinterpret_cast<int*>(d + nobs_at);
    r->h_cams = reinterpret_cast<DevCam*>(h);
    r->h_obs = reinterpret_cast<DevObs*>(h + obs_at);
    r->h_nobs = reinterpret_cast<int*>(h + nobs_at);
  } catch (const FlashError& ex) {
    delete r;
    return flash::record_error(ex.st, ex.what());
  }
  *out = r;
  return FLASH_OK;
}

flash_status flash_renderer_destroy(flash_renderer* r) {
  if (!r) return flash::record_error(FLASH_ERR_INVALID_ARG, "null renderer");
  delete r;
  return FLASH_OK;
}

flash_status flash_render(flash_renderer* r, const float* x_dev, int64_t ld, const flash_obstacle* obstacles,
                          const int32_t* n_obstacles, const flash_camera* cams, int32_t width, int32_t height,
                          float* depth_dev, int32_t* instance_dev, float* points_dev) {
  if (!r || !cams || width <= 0 || height <= 0 || (!x_dev && r->voff.back() > 0))
    return flash::record_error(FLASH_ERR_INVALID_ARG, "null renderer, cameras or positions, or empty image");
  if (ld < r->voff.back()) return flash::record_error(FLASH_ERR_INVALID_ARG, "ld below the total vertex count");
  const int ne = r->n_envs;
  for (int e = 0; e < ne; ++e) {
    const int no = n_obstacles ? n_obstacles[e] : 0;
    if (no < 0 || no > FLASH_MAX_OBSTACLES || (no > 0 && !obstacles))
      return flash::record_error(FLASH_ERR_INVALID_ARG, "invalid obstacle count of env " + std::to_string(e));
    if (!(cams[e].fx > 0) || !(cams[e].fy > 0))
      return flash::record_error(FLASH_ERR_INVALID_ARG, "camera focal lengths must be positive");
    DevCam& c = r->h_cams[e];
    for (int k = 0; k < 3; ++k) c.o[k] = (float)cams[e].position[k];
    for (int k = 0; k < 9; ++k) c.R[k] = (float)cams[e].rot[k];
    c.cull = rotation_inverse(cams[e].rot, c.inv) ? 1 : 0;
    c.fx = (float)cams[e].fx; c.fy = (float)cams[e].fy; c.cx = (float)cams[e].cx; c.cy = (float)cams[e].cy;
    r->h_nobs[e] = no;
    for (int q = 0; q < no; ++q) {
      const flash_obstacle& ob = obstacles[(size_t)e * FLASH_MAX_OBSTACLES + q];
      if (ob.kind != FLASH_PLANE && ob.kind != FLASH_BOX && ob.kind != FLASH_CAPSULE)
        return flash::record_error(FLASH_ERR_INVALID_ARG, "unknown obstacle kind");
      DevObs& d = r->h_obs[(size_t)e * FLASH_MAX_OBSTACLES + q];
      for (int k = 0; k < 3; ++k) { d.c[k] = (float)ob.center[k]; d.size[k] = (float)ob.size[k]; }
      for (int k = 0; k < 9; ++k) d.R[k] = (float)ob.rot[k];
      d.kind = ob.kind;
    }
  }
  try {
    HIPCHK(hipMemcpyAsync(r->d_cams, r->h_frame, r->frame_bytes, hipMemcpyHostToDevice, r->stream));
    if (r->max_subtrees > 0)
      hipLaunchKernelGGL(k_refit, dim3((unsigned)r->max_subtrees, (unsigned)ne), dim3(kRefitBlock), 0, r->stream, x_dev,
                         (long long)ld, r->d_envs, r->d_cams, 0, r->d_boxes, r->d_tris);
    if (r->any_top)
      hipLaunchKernelGGL(k_refit, dim3(1, (unsigned)ne), dim3(kRefitBlock), 0, r->stream, x_dev, (long long)ld,
                         r->d_envs, r->d_cams, 1, r->d_boxes, r->d_tris);
    const int tx = (width + kTile - 1) / kTile, ty = (height + kTile - 1) / kTile;
    // Subtrees are picked per tile where an image has at least as many tiles as a surface has entries, so that a
    // tile sees few of them: 48 frames of 640 x 480 784 us with, 919 without (whole calls, a 64800-triangle sheet),
    // of 320 x 240 418 and 446; below, testing a tile's many entries costs what it saves (16 frames of 128 x 128
    // 164 with, 148 without, one frame 85 and 69).
    const bool pick = tx * ty >= kMaxEntries;
    // a node leaves at most three children on the stack on the way down
    const size_t lds = (size_t)kTile * kTile * sizeof(int) * (3 * (pick ? r->max_levels : r->max_depth) + 1);
    const auto kernel = pick ? k_render<true> : k_render<false>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(tx * ty), (unsigned)ne), dim3(kTile * kTile), lds, r->stream,
                       (const float4*)r->d_tris, r->d_envs, (const float*)r->d_boxes, r->d_cams, r->d_obs, r->d_nobs,
                       width, height, tx, depth_dev, instance_dev, points_dev);
    HIPCHK(hipGetLastError());
    // the host staging arrays are reused by the next call: let the copies finish
    HIPCHK(hipStreamSynchronize(r->stream));
  } catch (const FlashError& ex) {
    return flash::record_error(ex.st, ex.what());
  }
  return FLASH_OK;
}

}  // extern "C"
