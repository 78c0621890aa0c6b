// Two steps of the hybrid scheme in one pass over the state (half-link
// membranes, both lattices, both storage precisions).
//
// A step moves its whole state through HBM and little else (one read and one
// write of every population, about one FP64 operation per byte), so the time
// of a long forward is the number of passes.  k_pair advances a tile of site
// columns from step k to step k + 2: while a workgroup walks the z layers of
// its tile it updates each layer to step k + 1 in registers, and the layer
// below it, whose neighbours at step k + 1 are then all known, to step k + 2.
//
// * A workgroup holds a rectangle of tix x tiy columns and a ring of one
//   column around it, one thread per column (no corners: the lattices have
//   no diagonal links).  Ring columns are updated to k + 1 only.
// * In a thread's column the z neighbours are values of its own (the layer
//   it updated before, the layer it updates now).  The x and y neighbours
//   come through LDS: two layers of the four x and y populations.
// * The state at k + 1 is rounded to the storage type before it is used, as
//   a stored state is: populations and M are bit for bit those of two single
//   steps.
// * Beyond an outer face a ring column is the column that the face stands
//   for: the wrapped one of the same field (modified periodic) or the same
//   column of the reflected image field (mirror), updated with that field's
//   phases and its own faces; the layers below 0 and above n2 - 1 likewise.
//   The pull through the face at step k + 1 then applies the face's factor
//   and conjugation as a single step does.
// * Loads of the next layer are issued before a layer's arithmetic, and one
//   barrier per layer separates the two LDS layers.
// * Addresses are a wave-uniform base of the layer and a 32-bit byte offset
//   per thread from the first field of the q-sample, so the image fields of a
//   q-sample have to begin within 4 GiB (the host takes single steps
//   otherwise).
//
// What it measured (us per step of a forward, single steps -> this, one
// session): 256^3 x 12 fields 4334 -> 3161, x 24 8902 -> 6270, 128^3 x 24 993
// -> 814, FP64 96^3 x 8 280 -> 216, D2Q5 512^2 x 48 180 -> 133.  On 256^3 x 12
// a pass that is not the first takes 6.43 ms, reads 1.5 times the state (16.6
// GB, the lines of the ring again for every tile) and writes it once (12.1
// GB): 4.5 TB/s together.  Neither that nor the vector units (busy for 40 % of
// the time) bound it alone: without its loads a pass took 60 % of its time,
// and the two workgroups of a compute unit hide the loads from each other only
// in part.  FP64 D3Q7 has one workgroup there (94 KB of LDS; 157 registers
// would allow three waves per SIMD, there are two), whose loads nothing hides.
#include <type_traits>

#include "btl_device.h"

namespace btl {

// Populations are reached through buffer descriptors: the wave-uniform address
// of a layer (in scalar registers, raw buffer of 32-bit range), a scalar
// offset of the plane and a 32-bit byte offset of the thread, so an access
// takes no 64-bit arithmetic per thread.
using Layer = __amdgpu_buffer_rsrc_t;
__device__ __forceinline__ Layer layer_at(const void* base, int64_t off, uint32_t bytes = ~0u) {
    char* p = const_cast<char*>(static_cast<const char*>(base)) + off;
    return __builtin_amdgcn_make_buffer_rsrc(p, 0, (int)bytes, 0x00020000);
}
// Offset of a store that a thread does not make: beyond the descriptor's range
// (a layer has at most 2^31 bytes, checked on the host), where the buffer
// instruction writes nothing.  A branch around the stores would leave the
// compiler not knowing how many are in flight, and it would wait for them.
constexpr uint32_t kNoStore = 0x80000000u;
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ float2 load_at(Layer l, uint32_t off, uint32_t plane, float2*) {
    const u32x2 r = __builtin_amdgcn_raw_buffer_load_b64(l, off, plane, 0);
    return make_float2(__uint_as_float(r.x), __uint_as_float(r.y));
}
__device__ __forceinline__ double2 load_at(Layer l, uint32_t off, uint32_t plane, double2*) {
    const u32x4 r = __builtin_amdgcn_raw_buffer_load_b128(l, off, plane, 0);
    return make_double2(__hiloint2double(r.y, r.x), __hiloint2double(r.w, r.z));
}
constexpr int kNonTemporal = 2;
__device__ __forceinline__ void store_at(Layer l, uint32_t off, uint32_t plane, double2 v, float2*) {
    const u32x2 r = {__float_as_uint((float)v.x), __float_as_uint((float)v.y)};
    __builtin_amdgcn_raw_buffer_store_b64(r, l, off, plane, kNonTemporal);
}
__device__ __forceinline__ void store_at(Layer l, uint32_t off, uint32_t plane, double2 v, double2*) {
    const u32x4 r = {(uint32_t)__double2loint(v.x), (uint32_t)__double2hiint(v.x),
                     (uint32_t)__double2loint(v.y), (uint32_t)__double2hiint(v.y)};
    __builtin_amdgcn_raw_buffer_store_b128(r, l, off, plane, kNonTemporal);
}
template <typename V>
__device__ __forceinline__ V pick(bool c, V a, V b) {
    return V{c ? a.x : b.x, c ? a.y : b.y};
}

template <typename V, int NQ, int NT, int WPE, bool FIRST>
__global__ void __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WPE, WPE)))
k_pair(PairArgs a) {
    constexpr double W0 = lattice_w0(NQ), W1 = lattice_w1(NQ);
    constexpr int pz = NQ == 7 ? 5 : 3;      // planes pz (+z) and pz + 1 (-z)
    constexpr int NX = NQ - 3;               // x (and y) populations, exchanged through LDS
    extern __shared__ double2 smem[];
    __shared__ double c_w[kMaxPhase], c_dec[kMaxPhase], c_trans[kTransSize];
    __shared__ int c_kind[4 * 6];
    __shared__ double2 c_red[2][NT / 64];
    __shared__ double2 c_exy[2][NT];         // reaction factors of the columns at steps k, k + 1
    __shared__ V xch[2 * NX * NT];           // [2][NX][NT]
    __shared__ uint4 c_pull[FIRST ? 1 : NT]; // byte offsets of the columns' x and y pulls
    __shared__ uint32_t c_image[FIRST ? 1 : NT];   // and of their images across z
    double2* c_ez = smem;                    // [4][zr]: columns of set 0 .. 2 at step k, own at k + 1
    double2* c_fac = smem + 4 * a.zr;        // [5][6]: sets 0 .. 3 at step k, own at step k + 1

    const int32_t lb = a.xcd ? xcd_tile((int32_t)blockIdx.x, (int32_t)gridDim.x)
                             : (int32_t)blockIdx.x;
    const int2 fbk = a.blk_field[lb];
    const int fi = fbk.x;
    const PairField& fd = a.fields[fi];
    const int32_t n0 = fd.n[0], n1 = fd.n[1], n2 = fd.n[2];
    const int32_t b = fbk.y;
    const int32_t tx = b % fd.tiles[0];
    const int32_t rb = b / fd.tiles[0];
    const int32_t ty = rb % fd.tiles[1];
    const int32_t z0 = (rb / fd.tiles[1]) * fd.zc;
    const int32_t z1 = min(n2, z0 + fd.zc);
    const bool mz = (fd.face_kind[4] & kFaceMirror) != 0;
    const int P = a.n_phase;
    const int t = (int)threadIdx.x;
    // layer j of the walk, z0 - 1 .. z1: the lattice layer it stands for, and
    // whether it belongs to the z image field
    auto layer_of = [&](int32_t j) -> int32_t {
        return j < 0 ? (mz ? 0 : n2 - 1) : j >= n2 ? (mz ? n2 - 1 : 0) : j;
    };
    auto beyond = [&](int32_t j) -> bool { return j < 0 || j >= n2; };

    if (t < P) {
        c_w[t] = a.w[t];
        c_dec[t] = a.decay[t];
    }
    for (int i = t; i < kTransSize; i += (int)blockDim.x) fill_transmitted(c_trans, a.trans, P, i);
    // sets: 0 the field itself, 1 .. 3 its image fields across x, y and z
    auto set_field = [&](int s) -> int { return s == 0 ? fi : fd.part[s - 1]; };
    for (int i = t; i < 30; i += (int)blockDim.x) {
        const int s = i / 6, f = i % 6;
        const PairField& o = a.fields[s == 4 ? fi : set_field(s)];
        c_fac[i] = (s == 4 ? a.tab1 : a.tab0)[o.tab + n0 + n1 + n2 + f];
        if (s < 4) c_kind[i] = o.face_kind[f];
    }
    const int32_t nl = z1 - z0 + 2;
    for (int i = t; i < 4 * nl; i += (int)blockDim.x) {
        const int s = i / nl, l = i % nl;
        const int32_t j = z0 - 1 + l, jv = layer_of(j);
        const PairField& o = a.fields[s == 3 ? fi : s == 0 && mz && beyond(j) ? fd.part[2]
                                                                             : set_field(s)];
        c_ez[s * a.zr + l] = (s == 3 ? a.tab1 : a.tab0)[o.tab + n0 + n1 + jv];
    }

    // the thread's column
    const int32_t bx = fd.tix + 2, by = NQ == 7 ? fd.tiy + 2 : 1;
    const int32_t ly = t / bx, lx = t - ly * bx;
    const int32_t x = tx * fd.tix - 1 + lx;
    const int32_t y = NQ == 7 ? ty * fd.tiy - 1 + ly : 0;
    const bool in_x = lx >= 1 && lx <= fd.tix && x < n0;
    const bool in_y = NQ == 7 ? ly >= 1 && ly <= fd.tiy && y < n1 : t < bx;
    const bool ring_x = in_y && !in_x && lx < bx && x <= n0;
    const bool ring_y = NQ == 7 && in_x && !in_y && ly < by && y <= n1;
    const bool inner = in_x && in_y;
    const bool active = inner || ring_x || ring_y;
    int set = 0;
    int32_t xv = min(max(x, 0), n0 - 1), yv = min(max(y, 0), n1 - 1);
    if (ring_x && (x < 0 || x >= n0)) {
        if (fd.face_kind[0] & kFaceMirror) set = 1;
        else xv = n0 - 1 - xv;
    }
    if (ring_y && (y < 0 || y >= n1)) {
        if (fd.face_kind[2] & kFaceMirror) set = 2;
        else yv = n1 - 1 - yv;
    }
    const int32_t st2 = n0 * n1;
    const uint32_t vs = (uint32_t)(xv + n0 * yv);
    const bool f0 = xv == 0, f1 = xv == n0 - 1, f2 = NQ == 7 && yv == 0, f3 = NQ == 7 && yv == n1 - 1;
    const bool xyface = f0 || f1 || f2 || f3;

    constexpr uint32_t VB = sizeof(V);
    const uint32_t psB = (uint32_t)st2 * VB;
    const int64_t zsB = (int64_t)NQ * psB;
    const char* srcg = static_cast<const char*>(a.src) + fd.gpop * (int64_t)VB;
    char* dstf = static_cast<char*>(a.dst) + fd.pop * (int64_t)VB;
    const uint32_t* words = a.words + fd.words;
    const uint32_t vst = inner ? vs * VB : kNoStore;
    V cw0, cw1;
    store2(&cw0, make_double2(W0, 0.0));
    store2(&cw1, make_double2(W1, 0.0));
    auto ld = [&](Layer l, uint32_t off, uint32_t plane, const V& c) -> V {
        if constexpr (FIRST) {
            (void)l;
            (void)off;
            (void)plane;
            return c;
        } else {
            (void)c;
            return load_at(l, off, plane, (V*)nullptr);
        }
    };

    // byte offsets of the column (from the layer's plane 0 of the q-sample's
    // first field): its own plane 0 and, in LDS, the x and y pulls and plane 0
    // of its image across z
    uint32_t vo = 0;
    auto column_field = [&](bool image) -> int { return image ? fd.part[2] : set_field(set); };
    auto set_offsets = [&](bool image) {
        if constexpr (!FIRST) {
            const PairField& o = a.fields[column_field(image)];
            const int32_t rel = (int32_t)(o.pop - fd.gpop);
            auto pull = [&](bool face, int f, int d, int32_t wrap, int32_t nb) -> uint32_t {
                const int db = (d & 1) ? d + 1 : d - 1;
                const uint32_t e =
                    !face ? (uint32_t)(rel + d * st2) + vs + (uint32_t)nb
                    : (o.face_kind[f] & kFaceMirror)
                        ? (uint32_t)((int32_t)(o.face_pop[f] - fd.gpop) + db * st2) + vs
                        : (uint32_t)(rel + d * st2) + vs + (uint32_t)wrap;
                return e * VB;
            };
            vo = ((uint32_t)rel + vs) * VB;
            c_pull[t] = make_uint4(pull(f0, 0, 1, n0 - 1, -1), pull(f1, 1, 2, -(n0 - 1), 1),
                                   NQ == 7 ? pull(f2, 2, 3, (n1 - 1) * n0, -n0) : 0u,
                                   NQ == 7 ? pull(f3, 3, 4, -(n1 - 1) * n0, n0) : 0u);
            c_image[t] = ((uint32_t)(int32_t)(o.face_pop[4] - fd.gpop) + vs) * VB;
        }
    };
    // reaction factor of the column at step k and the row of its faces
    int fs = set;
    auto set_phase = [&](bool image) {
        const PairField& o = a.fields[column_field(image)];
        c_exy[0][t] = cmul(a.tab0[o.tab + xv], a.tab0[o.tab + n0 + yv]);
        fs = image ? 3 : set;
    };
    c_exy[1][t] = cmul(a.tab1[fd.tab + xv], a.tab1[fd.tab + n0 + yv]);
    // LDS slots of the x and y pulls at step k + 1: the neighbouring thread,
    // through a mirrored face its reflected direction
    // (two 16-bit slots to a register)
    uint32_t s12 = t * 0x10001u, s34 = t * 0x10001u;
    if (inner) {
        const bool mx = (fd.face_kind[0] & kFaceMirror) != 0, my = (fd.face_kind[2] & kFaceMirror) != 0;
        s12 = (uint32_t)(t - 1 + (mx && f0 ? NT : 0)) |
              (uint32_t)(t + 1 + (mx && f1 ? 0 : NT)) << 16;
        if constexpr (NQ == 7)
            s34 = (uint32_t)(t - bx + (my && f2 ? 3 * NT : 2 * NT)) |
                  (uint32_t)(t + bx + (my && f3 ? 2 * NT : 3 * NT)) << 16;
    }

    struct Loads {
        uint32_t word;
        V g[NQ];          // g[pz] is carried, not loaded
        V own[NQ - 1];    // own[pz - 1] is carried, not loaded
    };
    auto issue = [&](int32_t jv, Loads& L) {
        const Layer l = layer_at(srcg, jv * zsB);
        L.word = __builtin_amdgcn_raw_buffer_load_b32(layer_at(words, (int64_t)jv * st2 * 4), vs * 4u,
                                                      0, 0);
        const uint4 v = c_pull[FIRST ? 0 : t];
        // a plane's pull and its own population one after the other: they
        // share cache lines, which the first-level cache holds only briefly
        // (a layer of the tile takes twice its size)
        L.g[0] = ld(l, vo, 0, cw0);
        L.g[1] = ld(l, v.x, 0, cw1);
        L.own[1] = ld(l, vo, psB, cw1);
        L.g[2] = ld(l, v.y, 0, cw1);
        L.own[0] = ld(l, vo, 2 * psB, cw1);
        if constexpr (NQ == 7) {
            L.g[3] = ld(l, v.z, 0, cw1);
            L.own[3] = ld(l, vo, 3 * psB, cw1);
            L.g[4] = ld(l, v.w, 0, cw1);
            L.own[2] = ld(l, vo, 4 * psB, cw1);
        }
        L.own[pz] = ld(l, vo, pz * psB, cw1);
        if (jv < n2 - 1) L.g[pz + 1] = ld(l, vo, (uint32_t)zsB + (pz + 1) * psB, cw1);
        else if (mz) L.g[pz + 1] = ld(l, c_image[FIRST ? 0 : t], pz * psB, cw1);
        else L.g[pz + 1] = ld(layer_at(srcg, 0), vo, (pz + 1) * psB, cw1);
    };
    // carried along the column: the pz pull and the direction-pz own
    // population of the layer to compute
    V cz_g = cw1, cz_o = cw1;
    auto load_carried = [&](int32_t jv) {
        const Layer l = layer_at(srcg, jv * zsB);
        if (jv > 0) cz_g = ld(layer_at(srcg, (jv - 1) * zsB), vo, pz * psB, cw1);
        else if (mz) cz_g = ld(l, c_image[FIRST ? 0 : t], (pz + 1) * psB, cw1);
        else cz_g = ld(layer_at(srcg, (n2 - 1) * zsB), vo, pz * psB, cw1);
        cz_o = ld(l, vo, (pz + 1) * psB, cw1);
    };
    auto through_face = [&](double2 v, int row, int krow, int f) -> double2 {
        if (c_kind[krow * 6 + f] & kFaceConj) v.y = -v.y;
        return cmul(v, c_fac[row * 6 + f]);
    };
    auto faces = [&](double2 (&g)[NQ], int row, int krow, bool low, bool high) {
        if (xyface) {
            if (f0) g[1] = through_face(g[1], row, krow, 0);
            if (f1) g[2] = through_face(g[2], row, krow, 1);
            if constexpr (NQ == 7) {
                if (f2) g[3] = through_face(g[3], row, krow, 2);
                if (f3) g[4] = through_face(g[4], row, krow, 3);
            }
        }
        if (low) g[pz] = through_face(g[pz], row, krow, 4);
        if (high) g[pz + 1] = through_face(g[pz + 1], row, krow, 5);
    };
    auto membranes = [&](double2 (&g)[NQ], uint32_t word, auto own) {
        if (word >> 4) {
            const double* row = c_trans + (word & 0xfu) * 16;
#pragma unroll
            for (int d = 1; d < NQ; ++d) g[d] = half_link(g[d], own(d), row[link_code(word, d)]);
        }
    };

    double2 M0 = make_double2(0.0, 0.0), M1 = make_double2(0.0, 0.0);
    // the layer below at step k + 1: rest and z populations (its x and y
    // populations are read back from LDS), the pz pull into it, its word
    V h0 = cw0, h5 = cw1, h6 = cw1, c5 = cw1;
    uint32_t word_p = 0;
    Loads L;
    V hn[NQ];
    // layer j, whose loads are in L, to step k + 1; inside: a layer of the chunk
    auto update = [&](int32_t j, int32_t jv, bool inside) {
        V own[NQ - 1];
#pragma unroll
        for (int d = 1; d < NQ; ++d) own[d - 1] = d == pz ? cz_o : L.own[d - 1];
        double2 g[NQ];
#pragma unroll
        for (int d = 0; d < NQ; ++d) g[d] = ld2(d == pz ? &cz_g : &L.g[d]);
        faces(g, fs, fs, jv == 0, jv == n2 - 1);
        membranes(g, L.word, [&](int d) { return own[d - 1]; });
        const int p = (int)(L.word & 0xfu);
        const double2 e = cmul(c_exy[0][t], c_ez[(fs == 3 ? 0 : fs) * a.zr + (j - z0 + 1)]);
        const double2 M = react_collide<NQ>(g, e, c_dec[p], c_w[p]);
#pragma unroll
        for (int d = 0; d < NQ; ++d) store2(&hn[d], g[d]);
        cz_g = copied(L.own[pz]);
        cz_o = copied(L.g[pz + 1]);
        if (inside && inner) {
            M0.x += M.x;
            M0.y += M.y;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // layer jp to step k + 2; up: its pull from the layer above
    auto finish = [&](int32_t jp, V up) {
        const V* r = xch + (jp & 1) * NX * NT;
        double2 g[NQ];
        g[0] = ld2(&h0);
        g[1] = ld2(r + (s12 & 0xffffu));
        g[2] = ld2(r + (s12 >> 16));
        if constexpr (NQ == 7) {
            g[3] = ld2(r + (s34 & 0xffffu));
            g[4] = ld2(r + (s34 >> 16));
        }
        g[pz] = ld2(&c5);
        g[pz + 1] = ld2(&up);
        faces(g, 4, 0, jp == 0, jp == n2 - 1);
        membranes(g, word_p, [&](int d) -> V {
            const int od = (d & 1) ? d + 1 : d - 1;
            return od == pz ? h5 : od == pz + 1 ? h6 : r[(od - 1) * NT + t];
        });
        const int p = (int)(word_p & 0xfu);
        const double2 e = cmul(c_exy[1][t], c_ez[3 * a.zr + (jp - z0 + 1)]);
        const double2 M = react_collide<NQ>(g, e, c_dec[p], c_w[p]);
        if (inner) {
            M1.x += M.x;
            M1.y += M.y;
        }
        const Layer l = layer_at(dstf, jp * zsB, (uint32_t)zsB);
#pragma unroll
        for (int d = 0; d < NQ; ++d) store_at(l, vst, d * psB, g[d], (V*)nullptr);
    };
    __syncthreads();
    const bool low_img = mz && z0 == 0, top_img = mz && z1 == n2;
    uint32_t word = 0;
    auto exchange = [&](int32_t j) {
        if (active) {
            V* w = xch + (j & 1) * NX * NT + t;
#pragma unroll
            for (int d = 0; d < NX; ++d) w[d * NT] = hn[d + 1];
        }
        word = L.word;
    };
    auto keep = [&]() {
        h0 = hn[0];
        h5 = hn[pz];
        h6 = hn[pz + 1];
        word_p = word;
    };
    if (__ballot(active) != 0) {
        // the layer below the chunk and the chunk's first two
        const int32_t jb = layer_of(z0 - 1), ja = layer_of(z1);
        set_offsets(low_img);
        set_phase(low_img);
        issue(jb, L);
        load_carried(jb);
        update(z0 - 1, jb, false);
        c5 = pick(low_img, hn[pz + 1], hn[pz]);
        if (low_img) {
            set_offsets(false);
            set_phase(false);
        }
        if (z0 == 0) load_carried(0);
        issue(z0, L);
        update(z0, z0, true);
        exchange(z0);
        keep();
        if (z0 + 1 < z1) {
            issue(z0 + 1, L);
            lds_barrier();
            update(z0 + 1, z0 + 1, true);
            exchange(z0 + 1);
            // One layer of the walk: layer j to step k + 2, layer j + 2 to
            // step k + 1.  Loads and stores wait on one in-order counter: the
            // loads are issued before the stores, so that waiting for them
            // leaves the stores in flight.
#pragma nounroll
            for (int32_t j = z0; j + 2 < z1; ++j) {
                issue(j + 2, L);
                __builtin_amdgcn_sched_barrier(0);
                finish(j, hn[pz + 1]);
                c5 = h5;
                keep();
                __builtin_amdgcn_sched_barrier(0);
                lds_barrier();
                __builtin_amdgcn_sched_barrier(0);
                update(j + 2, j + 2, true);
                exchange(j + 2);
            }
            if (!top_img) issue(ja, L);
            finish(z1 - 2, hn[pz + 1]);
            c5 = h5;
            keep();
        } else if (!top_img) {
            issue(ja, L);
        }
        lds_barrier();
        // the layer above the chunk
        if (top_img) {
            set_offsets(true);
            set_phase(true);
            issue(ja, L);
        }
        if (z1 == n2) load_carried(ja);
        update(z1, ja, false);
        finish(z1 - 1, pick(top_img, hn[pz], hn[pz + 1]));
    } else {
        // a wave without columns keeps the barriers
        for (int32_t j = z0; j < z1; ++j) lds_barrier();
    }

    if (fd.q < 0) return;   // image fields do not enter the signal
    const double m0x = wave_sum(M0.x), m0y = wave_sum(M0.y);
    const double m1x = wave_sum(M1.x), m1y = wave_sum(M1.y);
    if ((t & 63) == 0) {
        c_red[0][t >> 6] = make_double2(m0x, m0y);
        c_red[1][t >> 6] = make_double2(m1x, m1y);
    }
    __syncthreads();
    if (t < 2) {
        double2 s = make_double2(0.0, 0.0);
        for (int i = 0; i < (int)blockDim.x / 64; ++i) {
            s.x += c_red[t][i].x;
            s.y += c_red[t][i].y;
        }
        a.partial[(size_t)(a.slot + t) * gridDim.x + fd.blk0 + b] = s;
    }
}

// Threads of a workgroup (one column each, the ring included) and wavefronts
// per SIMD that the registers of a column are held to.  D3Q7 in FP32: 127
// registers, four wavefronts, two workgroups of 512 to a compute unit (256
// threads, more of it ring, took 13 % longer on 256^3 x 12).
constexpr int kPairThreads7 = 512, kPairThreads5 = 320;

template <typename V, int NQ, int NT, int WPE>
static hipError_t launch_pair_t(const PairArgs& a, int32_t n_blocks, int32_t threads,
                                hipStream_t st) {
    const size_t lds = (size_t)(4 * a.zr + 30) * sizeof(double2);
    const dim3 g(n_blocks), t(threads);
    if (threads > NT || threads % 64) return hipErrorInvalidValue;
    if (a.first)
        hipLaunchKernelGGL((k_pair<V, NQ, NT, WPE, true>), g, t, lds, st, a);
    else
        hipLaunchKernelGGL((k_pair<V, NQ, NT, WPE, false>), g, t, lds, st, a);
    return hipGetLastError();
}

int32_t pair_max_threads(int nq) { return nq == 5 ? kPairThreads5 : kPairThreads7; }

hipError_t launch_pair(int prec, const PairArgs& a, int32_t n_blocks, int32_t threads,
                       hipStream_t st) {
    if (prec == 1)
        return a.nq == 5 ? launch_pair_t<float2, 5, kPairThreads5, 4>(a, n_blocks, threads, st)
                         : launch_pair_t<float2, 7, kPairThreads7, 4>(a, n_blocks, threads, st);
    return a.nq == 5 ? launch_pair_t<double2, 5, kPairThreads5, 4>(a, n_blocks, threads, st)
                     : launch_pair_t<double2, 7, kPairThreads7, 3>(a, n_blocks, threads, st);
}

}  // namespace btl
