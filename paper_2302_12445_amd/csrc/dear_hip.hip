// libdear: HIP kernels (gfx950) and context for DeAR's decoupled gradient aggregation.
//
// All three phases are HBM-bandwidth bound (about 0.2 flop per byte), so the kernels are
// plain streaming kernels: 16-byte vector accesses, one workgroup per tile of one
// layer/shard run, many independent loads in flight per lane, no matrix cores.
//
// Packing (copy into the fusion buffer, paper Sec. IV-A / V-A) is never materialised:
// a tile table maps every run of bucket positions to (layer, element range,
// owning shard, shard-buffer offset), and the reduce-scatter reads the per-layer tensors
// directly while the all-gather writes them directly.
//
// Alignment: layer tensors start 16-byte aligned, so 16-byte vectors counted from the
// tensor start are always aligned on the tensor side (for all P replicas alike).  Layers
// are packed densely in a bucket, so the matching shard-buffer addresses are only
// 4-byte aligned; those accesses are issued as 16-byte accesses with 4-byte alignment,
// which global memory instructions allow for dword-aligned addresses.
//
// Bit-exactness: fp32 adds in the ring order of the owning shard, one rounding per
// operation, no contraction (file compiled with -ffp-contract=off, and see the pragma).
#include <hip/hip_runtime.h>

#include <cstring>
#include <memory>
#include <new>
#include <numeric>
#include <type_traits>
#include <vector>

#include "dear_internal.h"

#pragma clang fp contract(off)

namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef f4 f4_dword_aligned __attribute__((aligned(4)));  // 16-byte access, 4-byte alignment

struct dear_ctx_impl {
    int32_t L = 0, B = 0, P = 0, g = 0;
    int device = 0;
    int32_t max_workgroups = 0;  // 0: one workgroup per work item
    int32_t wave_priority = 0;   // wave priority (0..3) of bounded-grid kernels
    int64_t row_len = 0;
    bool replicas_alike = true;  // almost all parts of an all-gather begin and end on 128-byte lines, alike in all replicas
    std::vector<int64_t> bucket_len, bucket_shard_len, bucket_shard_base;
    std::vector<int64_t> tile_begin;  // [B+1] range of bucket b's tiles in the tile table
    std::vector<int64_t> whole_begin;  // [B+1] how many of the tiles before bucket b are whole,
    std::vector<int64_t> long_begin;   // [B+1] how many lie in more than one part of the reduce-scatter,
    std::vector<int64_t> cut_begin;    // [B+1] and how many begin or end inside a vector of gradients
    std::vector<int64_t> layer_sizes;
    void *d_tables = nullptr;         // one allocation: the four tables below
    dear_tile *d_tiles = nullptr;
    struct layer_place *d_places = nullptr;  // [L]
    const void **d_grad = nullptr;    // [P*L] device pointers
    float **d_param = nullptr;        // [P*L] device pointers
};

// Where a layer lies in the shard buffers: element i is position e = offset + i of its bucket, slot
// e % shard_len of shard e / shard_len, whose slots start at shard_base of the worker's row.
struct layer_place {
    int64_t offset, shard_len, shard_base;
    double inv_shard_len;
};

// ------------------------------------------------------------------------------- kernels

// Launch-shape and cache-hint choices, fixed at build time (measured on MI355X; the
// defaults are the fastest found).  *_U = 16-byte vectors per lane; a tile of
// DEAR_TILE_ELEMS is shared by TILE_VECS / (U * DEAR_BLOCK) workgroups.
#ifndef DEAR_RS_NT_LOAD
#define DEAR_RS_NT_LOAD 1
#endif
#ifndef DEAR_RS_NT_STORE
#define DEAR_RS_NT_STORE 1
#endif
#ifndef DEAR_AG_NT_LOAD
#define DEAR_AG_NT_LOAD 0
#endif
#ifndef DEAR_AG_CHUNK_BYTES
#define DEAR_AG_CHUNK_BYTES (16 << 20)  // shard bytes whose P copies are written back to back
#endif
#ifndef DEAR_AG_NT_STORE
#define DEAR_AG_NT_STORE 1
#endif
#ifndef DEAR_UPD_U
#define DEAR_UPD_U 1
#endif
#ifndef DEAR_UPD_NT_LOAD
#define DEAR_UPD_NT_LOAD 1
#endif
#ifndef DEAR_UPD_NT_STORE
#define DEAR_UPD_NT_STORE 1
#endif

// Pointers read from the pointer tables are generic; every tensor lives in global
// memory, and saying so lets the compiler use global_load / global_store.
#define DEAR_GLOBAL __attribute__((address_space(1)))
#define DEAR_CONSTANT __attribute__((address_space(4)))  // tables, which no kernel writes: scalar loads
typedef const DEAR_GLOBAL u4 *global_u4_in;
typedef DEAR_GLOBAL f4 *global_f4_out;
typedef const DEAR_GLOBAL f4_dword_aligned *global_f4u_in;
typedef DEAR_GLOBAL f4_dword_aligned *global_f4u_out;

template <bool NT, class Ptr>
__device__ __forceinline__ auto load_vec(Ptr p)
{
    if (NT) return __builtin_nontemporal_load(p);
    return *p;
}

template <bool NT, class Ptr, class V>
__device__ __forceinline__ void store_vec(Ptr p, V v)
{
    if (NT)
        __builtin_nontemporal_store(v, p);
    else
        *p = v;
}

// 16-byte accesses to shard buffers, whose addresses are only 4-byte aligned.
template <bool NT>
__device__ __forceinline__ f4 load_f4_dword_aligned(const float *p)
{
    global_f4u_in q = (global_f4u_in)p;
    if (NT) return __builtin_nontemporal_load(q);
    return *q;
}

template <bool NT>
__device__ __forceinline__ void store_f4_dword_aligned(float *p, f4 v)
{
    global_f4u_out q = (global_f4u_out)p;
    if (NT)
        __builtin_nontemporal_store(v, q);
    else
        *q = v;
}

__device__ __forceinline__ int ring_worker(int start, int k, int P)
{
    int p = start + k;  // start < P and k < P, so one wrap suffices
    return p >= P ? p - P : p;
}

// One gradient element: its bits as they lie in memory, and their value.
template <bool BF16>
__device__ __forceinline__ uint32_t grad_bits(const void *base, int64_t i)
{
    if (BF16) return ((const DEAR_GLOBAL uint16_t *)base)[i];
    return ((const DEAR_GLOBAL uint32_t *)base)[i];
}

template <bool BF16>
__device__ __forceinline__ float grad_value(uint32_t bits)
{
    return __uint_as_float(BF16 ? bits << 16 : bits);
}

// The first and last 16-byte vector of a run [a, c) may be partial.  Lanes 0 .. VE-1 take an element each
// of the first and the next VE lanes of the last, if that vector is among [v_first, v_first + vecs); returns
// the lane's element, or -1.  (One lane that walks over its elements, and over the replicas for each, is a
// chain of up to (VE-1) * P loads, some 50 us at P = 8 with bf16: longer than a launch over a small bucket.
// us per iteration with such lanes -> with a lane per element: 2.9 M elements in 313 tensors P = 64 454 -> 369,
// 20 M elements in 604 tensors P = 7 bf16 234 -> 225, ResNet-50-shaped P = 8 367 -> 362.)
template <int VE>
__device__ __forceinline__ int64_t edge_element(int64_t a, int64_t c, int64_t v_first, int vecs)
{
    const int tid = threadIdx.x;
    const int64_t head = a / VE, tail = c / VE;
    const int64_t head_end = (a + VE - 1) / VE * VE < c ? (a + VE - 1) / VE * VE : c;
    if (tid < VE) {
        const int64_t e = head * VE + tid;
        if (head >= v_first && head < v_first + vecs && e >= a && e < head_end) return e;
    } else if (tid < 2 * VE) {
        const int64_t e = tail * VE + tid - VE;
        if (tail >= v_first && tail < v_first + vecs && e >= head_end && e < c) return e;
    }
    return -1;
}

// acc += the VE gradient elements held in one 16-byte vector (bf16 widens exactly).
template <bool BF16, int VE>
__device__ __forceinline__ void add_vector(float (&acc)[VE], const u4 r)
{
    if (BF16) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            acc[2 * j] = acc[2 * j] + __uint_as_float(r[j] << 16);
            acc[2 * j + 1] = acc[2 * j + 1] + __uint_as_float(r[j] & 0xffff0000u);
        }
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[j] = acc[j] + __uint_as_float(r[j]);
    }
}

// Launch width.  By default every work item (a part of a tile, a block of update vectors)
// gets a workgroup of its own: BOUNDED = false, the grid equals the item count and the
// hardware's in-order workgroup dispatch paces the memory streams.  A context may bound the
// grid (dear_ctx_set_max_workgroups): BOUNDED = true, each workgroup strides over the items.
// That is for running beside compute kernels on the same GPU: a few hundred resident
// workgroups with many loads in flight each disturb a GEMM's memory latency far less than
// a full grid.  `prio` (dear_ctx_set_wave_priority) raises the wave priority of such a
// kernel: its wavefronts then win instruction issue against an MFMA-saturated neighbour,
// which makes the aggregation faster and the neighbour slower.
template <bool BOUNDED, class Body>
__device__ __forceinline__ void for_each_item(unsigned n_items, int prio, Body body)
{
    if (!BOUNDED) {
        body(blockIdx.x);
    } else {
        if (prio == 1)
            __builtin_amdgcn_s_setprio(1);
        else if (prio == 2)
            __builtin_amdgcn_s_setprio(2);
        else if (prio == 3)
            __builtin_amdgcn_s_setprio(3);
        for (unsigned item = blockIdx.x; item < n_items; item += gridDim.x) body(item);
    }
}

// Orders LDS traffic among the lanes of ONE wavefront (each wavefront of the reduce-scatter
// owns its own staging area, so no other wavefront is involved): the hardware performs a
// wavefront's LDS operations in issue order, so all that is needed is that the compiler
// keeps the stores before and the loads after this point.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Where a reduce-scatter result goes: any of
//   RS_GBAR    gbar is stored to the gradient shard buffer;
//   RS_UPDATE  the SGD-momentum update of the slot is applied at once (v = mu*v + gbar; w = w - lr*v, the
//              same four separately rounded operations as shard_update_kernel) while gbar is in registers.
//              Without RS_GBAR gbar is never written, which saves its 4-byte write and 4-byte re-read per
//              element; with it only the re-read is saved;
//   RS_W_NEXT  the next launch reads w, and finds it in the 256 MB last-level cache (iteration_caches_w): w is stored
//              with the ordinary cache policy.
//   RS_GATHER  (with RS_UPDATE) the new w goes to every replica's layer tensor from the registers it was computed in: the
//              whole iteration in one launch, and no launch reads w again (iteration_gathers_at_once).
typedef int rs_mode;
constexpr rs_mode RS_GBAR = 1, RS_UPDATE = 2, RS_W_NEXT = 4, RS_GATHER = 8;

template <rs_mode MODE>
struct rs_sink {
    float *__restrict__ g;  // RS_GBAR: gradient shards
    float *__restrict__ w;  // RS_UPDATE: parameter shards
    float *__restrict__ v;  // RS_UPDATE: momentum shards
    float lr, mu;
    float *const *__restrict__ params;  // RS_GATHER: [P*L] layer tensors
};

__device__ __forceinline__ void sgd_momentum(float gbar, float &w, float &v, float lr, float mu)
{
    const float t1 = mu * v;
    v = t1 + gbar;
    const float t2 = lr * v;
    w = w - t2;
}

// One 16-byte piece of results at shard-buffer element index `idx` (4-byte aligned).  Callers
// that update pass the slot's w and v, loaded early so the loads overlap the gradient loads; returns the new w.
template <rs_mode MODE>
__device__ __forceinline__ f4 emit_piece(const rs_sink<MODE> &o, int64_t idx, f4 gbar, f4 w, f4 v)
{
    if (MODE & RS_GBAR) store_f4_dword_aligned<DEAR_RS_NT_STORE>(o.g + idx, gbar);
    if (MODE & RS_UPDATE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float wj = w[j], vj = v[j];
            sgd_momentum(gbar[j], wj, vj, o.lr, o.mu);
            w[j] = wj;
            v[j] = vj;
        }
        store_f4_dword_aligned<DEAR_RS_NT_STORE>(o.v + idx, v);
        store_f4_dword_aligned<DEAR_RS_NT_STORE && !(MODE & RS_W_NEXT)>(o.w + idx, w);
    }
    return w;
}

template <rs_mode MODE>
__device__ __forceinline__ float emit_elem(const rs_sink<MODE> &o, int64_t idx, float gbar)
{
    float w = 0.0f;
    if (MODE & RS_GBAR) o.g[idx] = gbar;
    if (MODE & RS_UPDATE) {
        float v = o.v[idx];
        w = o.w[idx];
        sgd_momentum(gbar, w, v, o.lr, o.mu);
        o.v[idx] = v;
        o.w[idx] = w;
    }
    return w;
}

// Body of the reduce-scatter for one workgroup's part of a tile.  ALL_FULL: the tile is a
// whole, aligned DEAR_TILE_ELEMS run, so no lane needs an edge check.  CH replicas are
// loaded per lane and vector before they are added; TAIL says P is not a multiple of CH.
template <bool BF16, int U, int CH, bool TAIL, bool ALL_FULL, rs_mode MODE>
__device__ __forceinline__ void reduce_scatter_tile(const dear_tile &t, int part,
                                                    const void *const *__restrict__ grad_tab, int L,
                                                    int P, float inv_P, const rs_sink<MODE> &o)
{
    constexpr int VE = BF16 ? 8 : 4;  // elements per 16-byte vector
    constexpr int PIECES = VE / 4;     // 16-byte result pieces per lane and vector
    // bf16, whole tile: a lane's 8 results are 32 bytes, so storing them directly would
    // leave each store instruction half dense (16 of every 32 bytes) and HBM would see
    // partial lines.  Each wavefront turns its 512 results through its own 2 KiB of LDS
    // so that both store instructions write 64 consecutive 16-byte pieces.
    constexpr bool TURN = BF16 && ALL_FULL;
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int64_t a = t.src_begin, c = a + t.count;
    const int64_t v_first = a / VE + (int64_t)part * (U * DEAR_BLOCK);
    if (!ALL_FULL && v_first * VE >= c) return;
    const int start = t.shard + 1 >= P ? 0 : t.shard + 1;

    int64_t vi[U];
    bool full[U];
    int64_t piece_idx[U][PIECES];  // shard-buffer element index of each result piece
    f4 w_new[U][PIECES];           // only RS_GATHER reads these three: new w of the pieces,
    float edge_w = 0.0f;           // of the lane's element of a partial vector,
    int64_t edge = -1;             // and that element, if the lane has one
    float acc[U][VE];
    f4 w_old[U][PIECES] = {}, v_old[U][PIECES] = {};  // only the updating sinks read them
#pragma unroll
    for (int u = 0; u < U; ++u) {
        vi[u] = v_first + u * DEAR_BLOCK + tid;
        const int64_t e0 = vi[u] * VE;
        full[u] = ALL_FULL || (e0 >= a && e0 + VE <= c);
#pragma unroll
        for (int j = 0; j < VE; ++j) acc[u][j] = -0.0f;
#pragma unroll
        for (int h = 0; h < PIECES; ++h) {
            if (TURN)  // piece h of the wave's 512-element run, lane-th 16 bytes of it
                piece_idx[u][h] = t.dst_begin + (v_first + u * DEAR_BLOCK + wave * 64) * VE - a + 256 * h + 4 * lane;
            else
                piece_idx[u][h] = t.dst_begin + (e0 - a) + 4 * h;
            if ((MODE & RS_UPDATE) && full[u]) {
                w_old[u][h] = load_f4_dword_aligned<DEAR_RS_NT_LOAD>(o.w + piece_idx[u][h]);
                v_old[u][h] = load_f4_dword_aligned<DEAR_RS_NT_LOAD>(o.v + piece_idx[u][h]);
            }
        }
    }

    for (int k0 = 0; k0 < P; k0 += CH) {
        global_u4_in src[CH];
#pragma unroll
        for (int kk = 0; kk < CH; ++kk) {
            const int k = (!TAIL || k0 + kk < P) ? k0 + kk : 0;
            src[kk] = (global_u4_in)grad_tab[(size_t)ring_worker(start, k, P) * L + t.layer];
        }
        u4 raw[U][CH];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (full[u]) {
#pragma unroll
                for (int kk = 0; kk < CH; ++kk)
                    if (!TAIL || k0 + kk < P) raw[u][kk] = load_vec<DEAR_RS_NT_LOAD>(src[kk] + vi[u]);
            }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (full[u]) {
#pragma unroll
                for (int kk = 0; kk < CH; ++kk)
                    if (!TAIL || k0 + kk < P) add_vector<BF16, VE>(acc[u], raw[u][kk]);
            }
    }

    if constexpr (TURN) {
        __shared__ float stage[DEAR_BLOCK / 64][64 * 8];
        float *sw = stage[wave];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            f4 lo, hi;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                lo[j] = acc[u][j] * inv_P;
                hi[j] = acc[u][4 + j] * inv_P;
            }
            *reinterpret_cast<f4 *>(sw + 8 * lane) = lo;
            *reinterpret_cast<f4 *>(sw + 8 * lane + 4) = hi;
            wave_lds_sync();
            const f4 o0 = *reinterpret_cast<const f4 *>(sw + 4 * lane);
            const f4 o1 = *reinterpret_cast<const f4 *>(sw + 256 + 4 * lane);
            wave_lds_sync();
            w_new[u][0] = emit_piece<MODE>(o, piece_idx[u][0], o0, w_old[u][0], v_old[u][0]);
            w_new[u][PIECES - 1] =
                emit_piece<MODE>(o, piece_idx[u][PIECES - 1], o1, w_old[u][PIECES - 1], v_old[u][PIECES - 1]);
        }
    } else {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (full[u]) {
#pragma unroll
                for (int h = 0; h < PIECES; ++h) {
                    f4 r;
#pragma unroll
                    for (int j = 0; j < 4; ++j) r[j] = acc[u][4 * h + j] * inv_P;
                    w_new[u][h] = emit_piece<MODE>(o, piece_idx[u][h], r, w_old[u][h], v_old[u][h]);
                }
            }
    }

    if (!ALL_FULL) {
        edge = edge_element<VE>(a, c, v_first, U * DEAR_BLOCK);  // CH replicas loaded together as above
        if (edge >= 0) {
            float s = -0.0f;
            for (int k0 = 0; k0 < P; k0 += CH) {
                float x[CH];
#pragma unroll
                for (int kk = 0; kk < CH; ++kk) {
                    const int k = (!TAIL || k0 + kk < P) ? k0 + kk : 0;
                    x[kk] = grad_value<BF16>(grad_bits<BF16>(grad_tab[(size_t)ring_worker(start, k, P) * L + t.layer], edge));
                }
#pragma unroll
                for (int kk = 0; kk < CH; ++kk)
                    if (!TAIL || k0 + kk < P) s = s + x[kk];
            }
            edge_w = emit_elem<MODE>(o, t.dst_begin + (edge - a), s * inv_P);
        }
    }

    if constexpr ((MODE & RS_GATHER) != 0) {
        const int64_t to_layer = a - t.dst_begin;  // from a slot's index to that of its element in the layer
#pragma unroll 4
        for (int q = 0; q < P; ++q) {
            DEAR_GLOBAL float *out = (DEAR_GLOBAL float *)o.params[(size_t)q * L + t.layer];
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (full[u]) {
#pragma unroll
                    for (int h = 0; h < PIECES; ++h)
                        store_vec<DEAR_AG_NT_STORE>((global_f4_out)(out + (to_layer + piece_idx[u][h])), w_new[u][h]);
                }
            if (!ALL_FULL && edge >= 0) out[edge] = edge_w;
        }
    }
}

// What comes behind the first D replicas: nothing (P = D: no loop in the code, whose lines a short launch waits for), as many
// again some times over, or that and a rest.
enum rest_of_replicas { REST_NONE, REST_BATCHES, REST_TAIL };

// Sum of all replicas in ring order from replica `start` on: one vector a lane, at `vec`, and with EDGE one element, at `elem`.
// D replicas are in flight: as soon as one has come and is added, the load of the one D further on takes its registers, with
// the pointers fetched another D ahead, so that a wavefront's loads never drain between batches.  Lanes without a
// vector or an element of their own are given an address in bounds, so that there is no branch between a load and its use
// but the uniform ones behind the loop.  P >= D, see rest_of_replicas.
template <bool BF16, int D, rest_of_replicas REST, bool VECTOR, bool EDGE, int VE>
__device__ __forceinline__ void sum_replicas(float (&acc)[VE], float &acc_edge, int64_t vec, int64_t elem,
                                             const void *const *__restrict__ grad_tab, int L, int P, int layer, int start)
{
    const void *src[D];
    u4 raw[D];
    uint32_t one[D];
    // the table's entries of this layer, by their distance in bytes from worker 0's (pointer_table_fits)
    const char DEAR_CONSTANT *const entries = (const char DEAR_CONSTANT *)(grad_tab + layer);
    const unsigned step = (unsigned)L * 8, end = (unsigned)P * step;
    unsigned at = (unsigned)start * step;
    auto pointers = [&]() {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            src[d] = *(const void *const DEAR_CONSTANT *)(entries + at);
            at += step;
            at = at == end ? 0 : at;
        }
    };
    auto load = [&](int d) {
        if (VECTOR) raw[d] = load_vec<DEAR_RS_NT_LOAD>((global_u4_in)src[d] + vec);
        if (EDGE) one[d] = grad_bits<BF16>(src[d], elem);
    };
    auto add = [&](int d) {
        if (VECTOR) add_vector<BF16, VE>(acc, raw[d]);
        if (EDGE) acc_edge = acc_edge + grad_value<BF16>(one[d]);
    };
    pointers();
#pragma unroll
    for (int d = 0; d < D; ++d)
        load(d);
    if (REST != REST_NONE && P > D) pointers();
    int k0 = D;
    for (; REST != REST_NONE && k0 + D <= P; k0 += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) {
            add(d);
            load(d);
            __builtin_amdgcn_sched_barrier(0);  // or all loads are put behind the last addition
        }
        pointers();  // behind the loads that use the last ones: a wait for one scalar load is a wait for all
    }
    const int left = P - k0;  // REST_TAIL: 1 .. D-1 replicas have not been asked for yet
#pragma unroll
    for (int d = 0; d < D; ++d) {
        add(d);
        if (REST == REST_TAIL && d < left) load(d);
    }
    if (REST == REST_TAIL) {
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (d < left) add(d);
    }
}

// A workgroup's part of a tile, DEAR_BLOCK vectors.  ALL_FULL: the tile is a whole, aligned DEAR_TILE_ELEMS run.  Otherwise
// the elements of the run's partial first and last vectors go along with the vectors, a lane each (edge_element): as a pass
// of their own behind the vectors they doubled the part's chain of loads.
template <bool BF16, int D, rest_of_replicas REST, bool ALL_FULL, rs_mode MODE>
__device__ __forceinline__ void reduce_scatter_part(const dear_tile &t, int part, const void *const *__restrict__ grad_tab,
                                                    int L, int P, float inv_P, const rs_sink<MODE> &o)
{
    constexpr int VE = BF16 ? 8 : 4, PIECES = VE / 4;
    constexpr bool TURN = BF16 && ALL_FULL;  // results go through LDS, see reduce_scatter_tile
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int64_t a = t.src_begin, c = a + t.count;
    const int64_t v_first = a / VE + (int64_t)part * DEAR_BLOCK, v_wave = v_first + wave * 64;
    if (!ALL_FULL && v_first * VE >= c) return;
    if (!ALL_FULL && wave > 0 && v_wave * VE >= c) return;  // the first wavefront has the partial vectors
    const int start = t.shard + 1 >= P ? 0 : t.shard + 1;
    const int64_t v_whole = (a + VE - 1) / VE;  // the run's first whole vector, if it has one
    const bool vectors = ALL_FULL || (v_whole + 1) * VE <= c;

    const int64_t edge = ALL_FULL ? -1 : edge_element<VE>(a, c, v_first, DEAR_BLOCK);
    float acc[VE], acc_edge = -0.0f;
#pragma unroll
    for (int j = 0; j < VE; ++j) acc[j] = -0.0f;
    if (vectors) {
        int64_t vec = v_wave + lane;
        const bool full = ALL_FULL || (vec * VE >= a && vec * VE + VE <= c);
        if (!full) vec = v_whole;
        int64_t piece_idx[PIECES];  // shard-buffer element index of each 16-byte piece of results
        f4 w_old[PIECES], v_old[PIECES], r[PIECES];
#pragma unroll
        for (int h = 0; h < PIECES; ++h) {
            piece_idx[h] = t.dst_begin - a + (TURN ? v_wave * VE + 256 * h + 4 * lane : vec * VE + 4 * h);
            if (MODE & RS_UPDATE) {
                w_old[h] = load_f4_dword_aligned<DEAR_RS_NT_LOAD>(o.w + piece_idx[h]);
                v_old[h] = load_f4_dword_aligned<DEAR_RS_NT_LOAD>(o.v + piece_idx[h]);
            }
        }
        sum_replicas<BF16, D, REST, true, !ALL_FULL>(acc, acc_edge, vec, edge >= 0 ? edge : a, grad_tab, L, P, t.layer, start);
#pragma unroll
        for (int h = 0; h < PIECES; ++h)
#pragma unroll
            for (int j = 0; j < 4; ++j) r[h][j] = acc[4 * h + j] * inv_P;
        if constexpr (TURN) {
            __shared__ float stage[DEAR_BLOCK / 64][64 * 8];
            float *sw = stage[wave];
            *reinterpret_cast<f4 *>(sw + 8 * lane) = r[0];
            *reinterpret_cast<f4 *>(sw + 8 * lane + 4) = r[PIECES - 1];
            wave_lds_sync();
            r[0] = *reinterpret_cast<const f4 *>(sw + 4 * lane);
            r[PIECES - 1] = *reinterpret_cast<const f4 *>(sw + 256 + 4 * lane);
            wave_lds_sync();
        }
        if (full)
#pragma unroll
            for (int h = 0; h < PIECES; ++h) emit_piece<MODE>(o, piece_idx[h], r[h], w_old[h], v_old[h]);
    } else {
        sum_replicas<BF16, D, REST, false, true>(acc, acc_edge, 0, edge >= 0 ? edge : a, grad_tab, L, P, t.layer, start);
    }
    if (edge >= 0) emit_elem<MODE>(o, t.dst_begin + (edge - a), acc_edge * inv_P);
}

// Reduce-scatter (paper Sec. III-A; Eq. 2 for the 1/P), one part of a tile a workgroup.
// Summation starts at worker s+1 and ends with worker s, the order in which the ring
// delivers the partial sums of chunk s to its owner.  The accumulator starts as -0.0f,
// the additive identity that keeps the first addend's bits (including a -0.0f).
// Bound by HBM: P streams read once.  With batches of replicas waited for together (the kernel below) a workgroup's loads drained
// before every next batch, and neighbouring tiles went to different XCDs.  us, that kernel / this one, one launch over all buckets
// (several sets of buffers in turn): BERT-Large-shaped bf16 P = 8 1190 / 1052 (5.7 / 6.4 TB/s of a plain read's 7.0), with update
// 1848 / 1743, ResNet-50-shaped fp32 P = 64 1099 / 1073, with update 1226 / 1153, P = 8 149 / 146 and 200 / 200; a launch per bucket:
// BERT-Large-shaped 1137 / 1094 and 1825 / 1772, ResNet-50-shaped P = 64 1120 / 1067 and 1207 / 1120, P = 8 157 / 157, with update the
// kernel below, 211.  reduce_scatter_shape_of says which form goes when.
template <bool BF16, int D, rest_of_replicas REST, bool TILES, rs_mode MODE>
__global__ __launch_bounds__(DEAR_BLOCK) void reduce_scatter_kernel(
    const dear_tile *__restrict__ tiles, const void *const *__restrict__ grad_tab, int L, int P,
    float inv_P, const rs_sink<MODE> o, unsigned n_items, unsigned run)
{
    constexpr int SPLIT = DEAR_TILE_ELEMS / ((BF16 ? 8 : 4) * DEAR_BLOCK), STEP = TILES ? 1 : SPLIT;
    const unsigned item = item_in_rows(blockIdx.x, run, n_items);
    const dear_tile t = tiles[item / STEP];
    const int first = item % STEP;
    if (__builtin_expect(t.layer >= 0 && t.count == DEAR_TILE_ELEMS, 1)) {  // first, where the code's lines come in order
#pragma unroll 1
        for (int part = first; part < SPLIT; part += STEP)
            reduce_scatter_part<BF16, D, REST, true, MODE>(t, part, grad_tab, L, P, inv_P, o);
    } else if (t.layer >= 0) {
#pragma unroll 1
        for (int part = first; part < SPLIT; part += STEP)
            reduce_scatter_part<BF16, D, REST, false, MODE>(t, part, grad_tab, L, P, inv_P, o);
    } else {  // padding slots: gbar = +0
        for (int i = first * DEAR_BLOCK + threadIdx.x; i < t.count; i += STEP * DEAR_BLOCK)
            emit_elem<MODE>(o, t.dst_begin + i, 0.0f);
    }
}

// The same in bounded grids, with the all-gather in the same launch (RS_GATHER), for what reduce_scatter_kernel cannot count, and
// where reduce_scatter_shape_of finds it faster.  SPLIT workgroups share a tile.  Replicas come in batches of CH here, waited for
// together: beside GEMMs, and with the writes of all replicas to follow, that is the better form (BERT-Large-shaped schedule, bf16 in
// bounded grids, ms: this one 32.2, loads that never drain 36.1).
template <bool BF16, int U, int CH, bool TAIL, bool BOUNDED, rs_mode MODE>
__global__ __launch_bounds__(DEAR_BLOCK) void reduce_scatter_batch_kernel(
    const dear_tile *__restrict__ tiles, const void *const *__restrict__ grad_tab, int L, int P,
    float inv_P, const rs_sink<MODE> o, unsigned n_items, int prio)
{
    constexpr int SPLIT = DEAR_TILE_ELEMS / ((BF16 ? 8 : 4) * DEAR_BLOCK * U);
    static_assert(SPLIT >= 1 && (SPLIT & (SPLIT - 1)) == 0, "U must divide the tile");
    for_each_item<BOUNDED>(n_items, prio, [&](unsigned item) {
        const dear_tile t = tiles[item / SPLIT];
        const int part = item % SPLIT;
        if (t.layer < 0) {  // padding slots: gbar = +0
            for (int i = part * DEAR_BLOCK + threadIdx.x; i < t.count; i += SPLIT * DEAR_BLOCK)
                emit_elem<MODE>(o, t.dst_begin + i, 0.0f);
        } else if (t.count == DEAR_TILE_ELEMS) {
            reduce_scatter_tile<BF16, U, CH, TAIL, true, MODE>(t, part, grad_tab, L, P, inv_P, o);
        } else {
            reduce_scatter_tile<BF16, U, CH, TAIL, false, MODE>(t, part, grad_tab, L, P, inv_P, o);
        }
    });
}

// SGD with momentum on contiguous shard slots (paper Eq. 1-2): v = mu*v + g; w = w - lr*v.
// An item is a block of a row (worker); each row segment is `vecs` 16-byte vectors long.  Bound by HBM, three streams read and
// two of them written; long launches over all buckets give each XCD items in a row (shard_update_run): 336 M elements 1117 -> 1068 us
// (6.0 -> 6.3 TB/s of a copy's 6.7), 110 M 377 -> 350, 32 M 106.6 -> 100.2.
constexpr int UPD_U = DEAR_UPD_U;      // vectors per lane, one workgroup per item
constexpr int UPD_U_BOUNDED = 4;       // bounded grid: more loads in flight per lane
template <int U, bool BOUNDED>
__global__ __launch_bounds__(DEAR_BLOCK) void shard_update_kernel(
    const float *__restrict__ g, float *__restrict__ w, float *__restrict__ v, int64_t row_stride,
    int64_t base, int64_t vecs, float lr, float mu, unsigned blocks_per_row, unsigned n_items, int prio, unsigned run)
{
    for_each_item<BOUNDED>(n_items, prio, [&](unsigned index) {
        const unsigned item = BOUNDED ? index : item_in_rows(index, run, n_items);
        const unsigned row = item / blocks_per_row, bx = item - row * blocks_per_row;
        const int64_t off = (int64_t)row * row_stride + base;
        const f4 *__restrict__ g4 = reinterpret_cast<const f4 *>(g + off);
        f4 *__restrict__ w4 = reinterpret_cast<f4 *>(w + off);
        f4 *__restrict__ v4 = reinterpret_cast<f4 *>(v + off);
        const int64_t first = (int64_t)bx * (U * DEAR_BLOCK) + threadIdx.x;
        f4 gg[U], ww[U], vv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = first + u * DEAR_BLOCK;
            if (i < vecs) {
                gg[u] = load_vec<DEAR_UPD_NT_LOAD>(g4 + i);
                ww[u] = load_vec<DEAR_UPD_NT_LOAD>(w4 + i);
                vv[u] = load_vec<DEAR_UPD_NT_LOAD>(v4 + i);
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t i = first + u * DEAR_BLOCK;
            if (i < vecs) {
                f4 nv, nw;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float t1 = mu * vv[u][j];
                    nv[j] = t1 + gg[u][j];
                    const float t2 = lr * nv[j];
                    nw[j] = ww[u][j] - t2;
                }
                store_vec<DEAR_UPD_NT_STORE>(v4 + i, nv);
                store_vec<DEAR_UPD_NT_STORE>(w4 + i, nw);
            }
        }
    });
}

// All-gather with the copy-back to the layer tensors folded in (paper Sec. III-A, IV-A).
//
// One workgroup copies one part of one tile to ONE replica.  Workgroups are ordered
// (chunk, replica, part): the hardware starts workgroups in index order, so at any moment
// the chip writes a long sequential run of one or two replicas instead of P interleaved
// streams, which HBM sustains markedly better; the chunk's shard values
// (DEAR_AG_CHUNK_BYTES: 16 MiB, i.e. 2 MiB in each XCD's 4 MiB L2, since a part is always read
// by the same XCD) are re-read for replicas 1..P-1 from L2, not HBM.
//
// A workgroup lives for about 1.3 us at full rate and moves 4 KiB, so what bounds the kernel beside HBM is
// the serial chain in front of its one load: kernel arguments, item decoding, tile, data.  The decoding
// therefore divides by multiplication (see divide), and the tensor's address is fetched behind the data.
// Measured with everything else equal, all-gather of P fp32 replicas, GB/s before -> after: BERT-Large-shaped
// P = 8 6307 -> 6515, BERT-Base-shaped P = 16 6341 -> 6523, ResNet-50-shaped P = 8 6535 -> 6618, 604 ragged
// tensors P = 7 6387 -> 7042.  Fewer resident workgroups lose here (they cost in-flight loads, 4 KiB each).
// Where a workgroup's stores begin decides how many cache lines are written in two halves, by two
// workgroups on different XCDs, and HBM takes halves of lines badly (fp32 replicas whose tensors start on
// 16-byte boundaries only: 5300 GB/s instead of 6800).  A run is therefore not cut at multiples of the tile of
// the layer's own index but where the replica's addresses are multiples of 128 bytes: every cut moves down by
// `shift` elements, the distance of the tensor's start from a line.  The run's first tile begins, and its last
// tile ends, where the run does.  us per iteration: 30 M elements in 60 such tensors P = 8 468 -> 441, P = 16 850
// -> 787, 20 M in 604 P = 7 bf16 225 -> 217, ResNet-50-shaped P = 64 2432 -> 2348.
template <bool INNER>
__device__ __forceinline__ void all_gather_tile(const dear_tile &t, int part, int shift, bool first, bool last,
                                                float *const DEAR_CONSTANT *out_entry, const float *__restrict__ src)
{
    // positions are counted from the tile's first element, so that they fit 32 bits; `low` says how the
    // element lies in its 16-byte vector and 128-byte line
    constexpr int VE = 4, LINE = 32, PART = VE * DEAR_BLOCK;
    const int tid = threadIdx.x;
    const int low = (int)(t.src_begin & (LINE - 1));
    const int lo = INNER || !first ? -shift : 0, hi = INNER || !last ? t.count - shift : t.count;
    const int begin = (INNER ? lo : lo - ((low + lo + shift) & (LINE - 1))) + part * PART;
    if (!INNER && begin >= hi) return;
    const int i = begin + VE * tid;
    f4 val;
    if (INNER) {
        val = load_f4_dword_aligned<DEAR_AG_NT_LOAD>(src + i);
        // the tensor's address is wanted only by the stores: its load rides behind the data's
        __builtin_amdgcn_sched_barrier(0);
        DEAR_GLOBAL float *out = (DEAR_GLOBAL float *)*out_entry + t.src_begin;
        store_vec<DEAR_AG_NT_STORE>((global_f4_out)(out + i), val);
        return;
    }
    DEAR_GLOBAL float *out = (DEAR_GLOBAL float *)*out_entry + t.src_begin;
    // partial vectors at the run's ends: lanes 0-3 take an element each of the first, lanes 4-7 of the last
    const int head = lo - ((low + lo) & (VE - 1)), tail = hi - ((low + hi) & (VE - 1));
    const int head_end = head < lo ? (head + VE < hi ? head + VE : hi) : lo;
    // a run's end can lie up to a line behind the tile's four parts: the last part reaches that far
    const int end = begin + PART + (part == AG_SPLIT - 1 ? LINE : 0);
    if (i >= lo && i + VE <= hi) store_vec<DEAR_AG_NT_STORE>((global_f4_out)(out + i), load_f4_dword_aligned<DEAR_AG_NT_LOAD>(src + i));
    if (end > begin + PART && tid < LINE / VE && i + PART + VE <= hi)
        store_vec<DEAR_AG_NT_STORE>((global_f4_out)(out + i + PART), load_f4_dword_aligned<DEAR_AG_NT_LOAD>(src + i + PART));
    if (tid < 2 * VE) {
        const int at = tid < VE ? head : tail, e = at + (tid & (VE - 1));
        if (at >= begin && at < end && (tid < VE ? e >= lo && e < head_end : e >= head_end && e < hi)) out[e] = src[e];
    }
}

// A part of a tile that is not whole, in a run whose cuts stay at multiples of the tile: short runs, and the ends
// of runs of tensors that start on lines.  Thousands of short tensors make a launch of mostly such parts, some of
// them empty, and what bounds it is the number of instructions in front of a part's load: the form above
// took 69 us for 3000 tensors of 512 elements at P = 8 where this one takes 53, 220 / 171 for 20000 of 300 at P = 4,
// 182 / 145 for 4000 of 701 at P = 16.  Elements of a partial vector go one after another in that vector's lane
// for the same reason (a lane for each: 56, 179, 156).
__device__ __forceinline__ void all_gather_short_tile(const dear_tile &t, int part, float *out_base,
                                                      const float *__restrict__ src)
{
    constexpr int VE = 4, PART = VE * DEAR_BLOCK;
    const int tid = threadIdx.x;
    const int mis = (int)t.src_begin & (VE - 1), begin = part * PART - mis;
    if (begin >= t.count) return;
    DEAR_GLOBAL float *out = (DEAR_GLOBAL float *)out_base + t.src_begin;
    const int i = begin + VE * tid;
    if (i >= 0 && i + VE <= t.count)
        store_vec<DEAR_AG_NT_STORE>((global_f4_out)(out + i), load_f4_dword_aligned<DEAR_AG_NT_LOAD>(src + i));
    else if (i < t.count)
        for (int j = 0; j < VE; ++j)
            if (i + j >= 0 && i + j < t.count) out[i + j] = src[i + j];
}

// Quotient and remainder of n < 2^31 by a divisor d whose inv_d = floor((2^32 - 1) / d) the host supplies:
// n * inv_d / 2^32 is above n / d - 1, so the estimate is at most one too small.  A division proper is a
// long serial chain of scalar and vector instructions at the head of every workgroup.
__device__ __forceinline__ unsigned divide(unsigned n, unsigned d, unsigned inv_d, unsigned &rem)
{
    unsigned q = __umulhi(n, inv_d);
    rem = n - q * d;
    if (rem >= d) {
        rem -= d;
        ++q;
    }
    return q;
}

// n_parts = tiles * AG_SPLIT; replicas p_first .. p_first+n_p-1 receive.  inv_n_p, inv_len: reciprocals (see divide)
// of n_p and of len, the number of workgroups per replica in the short last chunk.
// Workgroups go to the eight XCDs in turn, and a part of a chunk belongs on one XCD for all replicas, whose L2 then
// holds the shard values: len is a multiple of 8 (workgroups behind the last part have nothing to do).  Right behind a short
// reduce-scatter + update the values are still in the L2 of the XCD that wrote them, so they are read there: `run` is
// the logarithm of the number of parts that one workgroup of that kernel had (fp32 0; bf16 in half tiles 1; all_gather_run).
// One launch of each, us per iteration without gbar, 1 M elements (an odd number of tiles) len as it falls / rounded:
// fp32 P = 4 13.7 / 11.5, P = 8 18.3 / 16.1, P = 16 29.6 / 27.6; 8 M fp32 P = 8 108.6 / 103.1, P = 16 195 / 187.  bf16, run 0 / 1:
// P = 4 1 M 12.1 / 10.7, 2 M 19.1 / 17.2, P = 8 1 M 16.1 / 14.7, 2 M 26.4 / 24.5, 3 M 36.0 / 34.6, P = 16 2 M 40.8 / 39.0;
// beyond, the values have left L2, and writes in this order cost: P = 8 10 M 100.9 / 101.6, P = 16 6 M 109 / 111, 20 M 355 / 368.
// EIGHTHS: in long launches every XCD takes an eighth of the chunk instead (all_gather_in_eighths).
template <unsigned RUN, bool EIGHTHS>
__global__ __launch_bounds__(DEAR_BLOCK) void all_gather_kernel(
    const dear_tile *__restrict__ tiles, float *const *__restrict__ param_tab, int L, int p_first,
    unsigned n_p, const float *__restrict__ shard_param, unsigned n_parts, unsigned inv_n_p, unsigned len,
    unsigned inv_len)
{
    static_assert((AG_SPLIT & (AG_SPLIT - 1)) == 0, "a part's tile is found by a shift");
    constexpr unsigned CHUNK = DEAR_AG_CHUNK_BYTES / (16 * DEAR_BLOCK);  // parts per chunk
    static_assert((CHUNK & (CHUNK - 1)) == 0, "whole chunks are told apart by a shift");
    const unsigned whole = n_parts / CHUNK;
    // item -> (chunk, replica, part within chunk)
    unsigned q, chunk = divide(blockIdx.x / CHUNK, n_p, inv_n_p, q), r = blockIdx.x % CHUNK;
    if (chunk >= whole) {
        chunk = whole;
        q = divide(blockIdx.x - whole * CHUNK * n_p, len, inv_len, r);
    }
    const unsigned id =
        chunk * CHUNK + (EIGHTHS ? all_gather_part_of_eighth(r, chunk < whole ? CHUNK : len) : all_gather_part(r, RUN));
    const dear_tile t = tiles[id / AG_SPLIT];
    const int part = id % AG_SPLIT;
    if (t.layer < 0 || id >= n_parts) return;  // behind the last part: a tile beyond the launch's, or the table's room
    const float *__restrict__ src = shard_param + t.dst_begin;
    float *const DEAR_CONSTANT *out =
        (float *const DEAR_CONSTANT *)param_tab + ((size_t)((unsigned)p_first + q) * (unsigned)L + (unsigned)t.layer);
    if (t.bucket == 0 && t.count == DEAR_TILE_ELEMS) {  // inside a run of tensors that start on lines
        all_gather_tile<true>(t, part, 0, false, false, out, src);
        return;
    }
    if (t.bucket <= (TILE_FIRST | TILE_LAST)) {
        if (t.count == DEAR_TILE_ELEMS)
            all_gather_tile<true>(t, part, 0, false, false, out, src);
        else
            all_gather_short_tile(t, part, *out, src);
        return;
    }
    const bool first = t.bucket & TILE_FIRST, last = t.bucket & TILE_LAST;
    const int shift = t.bucket & TILE_OWN_SHIFT ? line_shift((uintptr_t)*out) : t.bucket >> TILE_SHIFT_BIT;
    if (t.count == DEAR_TILE_ELEMS && (shift == 0 || !(first || last)))
        all_gather_tile<true>(t, part, shift, first, last, out, src);
    else
        all_gather_tile<false>(t, part, shift, first, last, out, src);
}

// Bounded-grid form of the all-gather: one item is a whole tile, read once and stored to all
// receiving replicas by the same workgroup.  Beside a GEMM the grid is too narrow to be
// bandwidth-bound, so what counts is bytes in flight per workgroup (4 loads, then 4 stores
// per replica), not the replica-sequential order of the full-grid kernel.
template <bool ALL_FULL>
__device__ __forceinline__ void all_gather_tile_all_replicas(const dear_tile &t,
                                                             float *const *__restrict__ param_tab, int L,
                                                             int p_first, int n_p,
                                                             const float *__restrict__ src)
{
    constexpr int VE = 4, U = DEAR_TILE_ELEMS / (VE * DEAR_BLOCK);
    const int tid = threadIdx.x;
    const int64_t a = t.src_begin, c = a + t.count;
    const int64_t v_first = a / VE;
    int64_t vi[U];
    bool full[U];
    f4 val[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        vi[u] = v_first + u * DEAR_BLOCK + tid;
        const int64_t e0 = vi[u] * VE;
        full[u] = ALL_FULL || (e0 >= a && e0 + VE <= c);
        if (full[u]) val[u] = load_f4_dword_aligned<DEAR_AG_NT_LOAD>(src + (e0 - a));
    }
    const int64_t e = ALL_FULL ? -1 : edge_element<VE>(a, c, v_first, U * DEAR_BLOCK);
    const float edge = e >= 0 ? src[e - a] : 0.0f;
    for (int q = 0; q < n_p; ++q) {
        DEAR_GLOBAL float *out = (DEAR_GLOBAL float *)param_tab[(size_t)(p_first + q) * L + t.layer];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (full[u]) store_vec<DEAR_AG_NT_STORE>((global_f4_out)out + vi[u], val[u]);
        if (e >= 0) out[e] = edge;
    }
}

__global__ __launch_bounds__(DEAR_BLOCK) void all_gather_bounded_kernel(
    const dear_tile *__restrict__ tiles, float *const *__restrict__ param_tab, int L, int p_first,
    int n_p, const float *__restrict__ shard_param, unsigned n_tiles, int prio)
{
    for_each_item<true>(n_tiles, prio, [&](unsigned item) {
        const dear_tile t = tiles[item];
        if (t.layer < 0) return;
        const float *__restrict__ src = shard_param + t.dst_begin;
        if (t.count == DEAR_TILE_ELEMS)
            all_gather_tile_all_replicas<true>(t, param_tab, L, p_first, n_p, src);
        else
            all_gather_tile_all_replicas<false>(t, param_tab, L, p_first, n_p, src);
    });
}

// Update and all-gather of a bucket in one kernel: a workgroup takes one tile (U = 4; a quarter with U = 1), applies the
// SGD-momentum update to the tile's slots (the same four separately rounded operations as
// shard_update_kernel), stores the new w and v to the shard buffers and the new w to all
// receiving replicas' layer tensors.  The updated value has to reach every replica from the
// workgroup that computed it, so the stores go to all replicas at once (P interleaved write
// streams) instead of replica by replica as in all_gather_kernel: for few replicas, short
// launches and bounded grids.
template <int U, bool ALL_FULL>
__device__ __forceinline__ void update_gather_tile(const dear_tile &t, int part, float *const *__restrict__ param_tab, int L,
                                                   int P, const float *__restrict__ g, float *__restrict__ w,
                                                   float *__restrict__ v, float lr, float mu)
{
    constexpr int VE = 4;
    const int tid = threadIdx.x;
    const int64_t a = t.src_begin, c = a + t.count;
    const int64_t v_first = a / VE + part * (U * DEAR_BLOCK);
    if (!ALL_FULL && v_first * VE >= c) return;
    int64_t vi[U];
    bool full[U];
    f4 gg[U], ww[U], vv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        vi[u] = v_first + u * DEAR_BLOCK + tid;
        const int64_t e0 = vi[u] * VE;
        full[u] = ALL_FULL || (e0 >= a && e0 + VE <= c);
        if (full[u]) {
            const int64_t slot = t.dst_begin + (e0 - a);
            gg[u] = load_f4_dword_aligned<DEAR_UPD_NT_LOAD>(g + slot);
            ww[u] = load_f4_dword_aligned<DEAR_UPD_NT_LOAD>(w + slot);
            vv[u] = load_f4_dword_aligned<DEAR_UPD_NT_LOAD>(v + slot);
        }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t e0 = vi[u] * VE;
        if (full[u]) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float wj = ww[u][j], vj = vv[u][j];
                sgd_momentum(gg[u][j], wj, vj, lr, mu);
                ww[u][j] = wj;
                vv[u][j] = vj;
            }
            const int64_t slot = t.dst_begin + (e0 - a);
            store_f4_dword_aligned<DEAR_UPD_NT_STORE>(v + slot, vv[u]);
            store_f4_dword_aligned<DEAR_UPD_NT_STORE>(w + slot, ww[u]);
        }
    }
    const int64_t e = ALL_FULL ? -1 : edge_element<VE>(a, c, v_first, U * DEAR_BLOCK);
    float edge = 0.0f;
    if (e >= 0) {
        const int64_t slot = t.dst_begin + (e - a);
        float vj = v[slot];
        edge = w[slot];
        sgd_momentum(g[slot], edge, vj, lr, mu);
        v[slot] = vj;
        w[slot] = edge;
    }
    for (int q = 0; q < P; ++q) {
        DEAR_GLOBAL float *out = (DEAR_GLOBAL float *)param_tab[(size_t)q * L + t.layer];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (full[u]) store_vec<DEAR_AG_NT_STORE>((global_f4_out)out + vi[u], ww[u]);
        if (e >= 0) out[e] = edge;
    }
}

template <int U, bool BOUNDED>
__global__ __launch_bounds__(DEAR_BLOCK) void update_all_gather_kernel(
    const dear_tile *__restrict__ tiles, float *const *__restrict__ param_tab, int L, int P,
    const float *__restrict__ g, float *__restrict__ w, float *__restrict__ v, float lr, float mu,
    unsigned n_items, int prio)
{
    constexpr int SPLIT = DEAR_TILE_ELEMS / (4 * DEAR_BLOCK * U);
    for_each_item<BOUNDED>(n_items, prio, [&](unsigned item) {
        const dear_tile t = tiles[item / SPLIT];
        const int part = item % SPLIT;
        if (t.layer < 0) {  // padding slots are updated like any other (their averaged gradient is +0)
            for (int i = part * DEAR_BLOCK + threadIdx.x; i < t.count; i += SPLIT * DEAR_BLOCK) {
                const int64_t slot = t.dst_begin + i;
                float wj = w[slot], vj = v[slot];
                sgd_momentum(g[slot], wj, vj, lr, mu);
                v[slot] = vj;
                w[slot] = wj;
            }
        } else if (t.count == DEAR_TILE_ELEMS) {
            update_gather_tile<U, true>(t, part, param_tab, L, P, g, w, v, lr, mu);
        } else {
            update_gather_tile<U, false>(t, part, param_tab, L, P, g, w, v, lr, mu);
        }
    });
}

// The two copies below take a quarter of a tile a workgroup, one 16-byte vector a lane: short workgroups in dispatch order, as
// in the all-gather.  BERT-Base-shaped at P = 8 (881 MB moved), us, whole tiles / halves / quarters: scatter 155 / 149 / 136,
// reshard 154 / 143 / 136 (6.5 TB/s, a plain copy reaches 6.65); 20 M ragged elements P = 7 31.0 / 29.5 / 28.7 and 32.0 / 30.0 / 30.0.
// Fewer resident workgroups cost: four per CU 139 and 153.
constexpr int COPY_PART = 4 * DEAR_BLOCK, COPY_SPLIT = DEAR_TILE_ELEMS / COPY_PART;

// Inverse of the all-gather for one worker: layer tensors -> owned shard slots.
__global__ __launch_bounds__(DEAR_BLOCK) void scatter_params_kernel(
    const dear_tile *__restrict__ tiles, float *const *__restrict__ param_tab, int L, int worker,
    float *__restrict__ shard_param)
{
    constexpr int VE = 4;
    const dear_tile t = tiles[blockIdx.x / COPY_SPLIT];
    const int tid = threadIdx.x, part = blockIdx.x % COPY_SPLIT;
    float *__restrict__ dst = shard_param + t.dst_begin;
    if (t.layer < 0) {
        for (int i = part * DEAR_BLOCK + tid; i < t.count; i += COPY_SPLIT * DEAR_BLOCK) dst[i] = 0.0f;
        return;
    }
    const int64_t a = t.src_begin, c = a + t.count;
    const int64_t v_first = a / VE + part * DEAR_BLOCK, e0 = (v_first + tid) * VE;
    if (v_first * VE >= c) return;
    const DEAR_GLOBAL float *in = (const DEAR_GLOBAL float *)param_tab[(size_t)worker * L + t.layer];
    if (e0 >= a && e0 + VE <= c)
        store_f4_dword_aligned<true>(dst + (e0 - a), __builtin_bit_cast(f4, load_vec<true>((global_u4_in)(in + e0))));
    const int64_t e = edge_element<VE>(a, c, v_first, DEAR_BLOCK);
    if (e >= 0) dst[e - a] = in[e];
}

// Shard buffer of one plan -> shard buffer of another over the same layers and workers: a workgroup
// takes a part of a tile of the new plan, finds where its first element lies in the old one and copies up to
// each old shard's end in turn.  Bound by HBM (4 bytes read, 4 written per element); both sides are only 4-byte
// aligned against each other, so vectors are counted from the piece's start.
// Going through a replica's tensors instead (gather, scatter, and gather again to give the tensors back)
// moves three times the bytes: re-planning BERT-Base-shaped at P = 8 took 1311 us that way and 831 this way.
__global__ __launch_bounds__(DEAR_BLOCK) void reshard_kernel(
    const dear_tile *__restrict__ tiles, const layer_place *__restrict__ places, int64_t from_row_len,
    const float *__restrict__ from, float *__restrict__ to)
{
    const dear_tile t = tiles[blockIdx.x / COPY_SPLIT];
    const int tid = threadIdx.x, skip = blockIdx.x % COPY_SPLIT * COPY_PART;
    const int count = t.count - skip < COPY_PART ? t.count - skip : COPY_PART;
    if (count <= 0) return;
    float *__restrict__ dst = to + t.dst_begin + skip;
    if (t.layer < 0) {
        for (int i = tid; i < count; i += DEAR_BLOCK) dst[i] = 0.0f;
        return;
    }
    const layer_place at = places[t.layer];
    const int64_t e = at.offset + t.src_begin + skip;
    int64_t shard = (int64_t)((double)e * at.inv_shard_len);  // off by one at most
    if (shard * at.shard_len > e) --shard;
    if ((shard + 1) * at.shard_len <= e) ++shard;
    int64_t slot = e - shard * at.shard_len;
    for (int done = 0; done < count; ++shard, slot = 0) {
        const int64_t room = at.shard_len - slot;
        const int n = room < count - done ? (int)room : count - done, i = 4 * tid;
        const float *__restrict__ src = from + shard * from_row_len + at.shard_base + slot;
        if (i + 4 <= n) store_f4_dword_aligned<true>(dst + done + i, load_f4_dword_aligned<true>(src + i));
        if (tid < n % 4) dst[done + n - n % 4 + tid] = src[n - n % 4 + tid];
        done += n;
    }
}

__host__ __device__ __forceinline__ dear_tile marked_tile(const dear_run &r, int64_t k, int64_t n)
{
    dear_tile t = tile_of_run(r, k);
    t.bucket |= (k == 0 ? TILE_FIRST : 0) | (k + 1 == n ? TILE_LAST : 0);
    return t;
}

// Tile table from runs, a workgroup a run.  The kernel takes some 3 us; what it saves is the host's time, which wrote and
// uploaded 32 bytes a tile and now 48 a run (BERT-Base-shaped, P = 8: 27000 tiles, 317 runs; making a context 150 us -> 45).
// A run's `bucket` goes into all its tiles, with notes on which of them are its first and its last.
__global__ __launch_bounds__(DEAR_BLOCK) void expand_runs_kernel(const dear_run *__restrict__ runs, dear_tile *__restrict__ tiles)
{
    const dear_run r = runs[blockIdx.x];
    const int64_t n = tiles_of_run(r);
    for (int64_t k = threadIdx.x; k < n; k += DEAR_BLOCK) tiles[r.first_tile + k] = marked_tile(r, k, n);
}

// ------------------------------------------------------------------------------- host side

inline bool misaligned(const void *p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

int check_call(const dear_ctx_impl *c, int32_t bucket)
{
    if (!c) return DEAR_EINVAL;
    if (bucket < -1 || bucket >= c->B) return DEAR_ERANGE;
    int dev = -1;  // the tables live on the device that was current at dear_ctx_create
    if (hipGetDevice(&dev) != hipSuccess) return DEAR_EHIP;
    if (dev != c->device) return DEAR_EINVAL;
    return DEAR_OK;
}

int check_shard_buffer(const void *p)
{
    if (!p) return DEAR_EINVAL;
    if (misaligned(p, 256)) return DEAR_EALIGN;
    return DEAR_OK;
}

// A bucket argument as a range of buckets: one, or (-1) all of them.
struct bucket_range {
    int32_t begin, end;
};

bucket_range buckets_of(const dear_ctx_impl *c, int32_t bucket)
{
    return bucket < 0 ? bucket_range{0, c->B} : bucket_range{bucket, bucket + 1};
}

int64_t tiles_of(const dear_ctx_impl *c, bucket_range r) { return c->tile_begin[r.end] - c->tile_begin[r.begin]; }

int64_t whole_tiles_of(const dear_ctx_impl *c, bucket_range r) { return c->whole_begin[r.end] - c->whole_begin[r.begin]; }
int64_t long_tiles_of(const dear_ctx_impl *c, bucket_range r) { return c->long_begin[r.end] - c->long_begin[r.begin]; }
int64_t cut_tiles_of(const dear_ctx_impl *c, bucket_range r) { return c->cut_begin[r.end] - c->cut_begin[r.begin]; }

int64_t elements_of(const std::vector<int64_t> &bucket_len, bucket_range r)
{
    return std::accumulate(bucket_len.begin() + r.begin, bucket_len.begin() + r.end, int64_t{0});
}

// Whether the launches were taken; says nothing of errors that other calls left behind.
bool expand_runs(const dear_run *runs, int64_t n_runs, dear_tile *tiles, hipStream_t st)
{
    for (; n_runs > 0; runs += MAX_GRID, n_runs -= MAX_GRID) {
        const int64_t n = n_runs < MAX_GRID ? n_runs : MAX_GRID;
        void *args[] = {&runs, &tiles};
        if (hipLaunchKernel(reinterpret_cast<const void *>(expand_runs_kernel), dim3(static_cast<unsigned>(n)), dim3(DEAR_BLOCK), args,
                            0, st) != hipSuccess)
            return false;
    }
    return true;
}

// Host memory that is not pinned -> device memory, stream-ordered.  The runtime takes copies of up to 16 KiB without waiting;
// behind queued work longer ones cost 7-10 us more of the GPU's time, so a table of a few such pieces goes in pieces
// (reduce-scatters with their tables back to back, us, one copy / pieces: 22 KB 177 / 167, 45 KB 152 / 143, 28 KB 43.6 / 35.0;
// 180 KB 150 / 163).
bool upload(unsigned char *to, const unsigned char *from, size_t bytes, hipStream_t st)
{
    constexpr size_t PIECE = 16 << 10, MOST = 64 << 10;
    const size_t step = bytes <= MOST ? PIECE : bytes;
    for (size_t at = 0; at < bytes; at += step)
        if (hipMemcpyAsync(to + at, from + at, bytes - at < step ? bytes - at : step, hipMemcpyHostToDevice, st) != hipSuccess)
            return false;
    return true;
}

int launch_status() { return hipGetLastError() == hipSuccess ? DEAR_OK : DEAR_EHIP; }

unsigned grid_width(int32_t max_workgroups, int64_t n_items)
{
    if (max_workgroups > 0 && n_items > max_workgroups) return static_cast<unsigned>(max_workgroups);
    return static_cast<unsigned>(n_items);
}

// LDS that a launch reserves for each workgroup, and nothing uses, so that `residency` of them share a CU's 160 KiB (4: five in
// fp32, whose kernel has no LDS of its own).
unsigned residency_lds(int residency)
{
    return residency == 0 ? 0 : residency == 1 ? 96 << 10 : residency == 2 ? 64 << 10 : residency == 3 ? 44 << 10 : 32 << 10;
}

// What a reduce-scatter launch is made from.  tiles, grads: device tables (a context's, or the static scratch's).  The
// launch may be one of several over all_tiles tiles, which hold all_elems elements and of which all_whole are whole, all_long lie in
// more than one part and all_cut are cut inside a vector.
struct rs_call {
    int P, L;
    const void *const *grads;
    int32_t max_workgroups;
    int prio;
    const dear_tile *tiles;
    int64_t n_tiles, all_tiles, all_elems, all_whole, all_long, all_cut;
    hipStream_t st;
};

template <bool BF16, rs_mode MODE, int U, int CH, bool TAIL>
void rs_launch_batch_as(const rs_call &c, const rs_sink<MODE> &o)
{
    constexpr int SPLIT = DEAR_TILE_ELEMS / ((BF16 ? 8 : 4) * DEAR_BLOCK * U);
    const unsigned n_items = static_cast<unsigned>(c.n_tiles * SPLIT);
    const dim3 grid(grid_width(c.max_workgroups, n_items));
    const int residency =
        (MODE & RS_GATHER) == 0 ? 0 : iteration_at_once_residency(BF16, (MODE & RS_GBAR) != 0, c.P, c.all_elems, c.all_tiles);
    auto launch = [&](auto kernel) {
        kernel<<<grid, dim3(DEAR_BLOCK), residency_lds(residency), c.st>>>(
            c.tiles, c.grads, c.L, c.P, 1.0f / static_cast<float>(c.P), o, n_items, c.prio);
    };
    // one launch for the iteration, and half tiles, are for unbounded grids only
    if constexpr ((MODE & RS_GATHER) == 0 && !(BF16 && U == 1))
        if (grid.x < n_items) return launch(reduce_scatter_batch_kernel<BF16, U, CH, TAIL, true, MODE>);
    launch(reduce_scatter_batch_kernel<BF16, U, CH, TAIL, false, MODE>);
}

// Replicas per load batch: the largest of 8/4/2/1 that divides P without a tail when
// P is small or a multiple of 4; otherwise batches of 8 with a predicated tail.
template <bool BF16, rs_mode MODE, int U>
void rs_launch_batch(const rs_call &c, const rs_sink<MODE> &o)
{
    if (c.P % 8 == 0)
        rs_launch_batch_as<BF16, MODE, U, 8, false>(c, o);
    else if (c.P % 4 == 0)
        rs_launch_batch_as<BF16, MODE, U, 4, false>(c, o);
    else if (c.P == 2)
        rs_launch_batch_as<BF16, MODE, U, 2, false>(c, o);
    else if (c.P == 1)
        rs_launch_batch_as<BF16, MODE, U, 1, false>(c, o);
    else
        rs_launch_batch_as<BF16, MODE, U, 8, true>(c, o);
}

template <bool BF16, rs_mode MODE>
void rs_launch_parts(const rs_call &c, const rs_sink<MODE> &o, const reduce_scatter_shape &shape)
{
    const unsigned n_items = static_cast<unsigned>(c.n_tiles * (shape.tiles ? 1 : reduce_scatter_split(BF16)));
    auto launch = [&](auto kernel) {
        kernel<<<dim3(n_items), dim3(DEAR_BLOCK), residency_lds(shape.residency), c.st>>>(
            c.tiles, c.grads, c.L, c.P, 1.0f / static_cast<float>(c.P), o, n_items, static_cast<unsigned>(shape.run));
    };
    auto launch_as = [&](auto depth, auto whole_tiles) {
        constexpr int D = decltype(depth)::value;
        constexpr bool TILES = decltype(whole_tiles)::value;
        if constexpr (!TILES)
            if (c.P == D) return launch(reduce_scatter_kernel<BF16, D, REST_NONE, TILES, MODE>);
        if constexpr (D > 1)
            if (c.P % D != 0) return launch(reduce_scatter_kernel<BF16, D, REST_TAIL, TILES, MODE>);
        if constexpr (D > 1 || TILES) launch(reduce_scatter_kernel<BF16, D, REST_BATCHES, TILES, MODE>);
    };
    auto launch_depth = [&](auto whole_tiles) {
        if (shape.depth == 8) return launch_as(std::integral_constant<int, 8>{}, whole_tiles);
        if (shape.depth == 4) return launch_as(std::integral_constant<int, 4>{}, whole_tiles);
        if (shape.depth == 2) return launch_as(std::integral_constant<int, 2>{}, whole_tiles);
        launch_as(std::integral_constant<int, 1>{}, whole_tiles);
    };
    if (shape.tiles)
        launch_depth(std::true_type{});
    else
        launch_depth(std::false_type{});
}

template <rs_mode MODE, bool BF16>
void rs_launch_type(const rs_call &c, const rs_sink<MODE> &o)
{
    if constexpr ((MODE & RS_GATHER) != 0) {
        if (BF16 && !iteration_at_once_half_tiles(c.all_elems, c.n_tiles)) return rs_launch_batch<BF16, MODE, BF16 ? 2 : 1>(c, o);
    } else {
        const int64_t parts = c.n_tiles * reduce_scatter_split(BF16);
        if (parts <= MAX_GRID && (c.max_workgroups == 0 || parts <= c.max_workgroups) && pointer_table_fits(c.P, c.L)) {
            const reduce_scatter_shape shape =
                reduce_scatter_shape_of(BF16, (MODE & RS_UPDATE) != 0, (MODE & RS_W_NEXT) != 0, c.P, c.all_elems, c.all_tiles, c.all_long,
                                        c.all_cut);
            if (shape.depth > 0) return rs_launch_parts<BF16, MODE>(c, o, shape);
        }
        if (BF16 && !reduce_scatter_half_tiles((MODE & RS_UPDATE) != 0, c.max_workgroups, c.all_elems, c.n_tiles, c.all_whole))
            return rs_launch_batch<BF16, MODE, BF16 ? 2 : 1>(c, o);
    }
    rs_launch_batch<BF16, MODE, 1>(c, o);
}

template <rs_mode MODE>
void rs_launch(bool bf16, const rs_call &c, const rs_sink<MODE> &o)
{
    if (bf16)
        rs_launch_type<MODE, true>(c, o);
    else
        rs_launch_type<MODE, false>(c, o);
}

// Up to this many tiles a context's table is cut on the host.  Making a context, us, on the host / with the kernel and the wait
// for it: 93 tiles 12.9 / 17, 2700 tiles 28 / 31, 5100 (300 tensors) 38 / 29, 5000 (100 tensors) 34 / 21, 27000 150 / 45.
constexpr int64_t HOST_TILES = 3072;

}  // namespace

struct dear_ctx_s : dear_ctx_impl {};

extern "C" int dear_ctx_create(const dear_plan_t *plan, int32_t grad_dtype,
                               const void *const *grad_ptrs, float *const *param_ptrs,
                               dear_ctx_t **out)
{
    if (!plan || !grad_ptrs || !param_ptrs || !out) return DEAR_EINVAL;
    if (grad_dtype != DEAR_F32 && grad_dtype != DEAR_BF16) return DEAR_EINVAL;
    if ((grad_dtype == DEAR_F32 ? 4 : 2) != plan->g) return DEAR_EINVAL;
    const size_t n_ptr = static_cast<size_t>(plan->P) * plan->L;
    for (size_t i = 0; i < n_ptr; ++i) {
        if (!grad_ptrs[i] || !param_ptrs[i]) return DEAR_EINVAL;
        if (misaligned(grad_ptrs[i], 16) || misaligned(param_ptrs[i], 16)) return DEAR_EALIGN;
    }
    std::unique_ptr<dear_ctx_s> c;
    std::vector<dear_run> runs;
    std::vector<unsigned char> image;  // what is uploaded: tiles or runs, layer places, gradient and parameter pointers
    int64_t n_runs = 0, n_tiles = 0;
    table_layout at{};
    try {
        c.reset(new dear_ctx_s);
        c->L = plan->L;
        c->B = plan->B;
        c->P = plan->P;
        c->g = plan->g;
        c->row_len = plan->row_len;
        c->bucket_len = plan->bucket_len;
        c->bucket_shard_len = plan->bucket_shard_len;
        c->bucket_shard_base = plan->bucket_shard_base;
        c->layer_sizes = plan->layer_sizes;
        c->tile_begin.assign(plan->B + 1, 0);
        c->whole_begin.assign(plan->B + 1, 0);
        c->long_begin.assign(plan->B + 1, 0);
        c->cut_begin.assign(plan->B + 1, 0);
        n_runs = dear_emit_runs(*plan, 0, plan->B, nullptr, 0, &n_tiles, c->tile_begin.data());
        runs.resize(n_runs);
        at = lay_out_tables(n_tiles <= HOST_TILES, n_tiles, n_runs, plan->L * sizeof(layer_place), n_ptr * sizeof(void *));
        image.resize(at.end - at.uploaded);
    } catch (const std::bad_alloc &) {
        return DEAR_ENOMEM;
    }
    if (n_tiles > 0x7fffffff / 16) return DEAR_EINVAL;  // item counts fit 31 bits, up to 16 a tile
    if (hipGetDevice(&c->device) != hipSuccess) return DEAR_EHIP;
    dear_emit_runs(*plan, 0, plan->B, runs.data(), n_runs, &n_tiles, nullptr);
    for (const dear_run &r : runs) {
        c->whole_begin[r.bucket + 1] += whole_tiles_of_run(r);
        c->long_begin[r.bucket + 1] += long_tiles_of_run(r, 16 / c->g);
        c->cut_begin[r.bucket + 1] += cut_tiles_of_run(r, 16 / c->g);
    }
    std::partial_sum(c->whole_begin.begin(), c->whole_begin.end(), c->whole_begin.begin());
    std::partial_sum(c->long_begin.begin(), c->long_begin.end(), c->long_begin.begin());
    std::partial_sum(c->cut_begin.begin(), c->cut_begin.end(), c->cut_begin.begin());
    c->replicas_alike = dear_mark_runs(*plan, param_ptrs, runs.data(), n_runs);
    const bool on_host = n_tiles <= HOST_TILES;
    if (on_host) {
        dear_tile *tiles = reinterpret_cast<dear_tile *>(image.data());
        for (const dear_run &r : runs)
            for (int64_t k = 0, n = tiles_of_run(r); k < n; ++k) tiles[r.first_tile + k] = marked_tile(r, k, n);
    } else {
        std::memcpy(image.data(), runs.data(), n_runs * sizeof(dear_run));
    }
    auto in_image = [&](size_t device_offset) { return image.data() + (device_offset - at.uploaded); };
    for (int32_t l = 0; l < plan->L; ++l) {
        const int32_t b = plan->layer_bucket[l];
        const int64_t S = plan->bucket_shard_len[b];
        const layer_place place{plan->layer_offset[l], S, plan->bucket_shard_base[b], 1.0 / static_cast<double>(S)};
        std::memcpy(in_image(at.places) + l * sizeof place, &place, sizeof place);
    }
    std::memcpy(in_image(at.grad), grad_ptrs, n_ptr * sizeof(void *));
    std::memcpy(in_image(at.param), param_ptrs, n_ptr * sizeof(void *));

    int rc = DEAR_OK;
    unsigned char *base = nullptr;
    if (hipMalloc(&c->d_tables, at.end) != hipSuccess) {
        c->d_tables = nullptr;
        rc = DEAR_ENOMEM;
    } else {
        c->d_tiles = static_cast<dear_tile *>(c->d_tables);
        base = static_cast<unsigned char *>(c->d_tables);
        unsigned char *const to = base + at.uploaded;
        if (on_host) {
            if (hipMemcpy(to, image.data(), image.size(), hipMemcpyHostToDevice) != hipSuccess) rc = DEAR_EHIP;
        } else {
            const bool sent = upload(to, image.data(), image.size(), nullptr) &&
                              expand_runs(reinterpret_cast<const dear_run *>(to), n_runs, c->d_tiles, nullptr);
            if (hipStreamSynchronize(nullptr) != hipSuccess || !sent) rc = DEAR_EHIP;
        }
    }
    if (rc != DEAR_OK) {
        (void)hipGetLastError();
        dear_ctx_destroy(c.release());
        return rc;
    }
    c->d_places = reinterpret_cast<layer_place *>(base + at.places);
    c->d_grad = reinterpret_cast<const void **>(base + at.grad);
    c->d_param = reinterpret_cast<float **>(base + at.param);
    *out = c.release();
    return DEAR_OK;
}

extern "C" int dear_ctx_set_max_workgroups(dear_ctx_t *c, int32_t max_workgroups)
{
    if (!c || max_workgroups < 0) return DEAR_EINVAL;
    c->max_workgroups = max_workgroups;
    return DEAR_OK;
}

extern "C" int dear_ctx_set_wave_priority(dear_ctx_t *c, int32_t priority)
{
    if (!c || priority < 0 || priority > 3) return DEAR_EINVAL;
    c->wave_priority = priority;
    return DEAR_OK;
}

extern "C" void dear_ctx_destroy(dear_ctx_t *c)
{
    if (!c) return;
    (void)hipDeviceSynchronize();
    if (c->d_tables) (void)hipFree(c->d_tables);
    delete c;
}

namespace {

// What a launch goes over: tiles begin .. begin+count-1 of the table, part of a call's `all_tiles` with `all_elems`.
struct tile_range {
    int64_t begin, count, all_tiles, all_elems, all_whole, all_long, all_cut;
};

tile_range range_of(const dear_ctx_impl *c, bucket_range r)
{
    return {c->tile_begin[r.begin], tiles_of(c, r),      tiles_of(c, r),     elements_of(c->bucket_len, r),
            whole_tiles_of(c, r),   long_tiles_of(c, r), cut_tiles_of(c, r)};
}

template <rs_mode MODE>
int launch_reduce_scatter(const dear_ctx_impl *c, tile_range t, const rs_sink<MODE> &o, hipStream_t st)
{
    if (t.count == 0) return DEAR_OK;
    const rs_call call{c->P, c->L, c->d_grad, c->max_workgroups, c->wave_priority, c->d_tiles + t.begin, t.count,
                       t.all_tiles, t.all_elems, t.all_whole, t.all_long, t.all_cut, st};
    rs_launch<MODE>(c->g == 2, call, o);
    return launch_status();
}

int launch_update(const dear_ctx_impl *c, bucket_range r, const float *shard_grad, float *shard_param,
                  float *shard_mom, float lr, float momentum, hipStream_t st)
{
    // All buckets: the P rows are back to back, so the whole buffer is one run.
    int64_t base = 0, elems = c->row_len * c->P;
    unsigned rows = 1;
    if (r.begin > 0 || r.end < c->B) {
        base = c->bucket_shard_base[r.begin];
        elems = c->bucket_shard_base[r.end - 1] + c->bucket_shard_len[r.end - 1] - base;
        rows = static_cast<unsigned>(c->P);
    }
    const int64_t vecs = elems / 4;  // shard lengths are multiples of DEAR_SHARD_ALIGN
    if (vecs == 0) return DEAR_OK;
    const bool bounded = c->max_workgroups > 0 &&
                         (vecs + UPD_U_BOUNDED * DEAR_BLOCK - 1) / (UPD_U_BOUNDED * DEAR_BLOCK) * rows > c->max_workgroups;
    const int64_t per_block = static_cast<int64_t>(bounded ? UPD_U_BOUNDED : UPD_U) * DEAR_BLOCK;
    const int64_t blocks = (vecs + per_block - 1) / per_block;
    const int64_t n_items = blocks * rows;
    if (n_items > (bounded ? 0x7fffffff : MAX_GRID)) return DEAR_EINVAL;
    if (bounded)
        shard_update_kernel<UPD_U_BOUNDED, true><<<dim3(c->max_workgroups), dim3(DEAR_BLOCK), 0, st>>>(
            shard_grad, shard_param, shard_mom, c->row_len, base, vecs, lr, momentum,
            static_cast<unsigned>(blocks), static_cast<unsigned>(n_items), c->wave_priority, 0);
    else
        shard_update_kernel<UPD_U, false><<<dim3(static_cast<unsigned>(n_items)), dim3(DEAR_BLOCK), 0, st>>>(
            shard_grad, shard_param, shard_mom, c->row_len, base, vecs, lr, momentum,
            static_cast<unsigned>(blocks), static_cast<unsigned>(n_items), 0, shard_update_run(rows, n_items));
    return launch_status();
}

// behind_update: the reduce-scatter + update of the same tiles is the launch before, with (caches_w) RS_W_NEXT.
int launch_all_gather(const dear_ctx_impl *c, tile_range t, const float *shard_param, int32_t first_worker,
                      int32_t n_workers, hipStream_t st, bool behind_update = false, bool caches_w = false)
{
    const int64_t count = t.count;
    if (count == 0) return DEAR_OK;
    if (!all_gather_fits(count, n_workers, c->max_workgroups)) return DEAR_EINVAL;
    const dear_tile *tiles = c->d_tiles + t.begin;
    if (all_gather_bounded(count, n_workers, c->max_workgroups)) {
        const unsigned width = grid_width(c->max_workgroups, count);
        all_gather_bounded_kernel<<<dim3(width), dim3(DEAR_BLOCK), 0, st>>>(
            tiles, c->d_param, c->L, first_worker, n_workers, shard_param, static_cast<unsigned>(count),
            c->wave_priority);
    } else {
        constexpr unsigned chunk = DEAR_AG_CHUNK_BYTES / (16 * DEAR_BLOCK);
        const unsigned n_parts = static_cast<unsigned>(count * AG_SPLIT), n_p = static_cast<unsigned>(n_workers);
        const unsigned whole = n_parts / chunk * chunk;
        const bool eighths = c->replicas_alike && all_gather_in_eighths(t.all_elems * count / t.all_tiles, count, n_workers);
        const unsigned run =
            eighths ? 0 : all_gather_run(c->g, caches_w, c->max_workgroups, c->P, t.all_elems, count, t.all_whole, t.all_long, t.all_cut,
                                         n_workers, behind_update);
        const all_gather_order o = all_gather_numbering(run, c->max_workgroups, whole, n_parts, n_workers);
        const auto kernel = eighths && o.len % 8 == 0 ? all_gather_kernel<0, true>
                            : o.run ? all_gather_kernel<1, false> : all_gather_kernel<0, false>;
        kernel<<<dim3((whole + o.len) * n_p), dim3(DEAR_BLOCK), 0, st>>>(
            tiles, c->d_param, c->L, first_worker, n_p, shard_param, n_parts, 0xffffffffu / n_p, o.len,
            0xffffffffu / (o.len ? o.len : 1));
    }
    return launch_status();
}

// Arguments of the calls that update: w, v and, where there is one, gbar are three different buffers.
int check_update_buffers(const float *shard_param, const float *shard_mom)
{
    int rc = check_shard_buffer(shard_param);
    if (rc == DEAR_OK) rc = check_shard_buffer(shard_mom);
    if (rc == DEAR_OK && shard_param == shard_mom) rc = DEAR_EINVAL;
    return rc;
}

int check_update_buffers(const float *shard_grad, const float *shard_param, const float *shard_mom)
{
    int rc = check_shard_buffer(shard_grad);
    if (rc == DEAR_OK) rc = check_update_buffers(shard_param, shard_mom);
    if (rc == DEAR_OK && (shard_grad == shard_param || shard_grad == shard_mom)) rc = DEAR_EINVAL;
    return rc;
}

}  // namespace

extern "C" int dear_reduce_scatter(dear_ctx_t *c, int32_t bucket, float *shard_grad, void *hip_stream)
{
    int rc = check_call(c, bucket);
    if (rc == DEAR_OK) rc = check_shard_buffer(shard_grad);
    if (rc != DEAR_OK) return rc;
    const rs_sink<RS_GBAR> o{shard_grad, nullptr, nullptr, 0.0f, 0.0f, nullptr};
    return launch_reduce_scatter(c, range_of(c, buckets_of(c, bucket)), o, static_cast<hipStream_t>(hip_stream));
}

extern "C" int dear_reduce_scatter_update(dear_ctx_t *c, int32_t bucket, float *shard_param,
                                         float *shard_mom, float lr, float momentum, void *hip_stream)
{
    int rc = check_call(c, bucket);
    if (rc == DEAR_OK) rc = check_update_buffers(shard_param, shard_mom);
    if (rc != DEAR_OK) return rc;
    const rs_sink<RS_UPDATE> o{nullptr, shard_param, shard_mom, lr, momentum, nullptr};
    return launch_reduce_scatter(c, range_of(c, buckets_of(c, bucket)), o, static_cast<hipStream_t>(hip_stream));
}

extern "C" int dear_shard_update(dear_ctx_t *c, int32_t bucket, const float *shard_grad,
                                 float *shard_param, float *shard_mom, float lr, float momentum,
                                 void *hip_stream)
{
    int rc = check_call(c, bucket);
    if (rc == DEAR_OK) rc = check_update_buffers(shard_grad, shard_param, shard_mom);
    if (rc != DEAR_OK) return rc;
    return launch_update(c, buckets_of(c, bucket), shard_grad, shard_param, shard_mom, lr, momentum,
                         static_cast<hipStream_t>(hip_stream));
}

extern "C" int dear_update_all_gather(dear_ctx_t *c, int32_t bucket, const float *shard_grad,
                                      float *shard_param, float *shard_mom, float lr, float momentum,
                                      void *hip_stream)
{
    int rc = check_call(c, bucket);
    if (rc == DEAR_OK) rc = check_update_buffers(shard_grad, shard_param, shard_mom);
    if (rc != DEAR_OK) return rc;
    const bucket_range r = buckets_of(c, bucket);
    const int64_t count = tiles_of(c, r), elems = elements_of(c->bucket_len, r), whole = whole_tiles_of(c, r);
    if (count == 0) return DEAR_OK;
    const dear_tile *tiles = c->d_tiles + c->tile_begin[r.begin];
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const unsigned width = grid_width(c->max_workgroups, count);
    if (update_all_gather_splits(elems, count, whole, c->P, c->max_workgroups)) {
        rc = launch_update(c, r, shard_grad, shard_param, shard_mom, lr, momentum, st);
        return rc == DEAR_OK ? launch_all_gather(c, range_of(c, r), shard_param, 0, c->P, st) : rc;
    }
    auto launch = [&](auto kernel, int64_t items, unsigned grid, int prio) {
        kernel<<<dim3(grid), dim3(DEAR_BLOCK), 0, st>>>(tiles, c->d_param, c->L, c->P, shard_grad, shard_param, shard_mom, lr,
                                                        momentum, static_cast<unsigned>(items), prio);
    };
    if (width < count)
        launch(update_all_gather_kernel<4, true>, count, width, c->wave_priority);
    else if (update_all_gather_quarters(elems, count, whole, c->P, c->max_workgroups))
        launch(update_all_gather_kernel<1, false>, count * 4, width * 4, 0);
    else
        launch(update_all_gather_kernel<4, false>, count, width, 0);
    return launch_status();
}

extern "C" int dear_all_gather_workers(dear_ctx_t *c, int32_t bucket, const float *shard_param,
                                       int32_t first_worker, int32_t n_workers, void *hip_stream)
{
    int rc = check_call(c, bucket);
    if (rc == DEAR_OK) rc = check_shard_buffer(shard_param);
    if (rc != DEAR_OK) return rc;
    if (first_worker < 0 || n_workers < 1 || first_worker > c->P - n_workers) return DEAR_ERANGE;
    return launch_all_gather(c, range_of(c, buckets_of(c, bucket)), shard_param, first_worker, n_workers,
                             static_cast<hipStream_t>(hip_stream));
}

extern "C" int dear_all_gather(dear_ctx_t *c, int32_t bucket, const float *shard_param, void *hip_stream)
{
    if (!c) return DEAR_EINVAL;
    return dear_all_gather_workers(c, bucket, shard_param, 0, c->P, hip_stream);
}

namespace {

// Reduce-scatter and update in one kernel, gbar stored only where it is wanted; MORE: RS_W_NEXT or RS_GATHER.
template <rs_mode MORE>
int launch_reduce_scatter_update(const dear_ctx_impl *c, tile_range t, float *shard_grad, float *shard_param,
                                 float *shard_mom, float lr, float momentum, hipStream_t st)
{
    if (shard_grad) {
        const rs_sink<RS_GBAR | RS_UPDATE | MORE> o{shard_grad, shard_param, shard_mom, lr, momentum, c->d_param};
        return launch_reduce_scatter(c, t, o, st);
    }
    const rs_sink<RS_UPDATE | MORE> o{nullptr, shard_param, shard_mom, lr, momentum, c->d_param};
    return launch_reduce_scatter(c, t, o, st);
}

}  // namespace

extern "C" int dear_iteration(dear_ctx_t *c, int32_t bucket, float *shard_grad, float *shard_param,
                              float *shard_mom, float lr, float momentum, void *hip_stream)
{
    int rc = check_call(c, bucket);
    if (rc == DEAR_OK)
        rc = shard_grad ? check_update_buffers(shard_grad, shard_param, shard_mom)
                        : check_update_buffers(shard_param, shard_mom);
    if (rc != DEAR_OK) return rc;
    const bucket_range all = buckets_of(c, bucket);
    auto group_from = [&](int32_t b) {
        bucket_range r{b, b + 1};
        while (r.end < all.end && tiles_of(c, bucket_range{b, r.end + 1}) <= ITERATION_TILES) ++r.end;
        return r;
    };
    for (bucket_range r{0, all.begin}; r.end < all.end;) {  // nothing is launched unless everything can be
        r = group_from(r.end);
        if (!all_gather_fits(tiles_of(c, r), c->P, c->max_workgroups)) return DEAR_EINVAL;
    }
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const tile_range whole = range_of(c, all);
    if (iteration_gathers_at_once(c->g, c->P, whole.all_elems, whole.count, shard_grad != nullptr, c->max_workgroups))
        return launch_reduce_scatter_update<RS_GATHER>(c, whole, shard_grad, shard_param, shard_mom, lr, momentum, st);
    for (bucket_range r{0, all.begin}; rc == DEAR_OK && r.end < all.end;) {
        r = group_from(r.end);
        const tile_range group = range_of(c, r);
        if (shard_grad && iteration_updates_apart(c->g, c->P, group.count)) {
            const rs_sink<RS_GBAR> o{shard_grad, nullptr, nullptr, 0.0f, 0.0f, nullptr};
            rc = launch_reduce_scatter(c, group, o, st);
            if (rc == DEAR_OK) rc = launch_update(c, r, shard_grad, shard_param, shard_mom, lr, momentum, st);
            if (rc == DEAR_OK) rc = launch_all_gather(c, group, shard_param, 0, c->P, st);
            continue;
        }
        const int64_t pieces = iteration_pieces(c->g, c->P, group.count, c->tile_begin[c->B]);
        for (int64_t i = 0; rc == DEAR_OK && i < pieces; ++i) {
            tile_range t = group;
            t.begin += group.count * i / pieces;
            t.count = group.begin + group.count * (i + 1) / pieces - t.begin;
            const bool caches_w = iteration_caches_w(c->g, c->P, t.count, c->tile_begin[c->B]);
            if (caches_w)
                rc = launch_reduce_scatter_update<RS_W_NEXT>(c, t, shard_grad, shard_param, shard_mom, lr, momentum, st);
            else
                rc = launch_reduce_scatter_update<0>(c, t, shard_grad, shard_param, shard_mom, lr, momentum, st);
            if (rc == DEAR_OK) rc = launch_all_gather(c, t, shard_param, 0, c->P, st, true, caches_w);
        }
    }
    return rc;
}

namespace {

// Workgroups for all parts of n_tiles tiles, in as many launches as HIP wants for them.
template <class Launch>
int launch_copies(int64_t n_tiles, Launch launch)
{
    constexpr int64_t MOST = MAX_GRID / COPY_SPLIT;
    int rc = DEAR_OK;
    for (int64_t first = 0; rc == DEAR_OK && first < n_tiles; first += MOST) {
        const int64_t n = n_tiles - first < MOST ? n_tiles - first : MOST;
        launch(first, dim3(static_cast<unsigned>(n * COPY_SPLIT)));
        rc = launch_status();
    }
    return rc;
}

}  // namespace

extern "C" int dear_scatter_params(dear_ctx_t *c, int32_t worker, float *shard_param, void *hip_stream)
{
    int rc = check_call(c, -1);
    if (rc != DEAR_OK) return rc;
    if (worker < 0 || worker >= c->P) return DEAR_ERANGE;
    rc = check_shard_buffer(shard_param);
    if (rc != DEAR_OK) return rc;
    return launch_copies(c->tile_begin[c->B], [&](int64_t first, dim3 grid) {
        scatter_params_kernel<<<grid, dim3(DEAR_BLOCK), 0, static_cast<hipStream_t>(hip_stream)>>>(
            c->d_tiles + first, c->d_param, c->L, worker, shard_param);
    });
}

extern "C" int dear_reshard(dear_ctx_t *from, dear_ctx_t *to, const float *shard_from, float *shard_to, void *hip_stream)
{
    int rc = check_call(from, -1);
    if (rc == DEAR_OK) rc = check_call(to, -1);
    if (rc == DEAR_OK) rc = check_shard_buffer(shard_from);
    if (rc == DEAR_OK) rc = check_shard_buffer(shard_to);
    if (rc != DEAR_OK) return rc;
    if (shard_from == shard_to || from->P != to->P || from->layer_sizes != to->layer_sizes) return DEAR_EINVAL;
    return launch_copies(to->tile_begin[to->B], [&](int64_t first, dim3 grid) {
        reshard_kernel<<<grid, dim3(DEAR_BLOCK), 0, static_cast<hipStream_t>(hip_stream)>>>(
            to->d_tiles + first, from->d_places, from->row_len, shard_from, shard_to);
    });
}

// ------------------------------------------------------------- entry point without allocation
//
// dear_reduce_scatter needs a context, and creating one allocates device memory for the tile
// table and the pointer table its kernel reads.  For callers that cannot allocate, the same
// kernel reads both tables from this file-scope device array instead.  Layout: gradient
// pointer table first, the runs on the next 256-byte boundary behind it, so that one copy of the
// bytes in use brings both up, then the tiles that expand_runs_kernel makes of them.  Every GPU the library
// runs on holds its own copy of the array until the process ends.
namespace {

constexpr size_t STATIC_MAX_PTRS = DEAR_STATIC_MAX_POINTERS;
constexpr size_t STATIC_MAX_TILES = DEAR_STATIC_MAX_TILES;  // and runs: each has a tile at least
constexpr size_t STATIC_PTR_BYTES = STATIC_MAX_PTRS * sizeof(void *);
constexpr size_t STATIC_RUN_BYTES = STATIC_MAX_TILES * sizeof(dear_run);
constexpr size_t STATIC_TILE_BYTES = STATIC_MAX_TILES * sizeof(dear_tile);
static_assert(STATIC_PTR_BYTES % 256 == 0 && STATIC_RUN_BYTES % 256 == 0, "the tables must start aligned");

__device__ __align__(256) unsigned char scratch[STATIC_PTR_BYTES + STATIC_RUN_BYTES + STATIC_TILE_BYTES];

// Host staging of pointers and runs (pageable, file scope: no heap use on this path), and of the tiles that the host cuts.
alignas(256) unsigned char host_stage[STATIC_PTR_BYTES + STATIC_RUN_BYTES];
dear_tile host_tiles[STATIC_MAX_TILES];

constexpr int MAX_DEVICES = 64;
unsigned char *scratch_of_device[MAX_DEVICES];  // device address of `scratch`, per GPU
hipEvent_t uploaded_on_device[MAX_DEVICES];     // behind the upload of the tables, per GPU

// `scratch` names a host-side stand-in in host code; the device address has to be asked for, and an event
// made, once per device, with that device current.
int static_scratch(int device, unsigned char **out)
{
    if (device < 0 || device >= MAX_DEVICES) return DEAR_EINVAL;
    if (!uploaded_on_device[device]) {
        hipEvent_t event = nullptr;
        if (hipEventCreateWithFlags(&event, hipEventDisableTiming) != hipSuccess || !event) {
            (void)hipGetLastError();
            return DEAR_EHIP;
        }
        uploaded_on_device[device] = event;
    }
    if (!scratch_of_device[device]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return DEAR_EHIP;
        }
        scratch_of_device[device] = static_cast<unsigned char *>(p);
    }
    *out = scratch_of_device[device];
    return DEAR_OK;
}

}  // namespace

extern "C" int dear_reduce_scatter_static(const dear_plan_t *plan, int32_t grad_dtype,
                                          const void *const *grad_ptrs, int32_t bucket, float *shard_grad,
                                          void *hip_stream)
{
    if (!plan || !grad_ptrs) return DEAR_EINVAL;
    if (grad_dtype != DEAR_F32 && grad_dtype != DEAR_BF16) return DEAR_EINVAL;
    if ((grad_dtype == DEAR_F32 ? 4 : 2) != plan->g) return DEAR_EINVAL;
    if (bucket < -1 || bucket >= plan->B) return DEAR_ERANGE;
    int rc = check_shard_buffer(shard_grad);
    if (rc != DEAR_OK) return rc;
    const size_t n_ptr = static_cast<size_t>(plan->P) * plan->L;
    if (n_ptr > STATIC_MAX_PTRS) return DEAR_ETOOBIG;
    const int32_t b_first = bucket < 0 ? 0 : bucket, b_last = bucket < 0 ? plan->B : bucket + 1;
    // only the gradient tensors of the buckets processed are dereferenced, but the whole table is checked
    for (size_t i = 0; i < n_ptr; ++i) {
        if (!grad_ptrs[i]) return DEAR_EINVAL;
        if (misaligned(grad_ptrs[i], 16)) return DEAR_EALIGN;
    }
    auto aligned = [](size_t n) { return (n + 255) & ~size_t(255); };
    const size_t runs_at = aligned(n_ptr * sizeof(void *));  // <= STATIC_PTR_BYTES
    int64_t n_tiles = 0;
    const int64_t n_runs = dear_emit_runs(*plan, b_first, b_last, reinterpret_cast<dear_run *>(host_stage + runs_at),
                                          STATIC_MAX_TILES, &n_tiles, nullptr);
    if (n_tiles > static_cast<int64_t>(STATIC_MAX_TILES)) return DEAR_ETOOBIG;
    if (n_tiles == 0) return DEAR_OK;
    int64_t n_whole = 0, n_long = 0, n_cut = 0;
    for (int64_t i = 0; i < n_runs; ++i) {
        const dear_run &r = reinterpret_cast<const dear_run *>(host_stage + runs_at)[i];
        n_whole += whole_tiles_of_run(r);
        n_long += long_tiles_of_run(r, 16 / plan->g);
        n_cut += cut_tiles_of_run(r, 16 / plan->g);
    }

    int device = -1;
    if (hipGetDevice(&device) != hipSuccess) return DEAR_EHIP;
    unsigned char *dev = nullptr;
    rc = static_scratch(device, &dev);
    if (rc != DEAR_OK) return rc;

    // Where the tiles are few more bytes than the runs, as with hundreds of short tensors, the host cuts them.  Calls back to back,
    // us, runs uploaded / tiles: 600 tensors P = 12 2 M elements (31 KB of tiles, 29 of runs) 45.4 / 43.0, 200 P = 16 3 M (28, 10)
    // 35.1 / 35.8, 400 P = 8 20 M (164, 20) 143.2 / 152.8.
    const bool on_host = n_tiles * sizeof(dear_tile) <= 2 * n_runs * sizeof(dear_run);
    if (on_host) {
        const dear_run *runs = reinterpret_cast<const dear_run *>(host_stage + runs_at);
        for (const dear_run *r = runs; r < runs + n_runs; ++r)
            for (int64_t k = 0, n = tiles_of_run(*r); k < n; ++k) host_tiles[r->first_tile + k] = tile_of_run(*r, k);
        std::memcpy(host_stage + runs_at, host_tiles, n_tiles * sizeof(dear_tile));  // fits: STATIC_RUN_BYTES are more
    }

    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {  // it cannot be waited for
        (void)hipGetLastError();
        return DEAR_EHIP;
    }
    for (size_t i = 0; i < n_ptr; ++i) reinterpret_cast<const void **>(host_stage)[i] = grad_ptrs[i];
    // Stream-ordered upload: earlier kernels of this stream that still read the scratch finish
    // first.  The staging memory is pageable and is reused by the next call, so the call waits for the
    // upload before it returns, but with the kernel behind it in the queue already: the GPU idles for the copy of the pointers
    // and runs and the making of the tiles, and not for the host's wake-up and launch.  Calls back to back, us, before (tiles
    // uploaded, stream drained, kernel launched) / now: 161 tensors P = 8 fp32 25 M elements 177 / 167, 11 tensors P = 8 bf16
    // 6 M 43.6 / 30.2, 30 tensors P = 6 bf16 60 M 193 / 168, 400 tensors P = 8 fp32 20 M 155 / 143, 600 P = 12 2 M 43.7 / 44.0.
    const size_t bytes = runs_at + (on_host ? n_tiles * sizeof(dear_tile) : n_runs * sizeof(dear_run));
    const dear_run *runs = reinterpret_cast<const dear_run *>(dev + runs_at);
    dear_tile *tiles = reinterpret_cast<dear_tile *>(dev + (on_host ? runs_at : aligned(bytes)));
    if (!upload(dev, host_stage, bytes, st) || !(on_host || expand_runs(runs, n_runs, tiles, st)) ||
        hipEventRecord(uploaded_on_device[device], st) != hipSuccess) {
        (void)hipStreamSynchronize(st);
        (void)hipGetLastError();
        return DEAR_EHIP;
    }
    const void *const *grad_tab = reinterpret_cast<const void *const *>(dev);
    const rs_sink<RS_GBAR> o{shard_grad, nullptr, nullptr, 0.0f, 0.0f, nullptr};
    const int64_t elems = elements_of(plan->bucket_len, bucket_range{b_first, b_last});
    rs_launch<RS_GBAR>(plan->g == 2, rs_call{plan->P, plan->L, grad_tab, 0, 0, tiles, n_tiles, n_tiles, elems, n_whole, n_long, n_cut, st}, o);
    rc = launch_status();
    if (hipEventSynchronize(uploaded_on_device[device]) != hipSuccess) {
        (void)hipGetLastError();
        return DEAR_EHIP;
    }
    return rc;
}
