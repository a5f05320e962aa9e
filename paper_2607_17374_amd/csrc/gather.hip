// A sampled layer kept in core, aggregated destination by destination.
//
// Broadcasting a sampled layer chunk by chunk costs every kept message a
// read and a write of its destination's fp32 accumulator row: with a fanout
// of at most a few dozen in-edges over many chunks nearly every message is a
// segment of its own.  A layer whose chunks all stay in device memory does
// not need the accumulators: the pushes copy the source rows into a table
// of the layer's own, and the last push (or a finalize with chunks missing,
// for the rows that are complete) evaluates
//     out[v] = act(phi_v * ((sum_{u in M(v)} w_u x_u) W) + b)
// in one kernel, by linearity the same value (the aggregate is formed
// before the linear map instead of after, Sec. 3.9), from the kept in-edge
// lists the sampler writes in destination order.  Nothing is sorted by
// chunk, and no work lists, counts or accumulators exist.
//
// What bounds it: a message costs one read of its source's input row (256 B
// at 128 bf16 inputs) instead of 1 KiB of transformed row and 2 KiB of
// accumulator row at 256 outputs.  12.5M destinations, 128 -> 256 bf16,
// fanout 15: the 5.8M with messages (35.6M of them) take 3.9 ms (13.8 GB
// counted, 3.5 TB/s of random rows; 390 TFLOP/s of products, the matrix cores
// busy for 0.70 of the compute units' busy cycles), the 6.7M without 1.2 ms
// (5.2 GB, 4.4 TB/s; 0.72), the table 1.5 ms (6.4 GB, 4.2 TB/s).  The
// broadcast took 18.9 ms of scatter and 8.6 ms of transform.
#include <algorithm>
#include <vector>

#include "gather.hpp"
#include "gemm_device.hpp"

namespace taurus {

// ------------------------------------------------------------------ types --

template <int DT>
struct GatherOp;
template <>
struct GatherOp<TAURUS_F32> {
    static constexpr int EP = 4;     // values of a 16-byte piece
    typedef float4 frag;
    static __device__ inline void add(float w, frag x, float (&a)[EP]) {
        a[0] = fmaf(w, x.x, a[0]);
        a[1] = fmaf(w, x.y, a[1]);
        a[2] = fmaf(w, x.z, a[2]);
        a[3] = fmaf(w, x.w, a[3]);
    }
};
template <>
struct GatherOp<TAURUS_BF16> {
    static constexpr int EP = 8;
    typedef uint4 frag;
    static __device__ inline void add(float w, frag x, float (&a)[EP]) {
        const uint32_t q[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int i = 0; i < 4; i++) {
            a[2 * i] = fmaf(w, __uint_as_float(q[i] << 16), a[2 * i]);
            a[2 * i + 1] = fmaf(w, __uint_as_float(q[i] & 0xffff0000u), a[2 * i + 1]);
        }
    }
};

// An fp32 value as the sum of three bf16 (8 significant bits each, by
// truncation, so that no part overflows and their sum is the value exactly):
// the products of an aggregate with the bf16 weights then lose nothing
// against fp32 operands.  A value that is not finite stays whole in the
// first part.
__device__ inline void split_bf16(const float (&a)[8], uint4& hi, uint4& mid, uint4& lo) {
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; i++) {
        uint32_t ph[2], pm[2], pl[2];
#pragma unroll
        for (int k = 0; k < 2; k++) {
            const float x = a[2 * i + k];
            const uint32_t xh = __float_as_uint(x) & 0xffff0000u;
            float r = x - __uint_as_float(xh);
            r = __builtin_isfinite(x) ? r : 0.0f;
            const uint32_t xm = __float_as_uint(r) & 0xffff0000u;
            ph[k] = xh;
            pm[k] = xm;
            pl[k] = __float_as_uint(r - __uint_as_float(xm));
        }
        h[i] = (ph[0] >> 16) | ph[1];
        m[i] = (pm[0] >> 16) | pm[1];
        l[i] = (pl[0] >> 16) | (pl[1] & 0xffff0000u);
    }
    hi = make_uint4(h[0], h[1], h[2], h[3]);
    mid = make_uint4(m[0], m[1], m[2], m[3]);
    lo = make_uint4(l[0], l[1], l[2], l[3]);
}

// --------------------------------------------------------- one wave's tile --
// A wave takes 16 destinations.  Lane (li, lk) sums, for destination li, the
// columns of the matrix cores' fragment layout (EP consecutive columns at
// EP*lk of every block of 4*EP), so the aggregates are the products' operands
// where they are: four lanes read 64 consecutive bytes of a source row, KB
// loads cover it, and U messages of each destination are in flight together.
// Weights are the products' first operand, so a lane ends with four (16-bit
// outputs: eight) consecutive output columns of one destination per block
// (pair), and stores them directly, 64 bytes of a row by four lanes.
template <int DT, int KB>
struct GatherTile {
    typedef GatherOp<DT> Op;
    typedef GemmOp<DT> Mm;
    typedef typename Op::frag frag;
    static constexpr int EP = Op::EP, KBLK = 4 * EP, U = KB >= 16 ? 1 : 16 / KB;

    // destination li of the tile: vertex, list start and length, first sources
    struct Dest {
        int64_t v, a;
        int d;
        bool live;
    };
    static __device__ inline int64_t vertex_at(const GatherArgs& g, int64_t pos) {
        return pos < g.n ? (g.order ? (int64_t)g.order[pos] : pos) : -1;
    }
    static __device__ inline Dest dest(const GatherArgs& g, int64_t v) {
        Dest t;
        t.v = v;
        t.a = 0;
        t.d = 0;
        t.live = v >= 0 && (!g.ready || g.ready[v]);
        if (t.live) {
            t.a = g.off[v];
            t.d = (int)(g.off[v + 1] - t.a);
        }
        return t;
    }
    static __device__ inline void load_ids(const GatherArgs& g, const Dest& t, int at, uint32_t (&id)[U]) {
#pragma unroll
        for (int j = 0; j < U; j++) id[j] = at + j < t.d ? g.src[t.a + at + j] : 0u;
    }
    static __device__ inline frag piece(const GatherArgs& g, int64_t u, int kb, int lk) {
        const char* X = static_cast<const char*>(g.X);
        return *reinterpret_cast<const frag*>(X + u * ((int64_t)g.K * (16 / EP)) + (kb * 4 + lk) * 16);
    }
    static __device__ inline int longest(int d) {  // of the wave's destinations
#pragma unroll
        for (int o = 8; o >= 1; o >>= 1) d = max(d, __shfl_xor(d, o, 64));
        return __builtin_amdgcn_readfirstlane(d);
    }
    // agg = the destination's weighted sum (GraphSAGE: its mean; otherwise
    // with the vertex's own message).  Rows are added at g.scale, a power of
    // two no larger than one over the longest list and the vertex itself, so
    // that a sum of large inputs does not overflow before the linear map; the
    // mean, or the output (store), takes it out again, exactly.
    static __device__ inline void aggregate(const GatherArgs& g, const Dest& t, int dmax, int lk, uint32_t (&id)[U],
                                            float (&agg)[KB][EP]) {
        const bool partial = g.K != KB * KBLK;  // some lanes' pieces lie past the row
#pragma unroll
        for (int kb = 0; kb < KB; kb++)
#pragma unroll
            for (int i = 0; i < EP; i++) agg[kb][i] = 0.f;
        for (int at = 0; at < dmax; at += U) {  // uniform over the wave
            frag r[U][KB];
            float w[U];
#pragma unroll
            for (int j = 0; j < U; j++) {
                if (at + j < t.d) {
                    w[j] = g.norm ? g.norm[id[j]] : g.scale;
#pragma unroll
                    for (int kb = 0; kb < KB; kb++)
                        if (!partial || kb * KBLK + EP * lk < g.K) r[j][kb] = piece(g, id[j], kb, lk);
                        else r[j][kb] = Mm::zero();
                }
            }
            uint32_t nid[U];
            load_ids(g, t, at + U, nid);
#pragma unroll
            for (int j = 0; j < U; j++) {
                if (at + j < t.d) {
#pragma unroll
                    for (int kb = 0; kb < KB; kb++) Op::add(w[j], r[j][kb], agg[kb]);
                }
            }
#pragma unroll
            for (int j = 0; j < U; j++) id[j] = nid[j];
        }
        if (g.sage) {
            const float sig = t.d > 0 ? g.unscale / (float)t.d : 0.0f;
#pragma unroll
            for (int kb = 0; kb < KB; kb++)
#pragma unroll
                for (int i = 0; i < EP; i++) agg[kb][i] *= sig;
        } else if (t.live) {
            const float w = g.norm ? g.norm[t.v] : g.scale;
#pragma unroll
            for (int kb = 0; kb < KB; kb++)
                if (!partial || kb * KBLK + EP * lk < g.K) Op::add(w, piece(g, t.v, kb, lk), agg[kb]);
        }
    }
    // Products of one k-block of the aggregate with NBG column blocks of
    // weights (wb(j): this lane's fragment of block j).  The large parts go
    // to acc, the small ones to acc2, which later takes the self half: two
    // chains of roundings as long as the ones of [W_agg | W_self] products
    // added at the end, not one of twice the length.
    template <int NBG, class WB>
    static __device__ inline void mul_agg(const float (&a)[EP], WB wb, floatx4 (&acc)[NBG], floatx4 (&acc2)[NBG]) {
        if constexpr (DT == TAURUS_F32) {
#pragma unroll
            for (int q = 0; q < NBG; q += 4) {
                frag b[4];
#pragma unroll
                for (int j = 0; j < 4; j++) b[j] = wb(q + j);
#pragma unroll
                for (int c = 0; c < 4; c++)
#pragma unroll
                    for (int j = 0; j < 4; j++)
                        acc[q + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            c == 0 ? b[j].x : c == 1 ? b[j].y : c == 2 ? b[j].z : b[j].w, a[c], acc[q + j], 0, 0, 0);
            }
        } else {
            uint4 hi, mid, lo;
            split_bf16(a, hi, mid, lo);
#pragma unroll
            for (int q = 0; q < NBG; q += 4) {
                frag b[4];
#pragma unroll
                for (int j = 0; j < 4; j++) b[j] = wb(q + j);
#pragma unroll
                for (int j = 0; j < 4; j++) acc2[q + j] = Mm::mma(b[j], lo, acc2[q + j]);
#pragma unroll
                for (int j = 0; j < 4; j++) acc[q + j] = Mm::mma(b[j], hi, acc[q + j]);
#pragma unroll
                for (int j = 0; j < 4; j++) acc2[q + j] = Mm::mma(b[j], mid, acc2[q + j]);
            }
        }
    }
    template <int NBG, class WB>
    static __device__ inline void mul_self(frag x, WB wb, floatx4 (&acc2)[NBG]) {
#pragma unroll
        for (int q = 0; q < NBG; q += 4) {
            frag b[4];
#pragma unroll
            for (int j = 0; j < 4; j++) b[j] = wb(q + j);
            if constexpr (DT == TAURUS_F32) {
#pragma unroll
                for (int c = 0; c < 4; c++)
#pragma unroll
                    for (int j = 0; j < 4; j++)
                        acc2[q + j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                            c == 0 ? b[j].x : c == 1 ? b[j].y : c == 2 ? b[j].z : b[j].w,
                            c == 0 ? x.x : c == 1 ? x.y : c == 2 ? x.z : x.w, acc2[q + j], 0, 0, 0);
            } else {
#pragma unroll
                for (int j = 0; j < 4; j++) acc2[q + j] = Mm::mma(b[j], x, acc2[q + j]);
            }
        }
    }
    // self row's piece of k-block kb
    static __device__ inline frag self(const GatherArgs& g, const Dest& t, int kb, int lk) {
        return t.live && kb * KBLK + EP * lk < g.K ? piece(g, t.v, kb, lk) : Mm::zero();
    }
    // first of the four output columns this lane holds of block j (gather_col)
    static __device__ inline int col(const GatherArgs& g, int j, int lk) {
        return g.pairs ? (j >> 1) * 32 + lk * 8 + (j & 1) * 4 : j * 16 + lk * 4;
    }
    // out row of the destination, columns of blocks nb0 .. nb0 + NBG - 1:
    // sums(j) gives the four of block nb0 + j.  The bias (padded to NBP
    // blocks) comes from LDS: a load from memory here would make the wave
    // wait for every older load, the next tiles' rows among them.
    template <int NBG, class Sums>
    static __device__ inline void store(const GatherArgs& g, const float* bias, const Dest& t, int nb0, int lk,
                                        Sums sums) {
        if (!t.live) return;
        const float out_scale = g.sage ? 1.0f : g.unscale;
        const float phi = g.norm ? out_scale / sqrtf((float)(t.d + 1)) : out_scale;
        auto value = [&](int j) {
            const int c = col(g, nb0 + j, lk);
            const floatx4 x = sums(j);
            const float4 b = *reinterpret_cast<const float4*>(bias + c);
            float4 z = make_float4(fmaf(phi, x[0], b.x), fmaf(phi, x[1], b.y), fmaf(phi, x[2], b.z),
                                   fmaf(phi, x[3], b.w));
            if (g.relu) {
                z.x = fmaxf(z.x, 0.f); z.y = fmaxf(z.y, 0.f);
                z.z = fmaxf(z.z, 0.f); z.w = fmaxf(z.w, 0.f);
            }
            return z;
        };
        if (g.pairs && (g.d_o & 7) == 0) {        // 16-bit outputs: eight columns a store
#pragma unroll
            for (int j = 0; j < NBG; j += 2) {
                const int c = col(g, nb0 + j, lk);
                if (c < g.d_o) {
                    const uint2 a = pack_out4(g.out_dtype, value(j)), b = pack_out4(g.out_dtype, value(j + 1));
                    *reinterpret_cast<uint4*>(static_cast<uint16_t*>(g.out) + t.v * g.d_o + c) =
                        make_uint4(a.x, a.y, b.x, b.y);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < NBG; j++) {
                const int c = col(g, nb0 + j, lk);
                if (c < g.d_o) store_out4(g.out, g.out_dtype, t.v * g.d_o + c, value(j));
            }
        }
    }
};

// Registers of the aggregates and the two accumulator sets decide how many
// waves a SIMD holds (the loads in flight and operands take about 70 more).
template <int DT, int KB, int NBG>
constexpr int gather_waves() {
    return KB * GatherOp<DT>::EP + 8 * NBG <= 64 ? 3 : 2;
}

// ------------------------------------------------- weights resident in LDS --
// Persistent: a workgroup holds its weights (at most RESIDENT_LDS bytes) in
// LDS and its waves take tiles on their own, without a barrier, so that some
// gather while others multiply.  The next tile's vertices, list bounds and
// first sources are requested before this tile's products.
//
// Positions [0, end) of g.order.  HALVES: both halves of a GraphSAGE layer
// (g.partial null), the aggregate of the other families, or, where the two
// halves' weights do not fit together, the aggregate's products alone,
// written to g.partial [end][d_o] for k_self_resident to add.
constexpr int RESIDENT_LDS = 144 << 10;
template <int DT, int KB, int NBG, int WAVES>
__global__ __launch_bounds__(256 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES)))
void k_gather_resident(GatherArgs g, int64_t end) {
    typedef GatherTile<DT, KB> Tile;
    typedef typename Tile::frag frag;
    constexpr int EP = Tile::EP, U = Tile::U;
    extern __shared__ uint4 lds_raw[];
    __shared__ float sBias[NBG * 16];
    frag* sW = reinterpret_cast<frag*>(lds_raw);
    for (int i = threadIdx.x; i < NBG * 16; i += blockDim.x) sBias[i] = i < g.d_o ? g.bias[i] : 0.f;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int kbn = (g.K + Tile::KBLK - 1) / Tile::KBLK;
    const bool self = g.sage && !g.partial;
    const int nfrag = kbn * (self ? 2 : 1) * NBG * 64;     // NBP = NBG
    for (int i = threadIdx.x; i < nfrag; i += blockDim.x) sW[i] = static_cast<const frag*>(g.W)[i];
    __syncthreads();
    const int nw = blockDim.x >> 6;
    const int64_t stride = (int64_t)gridDim.x * nw * 16;
    // consecutive tiles go to different workgroups: in the order by length the
    // first ones hold the longest lists, and a compute unit that took them all
    // was the kernel's tail (1M vertices, 4M edges, fanout 512, 64 -> 64 fp32:
    // 1.18 ms, 0.82 ms this way)
    int64_t pos = ((int64_t)(threadIdx.x >> 6) * gridDim.x + blockIdx.x) * 16 + li;
    auto vertex = [&](int64_t p) { return p < end ? Tile::vertex_at(g, p) : (int64_t)-1; };
    typename Tile::Dest t = Tile::dest(g, vertex(pos));
    uint32_t id[U];
    Tile::load_ids(g, t, 0, id);
    int64_t vn = vertex(pos + stride);
    for (; pos - li < end; pos += stride) {       // uniform over the wave
        const typename Tile::Dest tn = Tile::dest(g, vn);
        vn = vertex(pos + 2 * stride);
        float agg[KB][EP];
        Tile::aggregate(g, t, Tile::longest(t.d), lk, id, agg);
        Tile::load_ids(g, tn, 0, id);
        floatx4 acc[NBG], acc2[NBG];
#pragma unroll
        for (int j = 0; j < NBG; j++) acc[j] = acc2[j] = floatx4{0.f, 0.f, 0.f, 0.f};
        auto weights = [&](int st) {
            const frag* w = sW + st * (NBG * 64) + lane;
            return [=](int j) { return w[j * 64]; };
        };
        frag x = Tile::Mm::zero();
        if (self) x = Tile::self(g, t, 0, lk);
#pragma unroll
        for (int kb = 0; kb < KB; kb++)
            if (kb < kbn) Tile::template mul_agg<NBG>(agg[kb], weights(kb), acc, acc2);
        if (self) {
            for (int kb = 0; kb < kbn; kb++) {
                const frag xn = kb + 1 < kbn ? Tile::self(g, t, kb + 1, lk) : x;
                Tile::template mul_self<NBG>(x, weights(kbn + kb), acc2);
                x = xn;
            }
        }
        if (g.partial) {
            if (t.live) {
#pragma unroll
                for (int j = 0; j < NBG; j++) {
                    const int c = Tile::col(g, j, lk);
                    if (c < g.d_o) *reinterpret_cast<floatx4*>(g.partial + pos * g.d_o + c) = acc[j] + acc2[j];
                }
            }
        } else {
            Tile::template store<NBG>(g, sBias, t, 0, lk, [&](int j) { return acc[j] + acc2[j]; });
        }
        t = tn;
    }
}

// GraphSAGE: the self half of positions [begin, n) of g.order, added to the
// aggregate's products in g.partial for positions before `parts`, the whole
// value past them (destinations without messages).  A streaming kernel: the
// rows of the next tile (two where registers allow) are in flight while one
// is multiplied.  6.7M rows 128 -> 256 bf16: 2.45 ms with the bias loaded from
// memory and 8-byte stores of integer-rounded values, 1.16 ms as it is.
template <int DT, int KB, int NBG, int WAVES>
__global__ __launch_bounds__(256 * WAVES) __attribute__((amdgpu_waves_per_eu(WAVES)))
void k_self_resident(GatherArgs g, int64_t begin, int64_t parts) {
    typedef GatherTile<DT, KB> Tile;
    typedef typename Tile::frag frag;
    extern __shared__ uint4 lds_raw[];
    __shared__ float sBias[NBG * 16];
    frag* sW = reinterpret_cast<frag*>(lds_raw);
    for (int i = threadIdx.x; i < NBG * 16; i += blockDim.x) sBias[i] = i < g.d_o ? g.bias[i] : 0.f;
    const int lane = threadIdx.x & 63, li = lane & 15, lk = lane >> 4;
    const int kbn = (g.K + Tile::KBLK - 1) / Tile::KBLK;
    const int nfrag = kbn * NBG * 64;
    for (int i = threadIdx.x; i < nfrag; i += blockDim.x) sW[i] = static_cast<const frag*>(g.W)[nfrag + i];
    __syncthreads();
    const int nw = blockDim.x >> 6;
    const int64_t stride = (int64_t)gridDim.x * nw * 16;
    int64_t pos = begin + ((int64_t)blockIdx.x * nw + (threadIdx.x >> 6)) * 16 + li;
    auto dest = [&](int64_t v) {                  // d stays 0: nothing here depends on it
        typename Tile::Dest t;
        t.v = v;
        t.a = 0;
        t.d = 0;
        t.live = v >= 0 && (!g.ready || g.ready[v]);
        return t;
    };
    // rows of the next DEPTH tiles in flight
    constexpr int DEPTH = KB <= 4 ? 2 : 1;
    frag x[DEPTH + 1][KB];
    typename Tile::Dest t[DEPTH + 1];
    auto rows = [&](int q) {
#pragma unroll
        for (int kb = 0; kb < KB; kb++) x[q][kb] = Tile::self(g, t[q], kb, lk);
    };
#pragma unroll
    for (int q = 0; q < DEPTH; q++) {
        t[q] = dest(Tile::vertex_at(g, pos + q * stride));
        rows(q);
    }
    int64_t vn = Tile::vertex_at(g, pos + DEPTH * stride);
    for (; pos - li < g.n; pos += stride) {       // uniform over the wave
        // the parts first: loads return in order, and these are needed first
        floatx4 part[NBG];
        const bool add = pos - li < parts;        // uniform
        if (add) {
#pragma unroll
            for (int j = 0; j < NBG; j++) {
                const int c = Tile::col(g, j, lk);
                part[j] = floatx4{0.f, 0.f, 0.f, 0.f};
                if (pos < parts && c < g.d_o) part[j] = *reinterpret_cast<const floatx4*>(g.partial + pos * g.d_o + c);
            }
        }
        t[DEPTH] = dest(vn);
        vn = Tile::vertex_at(g, pos + (DEPTH + 1) * stride);
        rows(DEPTH);
        floatx4 own[NBG];
#pragma unroll
        for (int j = 0; j < NBG; j++) own[j] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kb = 0; kb < KB; kb++) {
            if (kb < kbn) {
                const frag* w = sW + kb * (NBG * 64) + lane;
                Tile::template mul_self<NBG>(x[0][kb], [=](int j) { return w[j * 64]; }, own);
            }
        }
        if (add) {
#pragma unroll
            for (int j = 0; j < NBG; j++) own[j] += part[j];
        }
        Tile::template store<NBG>(g, sBias, t[0], 0, lk, [&](int j) { return own[j]; });
#pragma unroll
        for (int q = 0; q < DEPTH; q++) {
            t[q] = t[q + 1];
#pragma unroll
            for (int kb = 0; kb < KB; kb++) x[q][kb] = x[q + 1][kb];
        }
    }
}

// ---------------------------------------------- weights streamed through LDS --
// Weights that do not fit, and layers of too few tiles to pay for loading
// them whole: a workgroup of four waves takes 64 destinations, and the
// weights pass through two LDS buffers of GS k-blocks each, the next stage's
// in registers while this one's products run (one k-block a stage left every
// stage waiting for its loads: 19 us a workgroup at 256 -> 172, of which the
// products take 8).
constexpr int GS = 2;
template <int DT, int KB, int NBG, int WAVES>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(WAVES)))
void k_gather_streamed(GatherArgs g) {
    typedef GatherTile<DT, KB> Tile;
    typedef typename Tile::frag frag;
    constexpr int EP = Tile::EP, U = Tile::U, SF = GS * NBG * 64, PER = SF / 256;
    __shared__ frag sB[2][SF];
    __shared__ float sBias[1024];                     // d_o <= 1024, whole column groups of it
    static_assert(1024 % (NBG * 16) == 0, "the last group's columns stay inside sBias");
    const int tid = threadIdx.x, lane = tid & 63, li = lane & 15, lk = lane >> 4;
    const frag* __restrict__ Wp = static_cast<const frag*>(g.W);
    const int kbn = (g.K + Tile::KBLK - 1) / Tile::KBLK;
    const int ast = (kbn + GS - 1) / GS;              // stages of a half
    const int nst = ast * (g.sage ? 2 : 1);
    auto load_w = [&](int st, int nb0, frag (&r)[PER]) {
        const int half = st >= ast, kb0 = (half ? st - ast : st) * GS;
#pragma unroll
        for (int q = 0; q < PER; q++) {
            const int i = q * 256 + tid, kb = kb0 + i / (NBG * 64), nb = nb0 + (i / 64) % NBG;
            r[q] = kb < kbn && nb < g.NBP ? Wp[((int64_t)(half * kbn + kb) * g.NBP + nb) * 64 + (i & 63)]
                                          : Tile::Mm::zero();
        }
    };
    for (int i = tid; i < g.NBP * 16; i += 256) sBias[i] = i < g.d_o ? g.bias[i] : 0.f;
    frag rw[PER];
    load_w(0, 0, rw);
    const typename Tile::Dest t =
        Tile::dest(g, Tile::vertex_at(g, (int64_t)blockIdx.x * 64 + (tid >> 6) * 16 + li));
    uint32_t id[U];
    Tile::load_ids(g, t, 0, id);
    float agg[KB][EP];
    Tile::aggregate(g, t, Tile::longest(t.d), lk, id, agg);
    for (int nb0 = 0; nb0 < g.NBP; nb0 += NBG) {      // uniform
        floatx4 acc[NBG], acc2[NBG];
#pragma unroll
        for (int j = 0; j < NBG; j++) acc[j] = acc2[j] = floatx4{0.f, 0.f, 0.f, 0.f};
        if (nb0 > 0) load_w(0, nb0, rw);
#pragma unroll
        for (int q = 0; q < PER; q++) sB[0][q * 256 + tid] = rw[q];
        __syncthreads();
        int st = 0;
        auto weights = [&](int k) {                   // k-block k of the current stage
            const frag* w = &sB[st & 1][k * NBG * 64 + lane];
            return [=](int j) { return w[j * 64]; };
        };
        auto next = [&]() {                           // the other buffer was last read before the last barrier
            if (st + 1 < nst) {
#pragma unroll
                for (int q = 0; q < PER; q++) sB[(st + 1) & 1][q * 256 + tid] = rw[q];
            }
            __syncthreads();
            st++;
        };
#pragma unroll
        for (int k0 = 0; k0 < KB; k0 += GS) {
            if (k0 < kbn) {                           // uniform
                if (st + 1 < nst) load_w(st + 1, nb0, rw);
#pragma unroll
                for (int k = 0; k < GS; k++) Tile::template mul_agg<NBG>(agg[k0 + k], weights(k), acc, acc2);
                next();
            }
        }
        if (g.sage) {
            frag x[GS];
#pragma unroll
            for (int k = 0; k < GS; k++) x[k] = Tile::self(g, t, k, lk);
            for (int k0 = 0; k0 < kbn; k0 += GS) {
                frag xn[GS];
                if (st + 1 < nst) load_w(st + 1, nb0, rw);
#pragma unroll
                for (int k = 0; k < GS; k++) xn[k] = Tile::self(g, t, k0 + GS + k, lk);
#pragma unroll
                for (int k = 0; k < GS; k++) Tile::template mul_self<NBG>(x[k], weights(k), acc2);
#pragma unroll
                for (int k = 0; k < GS; k++) x[k] = xn[k];
                next();
            }
        }
        Tile::template store<NBG>(g, sBias, t, nb0, lk, [&](int j) { return acc[j] + acc2[j]; });
    }
}

template <int DT, int KB, int NBG>
static void launch_resident(const GatherArgs& g, int cus, hipStream_t s) {
    constexpr int per = gather_waves<DT, KB, NBG>(), waves = 4 * per;
    const size_t half = (size_t)(ceil_div(g.K, GatherTile<DT, KB>::KBLK) * NBG) << 10;
    auto set_lds = [](const void* kernel, size_t bytes) {
        TAURUS_HIP(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes));
    };
    auto blocks = [&](int64_t positions) { return (unsigned)std::min<int64_t>(cus, ceil_div(positions, 16 * waves)); };
    // a GraphSAGE layer's destinations without messages take the self half
    // alone, and all of them do when the halves do not fit together
    const int64_t nz = g.sage ? g.nonzero : g.n;
    const bool split = g.sage && g.partial;
    if (nz > 0) {
        const size_t lds = g.sage && !split ? 2 * half : half;
        auto kernel = k_gather_resident<DT, KB, NBG, per>;
        set_lds(reinterpret_cast<const void*>(kernel), lds);
        kernel<<<blocks(nz), 64 * waves, lds, s>>>(g, nz);
        TAURUS_CHECK_LAUNCH();
    }
    const int64_t begin = split ? 0 : nz;
    if (g.sage && begin < g.n) {
        auto kernel = k_self_resident<DT, KB, NBG, 2>;
        set_lds(reinterpret_cast<const void*>(kernel), half);
        kernel<<<(unsigned)std::min<int64_t>(cus, ceil_div(g.n - begin, 16 * 8)), 512, half, s>>>(g, begin,
                                                                                               split ? nz : 0);
        TAURUS_CHECK_LAUNCH();
    }
}

// Resident weights: when a half fits, and every wave has at least about four
// tiles to spread their loading over.
static bool gather_resident(const GatherArgs& g, int dtype, int cus) {
    const int64_t kbn = ceil_div(g.K, dtype == TAURUS_F32 ? 16 : 32);
    return g.order && g.NBP <= 16 && ((kbn * g.NBP) << 10) <= RESIDENT_LDS && g.n >= (int64_t)cus * 12 * 16 * 4;
}

static int compute_units() {
    int dev = 0, cus = 0;
    TAURUS_HIP(hipGetDevice(&dev));
    TAURUS_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    return std::max(1, cus);
}

int64_t gather_partial_rows(const GatherArgs& g, int dtype) {
    const int64_t kbn = ceil_div(g.K, dtype == TAURUS_F32 ? 16 : 32);
    if (!g.sage || !gather_resident(g, dtype, compute_units()) || ((2 * kbn * g.NBP) << 10) <= RESIDENT_LDS) return 0;
    return g.nonzero;
}

template <int DT, int KB>
static void launch_gather(const GatherArgs& g, hipStream_t s) {
    const int cus = compute_units();
    if (gather_resident(g, DT, cus)) {
        if (g.NBP <= 4) launch_resident<DT, KB, 4>(g, cus, s);
        else if (g.NBP <= 8) launch_resident<DT, KB, 8>(g, cus, s);
        else if (g.NBP <= 12) launch_resident<DT, KB, 12>(g, cus, s);
        else launch_resident<DT, KB, 16>(g, cus, s);
    } else {
        const unsigned blocks = (unsigned)ceil_div(g.n, 64);
        if (g.NBP == 4) k_gather_streamed<DT, KB, 4, gather_waves<DT, KB, 4>()><<<blocks, 256, 0, s>>>(g);
        else k_gather_streamed<DT, KB, 8, gather_waves<DT, KB, 8>()><<<blocks, 256, 0, s>>>(g);
        TAURUS_CHECK_LAUNCH();
    }
}

void gather_layer(const GatherArgs& g, int dtype, hipStream_t s) {
    if (g.n <= 0) return;
    if (g.K <= 0 || g.K > GATHER_MAX_K || g.K % (dtype == TAURUS_F32 ? 4 : 8) || g.d_o % 4)
        fail(TAURUS_E_INVALID, "gather: widths %d, %d", g.K, g.d_o);
    const int kb = (int)ceil_div(g.K, dtype == TAURUS_F32 ? 16 : 32);
    if (dtype == TAURUS_F32) {
        if (kb <= 4) launch_gather<TAURUS_F32, 4>(g, s);
        else if (kb <= 8) launch_gather<TAURUS_F32, 8>(g, s);
        else launch_gather<TAURUS_F32, 16>(g, s);
    } else if (dtype == TAURUS_BF16) {
        if (kb <= 2) launch_gather<TAURUS_BF16, 2>(g, s);
        else if (kb <= 4) launch_gather<TAURUS_BF16, 4>(g, s);
        else launch_gather<TAURUS_BF16, 8>(g, s);
    } else {
        fail(TAURUS_E_INVALID, "gather: dtype %d", dtype);
    }
}

// ---------------------------------------------------------------- weights --

int gather_blocks_n(int d_o) { return (int)ceil_div(d_o, 64) * 4; }

static uint32_t bits_of(uint16_t x) { return x; }
static uint32_t bits_of(float x) {
    uint32_t u;
    std::memcpy(&u, &x, 4);
    return u;
}

// Fragments of a row-major W (row stride ld) [K][d_o] after those already in
// packed: block (kb, nb) holds, for lane (i, lk), the EP consecutive k at
// kb*KBLK + EP*lk of column 16*nb + i, or with pairs (16-bit outputs, so that
// a lane's columns of two blocks make one 16-byte store) column
// 32*(nb/2) + 8*(i/4) + 4*(nb%2) + i%4; zeros past K and d_o.  True when every
// packed value is finite (exp: the type's exponent bits).
template <class T, class Cvt>
static bool pack(const float* W, int ld, int K, int d_o, bool pairs, int ep, uint32_t exp, Cvt cvt,
                 std::vector<T>& packed) {
    const int kbn = (int)ceil_div(K, 4 * ep), nbp = gather_blocks_n(d_o);
    const size_t base = packed.size();
    packed.resize(base + (size_t)kbn * nbp * 64 * ep, T(0));
    T* p = packed.data() + base;
    bool finite = true;
    for (int kb = 0; kb < kbn; kb++)
        for (int nb = 0; nb < nbp; nb++)
            for (int l = 0; l < 64; l++, p += ep) {
                const int i = l & 15, k0 = kb * 4 * ep + ep * (l >> 4);
                const int col = pairs ? 32 * (nb >> 1) + 8 * (i >> 2) + 4 * (nb & 1) + (i & 3) : 16 * nb + i;
                if (col >= d_o) continue;
                for (int c = 0; c < ep && k0 + c < K; c++) {
                    p[c] = cvt(W[(size_t)(k0 + c) * ld + col]);
                    finite &= (bits_of(p[c]) & exp) != exp;
                }
            }
    return finite;
}

bool gather_pack_f32(const float* W, int ld, int K, int d_o, bool pairs, std::vector<float>& packed) {
    return pack(W, ld, K, d_o, pairs, 4, 0x7f800000u, [](float x) { return x; }, packed);
}
bool gather_pack_bf16(const float* W, int ld, int K, int d_o, bool pairs, std::vector<uint16_t>& packed) {
    return pack(W, ld, K, d_o, pairs, 8, 0x7f80u, [](float x) { return host_f32_to_bf16(x); }, packed);
}

// -------------------------------------------------------------- row table --

// One word a thread while the chunk fills the grid (four, requested before
// the first store: 7.5 -> 20 us for 65,536 rows of 256 bytes).
template <class W>
__global__ __launch_bounds__(256) void k_copy_rows(const W* __restrict__ in, W* __restrict__ out, int64_t words) {
    const int64_t stride = (int64_t)gridDim.x * 256;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += stride) out[i] = in[i];
}

// rows of a multiple of 16 bytes; x may be aligned to 4 only
void gather_copy_rows(const void* x, void* table, int64_t bytes, hipStream_t s) {
    if (bytes <= 0) return;
    const bool wide = reinterpret_cast<uintptr_t>(x) % 16 == 0;
    const int64_t words = bytes / (wide ? 16 : 4);
    const int64_t blocks = std::min<int64_t>(ceil_div(words, 256), 4096);
    if (wide)
        k_copy_rows<uint4><<<(unsigned)blocks, 256, 0, s>>>(static_cast<const uint4*>(x), static_cast<uint4*>(table),
                                                            words);
    else
        k_copy_rows<uint32_t><<<(unsigned)blocks, 256, 0, s>>>(static_cast<const uint32_t*>(x),
                                                               static_cast<uint32_t*>(table), words);
    TAURUS_CHECK_LAUNCH();
}

// ------------------------------------------------------------------ order ----

// Destinations in descending order of their list lengths, stably, so that
// the 16 of a wave have lists of about one length (a wave takes as many
// rounds as its longest list needs) and the long ones start first.
__global__ void k_length_keys(const int64_t* __restrict__ off, int64_t n, int k, uint32_t* __restrict__ keys,
                              uint32_t* __restrict__ vals) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= n) return;
    keys[v] = (uint32_t)(k - (int)(off[v + 1] - off[v]));
    vals[v] = (uint32_t)v;
}

uint32_t* gather_order(const int64_t* off, int64_t n, int k, Arena& arena, Arena& tmp, int* bad, int bad_bit,
                       hipStream_t s) {
    SortBuffers32 sb{{tmp.alloc<uint32_t>(n, "list lengths"), tmp.alloc<uint32_t>(n, "list lengths (ping-pong)")},
                     {arena.alloc<uint32_t>(n, "destination order"),
                      arena.alloc<uint32_t>(n, "destination order (ping-pong)")},
                     0};
    k_length_keys<<<(unsigned)ceil_div(n, 256), 256, 0, s>>>(off, n, k, sb.keys[0], sb.vals[0]);
    TAURUS_CHECK_LAUNCH();
    radix_sort_u32(sb, n, bits_for(k), tmp, s, bad, bad_bit);
    arena.free_ptr(sb.vals[1 - sb.cur]);
    return sb.vals[sb.cur];
}

// ------------------------------------------------------------- GCN norms ----

// A hub's counter takes one atomic from every list that holds it, about 9 ns
// each, one after the other (2M lists with one source in common: 18 ms).  A
// workgroup adds up its tile of entries in LDS first: a source takes one of
// its two slots of a table by its first entry there and leaves in one atomic;
// entries that find both slots taken go to memory themselves.  A frequent
// source is among a tile's first entries, when nearly every slot is free.
constexpr int SRC_TILE = 4096;
__global__ __launch_bounds__(256) void k_source_counts(const uint32_t* __restrict__ src, int64_t kept,
                                                       int32_t* __restrict__ deg) {
    constexpr uint32_t FREE = ~0u;  // no source: IDs are below 2^31
    __shared__ uint32_t tag[SRC_TILE];
    __shared__ int32_t count[SRC_TILE];
    for (int i = threadIdx.x; i < SRC_TILE; i += 256) {
        tag[i] = FREE;
        count[i] = 0;
    }
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * SRC_TILE;
    uint32_t u[SRC_TILE / 256];
#pragma unroll
    for (int r = 0; r < SRC_TILE / 256; r++) {
        const int64_t i = base + r * 256 + threadIdx.x;
        u[r] = i < kept ? src[i] : FREE;
    }
#pragma unroll
    for (int r = 0; r < SRC_TILE / 256; r++) {
        if (u[r] == FREE) continue;
        int slot = (int)((u[r] * 0x9e3779b1u) >> 20);   // [0, SRC_TILE)
        uint32_t t = atomicCAS(&tag[slot], FREE, u[r]);
        if (t != FREE && t != u[r]) {
            slot ^= 1;
            t = atomicCAS(&tag[slot], FREE, u[r]);
        }
        if (t == FREE || t == u[r]) atomicAdd(&count[slot], 1);
        else atomicAdd(&deg[u[r]], 1);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < SRC_TILE; i += 256)
        if (count[i]) atomicAdd(&deg[tag[i]], count[i]);
}
static_assert(SRC_TILE == 1 << 12, "the hash keeps 12 bits");
// counts become norms in place
__global__ void k_source_norms(int64_t n, float scale, float* __restrict__ norm) {
    const int64_t u = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (u < n) norm[u] = scale / sqrtf((float)(__float_as_int(norm[u]) + 1));
}

void gather_norms(const uint32_t* src, int64_t kept, int64_t n, float scale, float* norm, hipStream_t s) {
    fill_i32(reinterpret_cast<int32_t*>(norm), n, 0, s);
    if (kept > 0) {
        k_source_counts<<<(unsigned)ceil_div(kept, SRC_TILE), 256, 0, s>>>(src, kept, reinterpret_cast<int32_t*>(norm));
        TAURUS_CHECK_LAUNCH();
    }
    k_source_norms<<<(unsigned)ceil_div(n, 256), 256, 0, s>>>(n, scale, norm);
    TAURUS_CHECK_LAUNCH();
}

// -------------------------------------------------- counts and readiness ----

// What the chunk index of these lists would hold (taurus_stats): segments
// (destination, source chunk), vertices with a segment from their own chunk,
// and the work units of segments of at most short_len and piece_len slots.
// The n destinations order[0 .. n) (null: 0 .. n); without messages they
// count nothing.
constexpr int LIST_WALK = 64;
__global__ __launch_bounds__(256) void k_list_counts(const int64_t* __restrict__ off,
                                                     const uint32_t* __restrict__ src,
                                                     const uint32_t* __restrict__ order, int64_t n, uint32_t C,
                                                     int short_len, int piece_len,
                                                     unsigned long long* __restrict__ out) {
    __shared__ unsigned int part[4][LIST_COUNTS];
    unsigned int c[LIST_COUNTS] = {};
    const int lane = threadIdx.x & 63;
    // a segment of len messages from chunk, of a vertex whose own chunk is own
    auto segment = [&](int len, uint32_t chunk, uint32_t own) {
        const int slots = len + (chunk == own ? 1 : 0);
        c[LC_SEGMENTS]++;
        c[LC_OWN] += chunk == own;
        if (slots <= short_len) {
            c[LC_SHORT]++;
        } else {
            const int pieces = (slots + piece_len - 1) / piece_len;
            c[LC_WAVE] += pieces;
            c[LC_SPLIT] += pieces > 1;
        }
    };
    const int64_t stride = (int64_t)gridDim.x * 256;
    const int64_t wave = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    for (int64_t p0 = 0; p0 < n; p0 += stride) {
        // the longest lists, first in the order, one to a wave
        const int64_t p = p0 + (order && p0 == 0 ? lane * (stride >> 6) + wave : wave * 64 + lane);
        int64_t a = 0;
        int d = 0;
        uint32_t own = 0;
        if (p < n) {
            const int64_t v = order ? (int64_t)order[p] : p;
            a = off[v];
            d = (int)(off[v + 1] - a);
            own = (uint32_t)v / C;
        }
        // a lane walks a list of at most LIST_WALK sources, four loads in flight
        if (d <= LIST_WALK) {
            uint32_t chunk = 0;
            int len = 0;
            for (int t = 0; t < d; t += 4) {
                uint32_t u[4];
#pragma unroll
                for (int j = 0; j < 4; j++) u[j] = t + j < d ? src[a + t + j] : 0u;
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    if (t + j >= d) break;
                    const uint32_t cu = u[j] / C;
                    if (cu != chunk) {
                        if (len) segment(len, chunk, own);
                        chunk = cu;
                        len = 0;
                    }
                    len++;
                }
            }
            if (len) segment(len, chunk, own);
        }
        // the wave takes the longer ones together, 64 sources a step: a lane
        // whose source starts a segment counts it once the next start is known
        for (uint64_t todo = __ballot(d > LIST_WALK); todo; todo &= todo - 1) {  // uniform
            const int l = __builtin_ctzll(todo);
            const int64_t la = __shfl(a, l);
            const int ld = __shfl(d, l);
            const uint32_t lown = (uint32_t)__shfl((int)own, l);
            uint32_t open = 0;     // the segment that reaches into this step
            int from = -1;
            for (int t = 0; t < ld; t += 64) {
                const uint32_t cu = t + lane < ld ? src[la + t + lane] / C : ~0u;
                uint32_t before = (uint32_t)__shfl_up((int)cu, 1);
                if (lane == 0) before = from < 0 ? ~cu : open;
                const uint64_t heads = __ballot(cu != ~0u && cu != before);
                if (!heads) continue;
                const int first = __builtin_ctzll(heads), last = 63 - __builtin_clzll(heads);
                if (from >= 0 && lane == 0) segment(t + first - from, open, lown);
                if (((heads >> lane) & 1) && lane < last) {
                    const uint64_t next = heads & ~((2ull << lane) - 1ull);
                    segment(__builtin_ctzll(next) - lane, cu, lown);
                }
                open = (uint32_t)__shfl((int)cu, last);
                from = t + last;
            }
            if (lane == 0) segment(ld - from, open, lown);
        }
    }
#pragma unroll
    for (int k = 0; k < LIST_COUNTS; k++) {
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) c[k] += __shfl_xor(c[k], o, 64);
        if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6][k] = c[k];
    }
    __syncthreads();
    if (threadIdx.x < LIST_COUNTS) {
        const int k = threadIdx.x;
        const unsigned long long t = (unsigned long long)part[0][k] + part[1][k] + part[2][k] + part[3][k];
        if (t) atomicAdd(&out[k], t);
    }
}

void gather_list_counts(const int64_t* off, const uint32_t* src, const uint32_t* order, int64_t n, int64_t C,
                        int short_len, int piece_len, unsigned long long* out, hipStream_t s) {
    fill_i32(reinterpret_cast<int32_t*>(out), 2 * LIST_COUNTS, 0, s);
    const unsigned blocks = (unsigned)std::max<int64_t>(1, std::min<int64_t>(ceil_div(n, 256), 2048));
    k_list_counts<<<blocks, 256, 0, s>>>(off, src, order, n, (uint32_t)C, short_len, piece_len, out);
    TAURUS_CHECK_LAUNCH();
}

// ready[v] = 1 when v's own chunk and every chunk its messages come from
// have been pushed; *left = vertices that are not
__global__ __launch_bounds__(256) void k_list_ready(const int64_t* __restrict__ off,
                                                    const uint32_t* __restrict__ src, int64_t n, uint32_t C,
                                                    const uint8_t* __restrict__ pushed, uint8_t* __restrict__ ready,
                                                    unsigned long long* __restrict__ left) {
    const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
    bool ok = v < n && pushed[(uint32_t)v / C];
    if (ok)
        for (int64_t t = off[v]; t < off[v + 1] && ok; t++) ok = pushed[src[t] / C] != 0;
    if (v < n) ready[v] = ok ? 1 : 0;
    const uint64_t b = __ballot(v < n && !ok);
    if ((threadIdx.x & 63) == 0 && b) atomicAdd(left, (unsigned long long)__popcll(b));
}

void gather_ready(const int64_t* off, const uint32_t* src, int64_t n, int64_t C, const uint8_t* pushed,
                  uint8_t* ready, unsigned long long* left, hipStream_t s) {
    fill_i32(reinterpret_cast<int32_t*>(left), 2, 0, s);
    k_list_ready<<<(unsigned)ceil_div(n, 256), 256, 0, s>>>(off, src, n, (uint32_t)C, pushed, ready, left);
    TAURUS_CHECK_LAUNCH();
}

}  // namespace taurus
