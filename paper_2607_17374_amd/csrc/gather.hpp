// Sampled layers kept in core, aggregated from their kept in-edge lists
// (gather.hip).
#pragma once

#include "internal.hpp"

namespace taurus {

constexpr int GATHER_MAX_K = 256;   // input width a wave's aggregates hold in registers

struct GatherArgs {
    const void* X;          // [n][K] source rows
    int64_t n;
    int K;
    const int64_t* off;     // [n+1] kept in-edges before each destination
    const uint32_t* src;    // their sources, ascending within a destination
    const void* W;          // packed weights: the aggregate's, then (sage) the self half's
    int NBP;                // 16-column blocks per k-block of W
    const float* bias;      // [d_o]
    const float* norm;      // GCN: d^_out(u)^-1/2 of the sampled graph, times scale, else null
    float scale, unscale;   // messages are summed at scale (GatherTile::aggregate); 1 / scale
    void* out;              // [n][d_o]
    int d_o, out_dtype, relu, sage;
    const uint8_t* ready;   // null: every destination
    const uint32_t* order;  // [n] the order destinations are taken in, or null
    int64_t nonzero;        // of which the first have messages (with order)
    float* partial;         // [gather_partial_rows][d_o], or null when that is 0
    int pairs;              // W's columns are packed for 16-bit outputs
};

uint16_t host_f32_to_bf16(float f);   // round to nearest even (gemm.hip)
// host weights [K][d_o] (row stride ld) appended as matrix-core fragments;
// false when one is not finite in the packed type
bool gather_pack_f32(const float* W, int ld, int K, int d_o, bool pairs, std::vector<float>& packed);
bool gather_pack_bf16(const float* W, int ld, int K, int d_o, bool pairs, std::vector<uint16_t>& packed);
int gather_blocks_n(int d_o);
// rows of g.partial the layer needs (0: none), from every other member
int64_t gather_partial_rows(const GatherArgs& g, int dtype);
void gather_layer(const GatherArgs& g, int dtype, hipStream_t s);
void gather_copy_rows(const void* x, void* table, int64_t bytes, hipStream_t s);

// destinations by descending list length (k at most); order from arena
constexpr int64_t GATHER_ORDER_MIN = 1 << 18;
uint32_t* gather_order(const int64_t* off, int64_t n, int k, Arena& arena, Arena& tmp, int* bad, int bad_bit,
                       hipStream_t s);
// norm[u] = scale * (in-edges of the lists with source u + 1)^-1/2
void gather_norms(const uint32_t* src, int64_t kept, int64_t n, float scale, float* norm, hipStream_t s);

enum { LC_SEGMENTS, LC_OWN, LC_SHORT, LC_WAVE, LC_SPLIT, LIST_COUNTS };
void gather_list_counts(const int64_t* off, const uint32_t* src, const uint32_t* order, int64_t n, int64_t C,
                        int short_len, int piece_len, unsigned long long* out, hipStream_t s);
void gather_ready(const int64_t* off, const uint32_t* src, int64_t n, int64_t C, const uint8_t* pushed,
                  uint8_t* ready, unsigned long long* left, hipStream_t s);

}  // namespace taurus
