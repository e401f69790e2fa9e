// Internal interface between the serving scheduler (serve.cpp) and the
// persistent multi-session kernels (k_serve.hip).
#pragma once

#include <vector>

#include "npm_internal.h"

namespace npm {

constexpr int kMaxRoundRequests = 256;

// One request of a round as the scheduler hands it to the launcher.
struct ServeRequest {
    int kind;                    // 0 query, 1 train
    int64_t n;
    const float *pos, *dir, *rad, *spdf;
    float *lobes, *pdf, *sdir, *spdf_out;
    double *stats;
    uint64_t seed;
    uint32_t stream_id;
    npm_ctx *ctx;
    int32_t session;
};

// Pinned host staging and device copy of a round's descriptors.
struct RoundBuffers {
    void *host = nullptr;
    void *dev = nullptr;
    size_t bytes = 0;
};

// The server's second stream (default priority) for rounds of both kinds, and
// the training scratch of a round: the per-tile dG of its batches and the bins
// of one of them.  The rounds of a server run one after the other on its
// stream, so one set serves them all.  It is sized when a session is created
// and not by the rounds: growing under traffic stalled them (a first load of 32
// sessions' 224 requests 800 -> 650 M vertices/s).
struct ServeBuf {
    uint32_t *p = nullptr;
    size_t words = 0;
};
struct ServeLanes {
    hipStream_t side = nullptr;
    hipEvent_t fork = nullptr, join = nullptr;
    ServeBuf dgt, cnt, items;
};

hipError_t serve_lanes_init(ServeLanes *l);
void serve_lanes_free(ServeLanes *l);
// Sizes the scratch for rounds of `vertices` training vertices of the sessions
// `nets`, or of the largest power-of-two part of them that `bytes` hold (none
// below kMinLaneVertices).  `s`, the rounds' stream, is drained before anything
// is freed.  A device without room leaves it smaller, down to nothing.
constexpr int64_t kMinLaneVertices = 2048;
void serve_lanes_size(ServeLanes *l, int64_t vertices, int64_t bytes,
                      const std::vector<Net> &nets, hipStream_t s);
hipError_t round_buffers_init(RoundBuffers *b);
void round_buffers_free(RoundBuffers *b);
// Whether the persistent kernels are instantiated for this network shape.
bool serve_supports(const npm_config *cfg);
// Enqueues one round on `s` (and beside it on the lanes' side stream, which `s`
// waits for): the persistent query kernel over every query of the round, the
// persistent backward kernel over every training batch, each batch's grid
// scatter, and the Adam step of each session that trained.
hipError_t serve_launch_round(RoundBuffers *b, ServeLanes *lanes,
                              const std::vector<ServeRequest> &reqs, hipStream_t s);

}  // namespace npm
