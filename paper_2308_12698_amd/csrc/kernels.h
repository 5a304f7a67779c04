/*
 * kernels.h -- internal interface between the C ABI (abi.hip) and the
 * gfx950 kernels (kernels.hip).  Not installed; not part of the ABI.
 */
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "quad_step.h"

namespace potato {

constexpr int kRows = 30;       /* state rows per agent, see include/potato.h */
constexpr int kCarryRows = 10;  /* rounding-carry rows per agent */
constexpr int kCkptRows = 40;   /* checkpoint slot: the state, then its carries */

/* Largest agent count: agent index times 4 (a byte offset into a row) must
 * fit 32 bits, which the kernels' row addressing relies on. */
constexpr int64_t kMaxAgents = int64_t(1) << 30;

/* Everything one rollout launch needs, passed by value as the kernel
 * argument (uniform, lands in scalar registers). */
struct StepArgs {
    float* rows;                 /* [kRows][ld] */
    int64_t ld;
    float* carry;                /* [kCarryRows][carry_ld] or null (uncompensated) */
    int64_t carry_ld;
    int64_t n;                   /* agents (lanes) */
    const uint8_t* type;         /* [ld] or null */
    const int32_t* perm;         /* [n] or null */
    const float* gains;          /* [9][gains_ld] or null */
    int64_t gains_ld;
    const float* motor_cmd;      /* [4][cmd_ld] */
    const float* wp;             /* [n_epochs][3][cmd_ld] */
    int64_t cmd_ld;
    int32_t n_epochs;
    int32_t resample;
    int64_t step0;               /* global index of this launch's first step */
    int32_t n_steps;             /* steps in this launch */
    int32_t k0;                  /* call-relative index of this launch's first step */
    float* ckpt;                 /* [slots][kCkptRows][ld] or null (needs carry) */
    int32_t ckpt_every;
    int32_t n_types;
    const TypeConst* table;      /* device [n_types] */
    const uint8_t* alive;        /* [ld] or null: 0 = dead, not advanced */
    int32_t n_groups;            /* classes of types grouped within a block (a per-agent
                                    type and no processing order), or 0: none */
    float* snap;                 /* [3][n] device view of pinned host memory, or null: every
                                    agent's position after this launch (not with ckpt) */
    Limits lim;
    /* dt/6 less its rounding lim.dt6 (cars and aircraft).  Last, since a field
     * before the others moves the quadrotors' step loop by some bytes: the
     * same instructions then took 2 to 4 % longer (9.9 -> 10.3 us per step at
     * 1,048,576 agents of the plain form). */
    float dt6_lo;
};

struct Variant {
    int mode;        /* 0 open loop, 1 closed loop */
    bool het;        /* per-agent type index, LDS table */
    bool gains;      /* per-agent gains */
    bool ckpt;       /* write checkpoints */
    bool perm;       /* processing order */
    bool carry;      /* rounding carries kept in a carry buffer */
    bool kinds;      /* the type table holds cars or fixed-wing aircraft */
};

/* Arguments of the adjoint (reverse sweep) launch. */
struct AdjArgs {
    const float* ckpt;           /* [slots][kCkptRows][ld] from the forward call */
    int64_t ld;
    int64_t n;
    const uint8_t* type;
    const int32_t* perm;
    const float* gains;
    int64_t gains_ld;
    const float* wp;
    int64_t cmd_ld;
    int32_t n_epochs;
    int32_t resample;
    int64_t step0;
    int32_t n_steps;
    int32_t K;                   /* checkpoint interval */
    const float* grad_final;     /* [30][ld] */
    float* grad_x0;              /* [17][ld]: rows 0-16 */
    float* grad_mem;             /* [13][ld] or null: rows 17-29 */
    float* grad_gains;           /* [9][ld] or null */
    float* tape;                 /* layouts at launch_adjoint */
    int64_t tape_ld;             /* threads in the grid (a multiple of 64) */
    int32_t n_types;
    const TypeConst* table;
    const uint8_t* alive;
    Limits lim;
};

/* Agents of a per-agent type in the caller's order (no checkpoints) are
 * stepped grouped by class (types of equal step budget and kind; 2 to
 * kMaxGroups classes) within chunks of up to kGroupWidths block widths.
 * Unless a grid is given, such a launch takes as many blocks as the chip
 * holds at once (fewer if the swarm needs fewer); each block owns
 * ceil(n / grid) agents, rounded up to a multiple of 64.  The sort takes
 * group_lds_words(block) words of LDS after the type table. */
constexpr int kGroupWidths = 4;
constexpr int kMaxGroups = 8;
__host__ __device__ constexpr int64_t group_lds_words(int block) {
    return 2 * (int64_t)kGroupWidths * (block / 64) * kMaxGroups + (int64_t)kGroupWidths * block +
           kMaxGroups * 64 + 2 * ((int64_t)kGroupWidths * (block / 64) + kMaxGroups) + 4 * kMaxGroups + 2;
}

/* Launch one rollout kernel (n_steps of args) on `stream`. */
hipError_t launch_rollout(const Variant& v, const StepArgs& a, int block, int grid_blocks,
                          hipStream_t stream);

/* Kernel function pointer of a launch (occupancy queries). */
const void* rollout_kernel(const Variant& v, const StepArgs& a);

/* Swarms of at most kLaneAgents quadrotors take four lanes per agent: 16
 * agents per wave, one wave on each of the chip's 1,024 SIMDs.  A wave that
 * has its SIMD to itself issues one instruction per 4 clocks at best, so a
 * step costs its instructions: 285 vector instructions against one agent
 * per lane's 523, 0.537 us per closed-loop step against 0.940 (open loop
 * 0.316 against 0.578), from 1,000 to 16,384 agents alike.  Two such waves
 * on a SIMD take turns (0.977 us at 24,000 agents), one wave of one agent
 * per lane does not mind how many of its lanes are used (0.940).
 * A launch of a single step is loads and stores, which one agent per lane
 * does in wider accesses: 4.20 us per launch against 4.86 at 10,000 agents,
 * 4.07 against 4.65 at 16,384; from two steps on four lanes are as fast.
 * With per-agent types four lanes are faster then too (4.5 against 10.5 us
 * at 1,000 agents: no grouping by class).  Swarms that run at once on streams
 * of their own share the SIMDs, which four lanes per agent fill sooner: 1,000
 * steps of two swarms of 1,000 to 16,384 agents take 0.55 to 1.0 ms (1.0 to
 * 1.4 with one lane), of four 1.0 to 1.9 (1.0 to 2.6), but of four of 5,000
 * agents 1.9 against 1.46. */
#ifndef POTATO_LANE_AGENTS
#define POTATO_LANE_AGENTS 16384
#endif
constexpr int64_t kLaneAgents = POTATO_LANE_AGENTS;
bool rollout_lanes(const Variant& v, const StepArgs& a);

/* Closed-loop swarms of more than kSpacedAgents (more than two waves per
 * SIMD) of one quadrotor type, or with cars or aircraft in a processing
 * order, and no agents left out, take the spaced rsq and sqrt of quad_step.h:
 * per step 9.87 -> 9.25 us at 1,048,576 quadrotors, 5.16 -> 4.91 at 524,288,
 * 2.75 -> 2.69 at 262,144, 2.33 -> 2.28 at 140,000 (but 1.53 -> 1.58 at
 * 131,072); mixed kinds in order 2.64 -> 2.38 at 150,000, 2.49 -> 2.43 at
 * 262,144, 4.52 -> 4.36 at 524,288, equal at 1M.  With an alive mask the host
 * does not know how many waves are live: quadrotors scattered over a swarm
 * would gain by it (10.3 -> 9.3 at 1M with a fifth dead), a quarter alive in
 * one piece loses (1.01 -> 1.16 at 140,000 and 262,144).
 * The others lose too: quadrotors of several types (2.63 -> 2.85 ms per 1,000
 * steps of 251,904, nearly all of which run every step; the spaced loop reads
 * its constants from LDS in every step, there by lane from entries of 176
 * bytes), kinds of which many agents are dead (the quadrotors alone 1.45 ->
 * 1.54 us per step at 262,144 in order, 2.1 -> 3.0 in the caller's), and kinds
 * in the caller's order gain nothing (2.95 either way). */
#ifndef POTATO_SPACED_AGENTS
#define POTATO_SPACED_AGENTS 131072
#endif
constexpr int64_t kSpacedAgents = POTATO_SPACED_AGENTS;
bool rollout_spaced(const Variant& v, const StepArgs& a);

/* Adjoint: kernel pointer (occupancy queries) and launch of grid_blocks
 * blocks.  One agent per thread, kAdjBlock threads per block, tape
 * [K][grid threads / 64][kTapeRows][64]; or, with `pipe`, kAdjPipeBlock
 * threads per block serving 64 agents with one recomputing and one
 * reversing wave, tape [grid][2][K][kTapeRows][64].  Either way the tape
 * takes K x kTapeRows x grid x block floats. */
const void* adjoint_kernel(bool het, bool gains, bool perm, bool pipe, bool stream = false);
hipError_t launch_adjoint(bool het, bool gains, bool perm, bool pipe, const AdjArgs& a, int grid_blocks,
                          hipStream_t stream);
size_t adjoint_lds_bytes(bool het, int n_types, bool pipe);

/* Launches whose tape (the 23 rows that every step writes and reads) does
 * not fit the 256 MB Infinity Cache with room to spare read it with loads
 * that leave the cache to the slots still to come: per step 3.36 -> 3.33 us
 * at 65,536 agents with 50 steps per segment, 3.28 -> 2.97 with 20 (231 MB),
 * 3.25 -> 3.11 at 49,152 with 50.  Smaller tapes stay in the caches, and the
 * plain loads are the better ones (8,192 agents, 20 steps per segment: 2.44
 * against 2.54).  One agent per thread: only where the waves come back to
 * their slots for further agents (14.65 -> 13.9 at 300,007 agents, 51.5 ->
 * 49.9 at 1,048,576; a single round at 131,072 is no faster, 5.97 against
 * 6.07). */
constexpr int64_t kStreamTapeBytes = int64_t(192) << 20;
bool adjoint_streams(bool pipe, const AdjArgs& a);
constexpr int kAdjBlock = 256;
constexpr int kAdjPipeBlock = 128;
/* Use the pipelined adjoint for small swarms (1) or never (0). */
#ifndef POTATO_ADJOINT_PIPE
#define POTATO_ADJOINT_PIPE 1
#endif

/* Dynamic LDS bytes of a launch: the limits, a.n_types type-table entries
 * and, when it groups its agents, the sort's words. */
size_t rollout_lds_bytes(const Variant& v, const StepArgs& a, int block);
bool rollout_grouped(const Variant& v, const StepArgs& a);

/* Processing order by type (see potato_order_by_type): workspace of
 * order_workspace_words(n, n_types) int32 words. */
int64_t order_workspace_words(int64_t n, int n_types);
hipError_t launch_order_by_type(const uint8_t* type, int64_t n, int n_types,
                                const int32_t* type_rank_dev, int32_t* perm,
                                int32_t* workspace, hipStream_t stream);

constexpr int kOrderBlock = 256;

/* Adds to *count the agents whose first n_rows rows hold a non-finite value. */
hipError_t launch_count_nonfinite(const float* rows, int64_t ld, int64_t n, int n_rows, unsigned long long* count,
                                  hipStream_t stream);

/* Collision detection on a hashed grid (see collide.hip). */
int64_t collision_workspace_bytes(int64_t n);
/* Largest swarm of the allocation-free collision entry point. */
constexpr int64_t kNoAllocMaxAgents = int64_t(1) << 20;
/* Device address (current device) and size of that entry point's static
 * workspace; the address is looked up once per device and kept. */
hipError_t collision_scratch(void** ptr, int64_t* bytes);
hipError_t launch_detect_collisions(const float* rows, int64_t ld, int64_t n, const uint8_t* type, int n_types,
                                    const float* radius_dev, float r_max, uint8_t* alive,
                                    unsigned long long* died, void* workspace, hipStream_t s);

}  // namespace potato
