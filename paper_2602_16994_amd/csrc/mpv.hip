// mpv.hip -- kernels and C ABI of the tree-verification library (gfx950 only).
//
// Path of one mpv_verify call (all on the caller's stream):
//   init_kernel            zero counters, default the per-node results, clear queue and team words
//   node_task_kernel       persistent workgroups of 256 lanes, three per compute unit, grouped in
//                          TEAMS of G workgroups that take tasks from a queue until none are left.
//                          A team splits every logit row by vocabulary range: each member keeps its
//                          part of the task's (target, draft) row pair on chip (registers + LDS),
//                          and every V-wide sum is a local partial plus one exchange of a few
//                          words between the members (through the L2 of their chiplet, 0.4 us; through
//                          memory, 0.7 to 1, where they are not on one).
//                          Node task, one per (tree, internal node) the rule needs:
//                            softmax statistics of the node's target and draft rows, then,
//                            for each child in list order, the probability the child is
//                            tested with (or, Traversal, its starting weight) and the residual
//                            mass after its rejection (a V-wide reduction per child, over the
//                            row pair kept on chip).  A task starts the tasks that follow
//                            from it: SpecInfer the accepted child, Traversal the children of
//                            positive weight; tasks of trees whose outcome is settled are
//                            dropped.  With per-node debug outputs every node's task runs.
//                          Sampling task, one per tree, started by the task that settles the
//                            tree: the uniform-dependent walk, then the team draws the bonus
//                            token by inverse CDF from the residual of the stopping node.
//                            (NSS, Naive, SpecTr: one per draw of the token-following walk.)
//                          The top-down rules draw as a part of the walk instead (draw_walk), from the part on chip.
//   walk_kernel, short_part_kernel, staged_part_kernel    the same for walks of the top-down rules, and for parts that the
//                          registers hold (with draws, and without)
// mpv_verify_merged (a shape per tree) adds shape_kernel, which works out every tree's tables.
// mpv_block_efficiency and mpv_acceptance_rates run the same kernels with every node task and
// no uniforms (see Args::estimate); mpv_nucleus_mask is a kernel of its own (mpv_nucleus.h).
//
// Why this is the same computation as the step-by-step rules: every distribution
// either rule draws from is (p - c q)_+ / W(c) for one scalar c per node state
// (since (x_+/W - q)_+ = (x - W q)_+ / W), and each node is tested after exactly
// one possible history, so its test probability does not depend on the uniforms.

#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <atomic>

#include "mpv.h"
#include "mpv_device.h"
#include "mpv_exchange.h"
#include "mpv_nucleus.h"

namespace mpv {

// ------------------------------------------------------------------ host/device tree tables

// Node numbers are below MPV_MAX_NODES = 64: one byte each (the tables live in LDS, where the three
// workgroups of a compute unit have 53 KB each).
struct TreeDesc {
    int32_t N;
    // Traversal, only what is needed, no team to spare: the node where the tree branches
    // (-1: not used) first handles its first child only; the rest of its work (a second task:
    // "resumed") is started when that child's subtree, split_mask in postorder positions, turns
    // out to be rejected as a whole.
    int32_t split_node;
    unsigned long long split_mask;
    int8_t parent[MPV_MAX_NODES];
    int8_t nchild[MPV_MAX_NODES];
    int8_t child_off[MPV_MAX_NODES];     // start of the node's children in child_list
    int8_t child_list[MPV_MAX_NODES];    // children of node 0, of node 1, ... ascending
    int8_t depth[MPV_MAX_NODES];
    int8_t postorder[MPV_MAX_NODES];     // depth-first, children (in list order) before their parent; root last
    int8_t rank[MPV_MAX_NODES];          // position of the node in postorder
    int8_t sub_lo[MPV_MAX_NODES];        // the node's subtree is postorder[sub_lo[n] .. rank[n]]
    int8_t cls[MPV_MAX_NODES];           // priority class of the node's task (see QueuePlan)
    int32_t class_off[8];                // QueuePlan::off again, for the kernels that read the tables from memory
};
static_assert(MPV_MAX_NODES <= 127 && sizeof(TreeDesc) % 8 == 0, "node numbers must fit a signed byte");

// The tables of one tree of a batch in which every tree has a shape of its own: one 64-bit word per
// node (a wave reads a tree's tables in one load, a lane a word), the fields of node n in word n except
// for child_list and postorder, which are lists: entry n.
constexpr int kShapeParent = 0, kShapeNChild = 6, kShapeChildOff = 11, kShapeChildList = 17, kShapeDepth = 23,
              kShapePostorder = 29, kShapeRank = 35, kShapeSubLo = 41, kShapeCls = 47, kShapeSplit = 48;
constexpr int kShapeNoSplit = 127;        // (7 bits in kShapeSplit: split_node, the same in every word)
static_assert(MPV_MAX_NODES <= 64 && MPV_MAX_CHILDREN < 32, "the fields of a shape word are too narrow");

constexpr int kMaxClasses = 4;
constexpr int kCtlIdle = 4 + 2 * kMaxClasses, kCtlFirst = kCtlIdle + 1, kCtlTreesDone = kCtlIdle + 2, kCtlWords = kCtlIdle + 3;
static_assert(kMaxClasses + 1 <= 8, "TreeDesc::class_off is too short");

// The task queue is one first-in-first-out queue per priority class; a free team is
// given the oldest task of the lowest class that has one.  Class 0: the nodes from the root down
// to the first node that branches (every tree needs them).  Class 1: the nodes below it, which
// a settled tree no longer needs.  (More classes are possible: the dispatcher takes any number
// up to kMaxClasses.  Ranking the subtrees of the branching node by the order in which the rule
// visits them was tried and lost to plain age order: it starves the later subtrees of the
// trees that end up needing all of them, and those trees decide when the launch ends.)
struct QueuePlan {
    int32_t nclass;
    int32_t off[kMaxClasses + 1];        // class c owns queue[off[c] .. off[c+1])
    // First tasks: the nodes whose tasks can run from the start, lowest class first; first task number h
    // is that of node init_node[h / B] of tree h % B.  They are never queued, the teams count them off.
    int8_t init_node[MPV_MAX_NODES];
    int32_t init_total;                  // first tasks
    int32_t root_is_leaf;                // no node task at all: the first tasks are the sampling tasks
    int32_t teams;                       // teams of the launch (the grid is teams * team_size workgroups)
    int32_t team_size;                   // G: workgroups that share one task
    int32_t part_vecs;                   // 16-byte vectors of a row per member (a multiple of 64)
    int32_t box_step;                    // words from one team's mailbox to the next
    int32_t same_xcd;                    // members of a team are 8 workgroup numbers apart (one chiplet, its L2)
    int32_t spare;                       // teams are left over from the start (not counting those that whole chiplets add)
};

constexpr int kMaxTeam = 16;                          // workgroups per team, at most
constexpr int kExchWords = 8;                         // 64-bit words one member hands over per exchange
constexpr int kMaxGrid = 768;                        // workgroups of a launch, at most (three per compute unit)

// Per-(tree,node) scalars kept in the workspace, all double, each [B*N].
struct Workspace {
    double* At;      // log2-partition of the target row (internal nodes)
    double* Ad;      // same for the draft row
    double* cfin;    // c of the node's final state (all children rejected); SpecTr: the division factor rho* (the token is drawn from (p - rho* q)_+)
    double* aux;     // block-efficiency estimate, Naive and SpecTr: p_res at the node's token (see estimate_wave);
                     // verification of trees that each have a shape of their own: the shape words (see load_shape)
    double* a0;      // Traversal: weight the node starts with (kNotReady until its parent's task publishes it)
    double* atest;   // probability the node is tested with
    int32_t* queue;      // entry = tree * N + node (node task) or B * N + tree (sampling task), -1 = not written yet
    // [0] appended: tasks ever queued or started directly, [1] completed: tasks finished or cancelled,
    // [2] exit: set when nothing is left, [3] lock: held by the team leader that is dispatching,
    // [4 + c] tail of class c: entries appended, [4 + kMaxClasses + c] head of class c: entries handed out,
    // [kCtlIdle] teams left waiting after the last round of dispatching (a hint), [kCtlFirst] first tasks
    // counted off, [kCtlTreesDone] trees whose outputs are written
    int32_t* qctl;
    int32_t* mailbox;    // [teams], QueuePlan::box_step words apart: kMailboxAbsent until the team has asked for a task, then kMailboxWaiting /
                         // kMailboxSoon, or the task handed to that team
    // Per tree, one bit per node at the node's position in postorder: `known` = the outcome of
    // the node's test is settled, `acc` = it is "accepted" (valid once known).  `decided` = the
    // sampling task has been queued (and, when only what the rule needs is computed, the
    // tree's remaining node tasks are cancelled).
    unsigned long long* known;
    unsigned long long* acc;
    int32_t* decided;
    int32_t* cur;        // [B] token-following walks: the node the walk has reached
    // Teams.  exch: [team][2][member][kExchWords] words of (sequence number << 32 | 32 bits of payload);
    // team_task: [team][2] the task the leader has taken and its flags, same packing.  The first line of a
    // team's area also serves its start (it is first written by exchange 2): word 0 counts the members that
    // have started, words 1 and 2 announce the first task.
    unsigned long long* exch;
    unsigned long long* team_task;
    struct LaunchBlock* launch;   // what node_task_kernel is launched with, written by init_kernel
};

// Every field has a default (null / 0): what a call does not set stays off.
struct Args {
    const void* zt = nullptr;
    const void* zd = nullptr;
    const int32_t* tokens = nullptr;
    const float* uniforms = nullptr;
    const float* draw_uniforms = nullptr;      // walks that draw a token at every node they visit
    int32_t* accept_len = nullptr;
    int32_t* path_nodes = nullptr;
    int32_t* path_tokens = nullptr;
    int32_t* bonus = nullptr;
    uint32_t* counters = nullptr;
    float* dbg_stats = nullptr;
    float* dbg_edge = nullptr;
    float* dbg_accept = nullptr;
    float* dbg_resid = nullptr;
    int32_t B = 0, N = 0, V = 0, max_depth = 0;
    float k32 = 0.f;       // float(log2(e)/T)
    int32_t walk = 0;    // 0: the rule names the stopping node (SpecInfer, Traversal); a token is drawn at every
                     // visited node and followed if it is a child's: 1 from p (NSS), 2 after the Naive test,
                     // 3 after the SpecTr tests
    int32_t lazy = 0;    // compute only what the rule needs (off when per-node debug output is wanted: then every node task runs)
    // Expected block efficiency instead of a verification (Sec. 5, Eq. 1-3): every node task runs
    // (lazy = 0), no uniforms are read, and what would be a tree's sampling task turns the per-node
    // results into reach probabilities.  reach_prob [B,N] may be null; expected [B].
    // estimate = 2: acceptance rates instead (App. C): per internal node, from its two rows and its
    // number of children alone; no tokens are read, nothing follows the node tasks.  alpha [B,N].
    int32_t estimate = 0;
    int32_t keep_counters = 0;   // the call continues an earlier one: init_kernel leaves the counters as they are
    int32_t per_tree = 0;        // every tree has a shape of its own: its tables are in Workspace::aux
    float* reach_prob = nullptr;
    float* expected = nullptr;
    float* alpha = nullptr;
    // Trees of distinct contexts, SpecTr: [B,N], the node an accepted child entry stands for (itself unless the
    // entry repeats a token drafted earlier under the same node); null: every entry stands for itself.
    const int32_t* context_node = nullptr;
};

// Everything node_task_kernel needs to know, in one block of the workspace: the kernel and the
// functions it calls read it through one pointer (as kernel arguments, passed on by reference, the
// three structures were copied into every lane's private memory).
struct Launch {
    QueuePlan q;
    Workspace ws;
    Args a;
};
struct LaunchBlock {
    Launch l;
    TreeDesc tree;
};
static_assert(sizeof(Launch) % 8 == 0, "the launch block is copied in whole words, the tree tables follow at once");

constexpr int kInitBlock = 256;
constexpr int kTaskBlock = 256;
constexpr int kTaskWaves = kTaskBlock / kWave;
constexpr int kTaskUnroll = 4;
// node tasks keep their part of a row pair on chip: per lane and row, kRegVecs 16-byte vectors in
// registers and kLdsVecs in LDS
constexpr int kRegVecs = 6;
constexpr int kLdsVecs = 6;
constexpr int kPartCapacity = (kRegVecs + kLdsVecs) * kTaskBlock;     // vectors of a row one member keeps
// upper bound on the polls of a dependency flag (about a second); see node_task_kernel
constexpr int kMaxSpins = 1 << 20;
// no wait inside a launch outlasts this (wall clock, 100 MHz ticks: 2 s)
constexpr long long kLaunchTimeoutTicks = 200000000ll;
// bit pattern (a NaN) of a starting weight that has not been published yet
constexpr unsigned long long kNotReady = ~0ull;
// wave tiles of the bonus sampler: 64 16-byte vectors; float rows have the smallest tiles
constexpr int kMaxTiles = MPV_MAX_VOCAB / (kWave * 4);
// task hand-over between the dispatcher and the teams (see "task queue")
constexpr int kMailboxWaiting = -1;                  // the team is idle
constexpr int kMailboxSoon = -2;                     // the team has asked ahead: it will be free shortly
constexpr int kMailboxAbsent = -3;                   // the team has not asked for anything yet
constexpr int kMailboxDispatch = -6;                  // the team is handed the dispatcher's lock
constexpr int kMailboxExit = -7;                      // nothing is left
constexpr int kMailboxWords = 1024;                   // the mailboxes' memory: as far apart as it allows
constexpr int kTaskExit = -1;                         // what a leader's wait returns when all is done
constexpr int kTaskNone = -2;                         // announced to a team that came too late for a first task
constexpr int kWorkerSlots = 8;                       // mailboxes per dispatcher lane
constexpr int kMaxTeams = kWave * kWorkerSlots;
static_assert(kMaxTeams <= kMailboxWords, "a mailbox for every team");
constexpr int kKindAcceptance = 100;                   // node_task_kernel instantiation for the acceptance rates (see there)
constexpr int kKindWalk = 200;                         // top-down rules, walks that draw their tokens themselves (walk_kernel)
constexpr int kKindShort = 300;                        // ... on parts that the registers hold (short_part_kernel)
constexpr int kKindShortAll = 400;                     // such parts without draws: every node's task, estimates (staged_part_kernel)
constexpr int method_of(int kind) { return kind >= kKindAcceptance ? MPV_METHOD_SPECINFER : kind; }

// LDS of node_task_kernel that the functions it calls use as well (file scope, so that they address
// it as LDS and not through generic pointers)
struct TaskShared {
    double part[kTaskWaves][4];                   // per-wave partial sums of a team reduction
    float partf[kTaskWaves][2];                   // per-wave reference exponents of the statistics
};
__shared__ TaskShared g_sh;
// the launch parameters (copied from the workspace at the start of node_task_kernel)
__shared__ __align__(16) int g_launch_words[sizeof(Launch) / sizeof(int)];
__device__ __forceinline__ const Launch& lds_launch() { return *reinterpret_cast<const Launch*>(g_launch_words); }
// the part of the row pair kept in LDS (target slots, then draft slots); the sampling task's table
// of tile masses uses the same memory
__shared__ uint4 g_rows[2 * kLdsVecs * kTaskBlock];
static_assert(sizeof(g_rows) >= kMaxTiles * sizeof(float), "tile masses do not fit in the kept-row LDS");
// the tree tables (copied from the workspace at the start of node_task_kernel)
__shared__ TreeDesc g_tree;
// Args::per_tree: the tree whose tables g_tree holds (-1: none yet); the first wave's business
__shared__ int g_tree_of;

// A value that is the same in every lane, for the compiler to keep in scalar registers.  Needed
// wherever a function that is not inlined receives it: arguments arrive in vector registers.
__device__ __forceinline__ int uniform_i32(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <class P>
__device__ __forceinline__ P* uniform_ptr(P* p) {
    const unsigned long long v = reinterpret_cast<unsigned long long>(p);
    const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(v)));
    const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(v >> 32)));
    return reinterpret_cast<P*>((static_cast<unsigned long long>(hi) << 32) | lo);
}
template <class S>
__device__ __forceinline__ S uniform_struct(const S& s) {
    static_assert(sizeof(S) % 4 == 0, "whole words only");
    S out;
    const int* src = reinterpret_cast<const int*>(&s);
    int* dst = reinterpret_cast<int*>(&out);
#pragma unroll
    for (int i = 0; i < static_cast<int>(sizeof(S) / 4); ++i) dst[i] = __builtin_amdgcn_readfirstlane(src[i]);
    return out;
}

// ------------------------------------------------------------------ trees that each have a shape of their own

__device__ __forceinline__ int tree_of_task(int t, int B, int N) {      // (node, sampling and resumed tasks)
    return uniform_i32(t >= B * N + B ? t - (B * N + B) : (t >= B * N ? t - B * N : t / N));
}

// First wave of a workgroup, when nobody else reads the tables (the other waves wait at a barrier):
// puts the tables of tree b into g_tree.  One load per tree change, about a microsecond; between
// tasks of one tree nothing is read.
__device__ __forceinline__ void load_shape(const unsigned long long* shapes, int N, int b) {
    if (uniform_i32(g_tree_of) == b) return;
    const int lane = threadIdx.x;
    const unsigned long long w = lane < N ? as_global(shapes)[static_cast<size_t>(b) * N + lane] : 0ull;
    const unsigned lo = static_cast<unsigned>(w), hi = static_cast<unsigned>(w >> 32);
    auto bits = [&](int at, int width) { return static_cast<int>((w >> at) & ((1ull << width) - 1ull)); };
    if (lane < N) {
        g_tree.parent[lane] = static_cast<int8_t>(lane ? bits(kShapeParent, 6) : -1);
        g_tree.nchild[lane] = static_cast<int8_t>(bits(kShapeNChild, 5));
        g_tree.child_off[lane] = static_cast<int8_t>(bits(kShapeChildOff, 6));
        g_tree.child_list[lane] = static_cast<int8_t>(bits(kShapeChildList, 6));
        g_tree.depth[lane] = static_cast<int8_t>(bits(kShapeDepth, 6));
        g_tree.postorder[lane] = static_cast<int8_t>(bits(kShapePostorder, 6));
        g_tree.rank[lane] = static_cast<int8_t>(bits(kShapeRank, 6));
        g_tree.sub_lo[lane] = static_cast<int8_t>(bits(kShapeSubLo, 6));
        g_tree.cls[lane] = static_cast<int8_t>(bits(kShapeCls, 1));
    }
    // the word of one node, the same in every lane
    auto word = [&](int n) {
        const unsigned long long l = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(lo), n));
        const unsigned long long h = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(hi), n));
        return (h << 32) | l;
    };
    const int split = static_cast<int>((word(0) >> kShapeSplit) & 127ull);
    unsigned long long mask = 0ull;
    if (split != kShapeNoSplit) {                      // the subtree of the first child, in postorder positions
        const int at = static_cast<int>((word(split) >> kShapeChildOff) & 63ull);
        const unsigned long long first = word(static_cast<int>((word(at) >> kShapeChildList) & 63ull));
        const int r_hi = static_cast<int>((first >> kShapeRank) & 63ull), r_lo = static_cast<int>((first >> kShapeSubLo) & 63ull);
        mask = ((r_hi >= 63) ? ~0ull : ((1ull << (r_hi + 1)) - 1ull)) & ~((1ull << r_lo) - 1ull);
    }
    if (lane == 0) {
        g_tree.split_node = split != kShapeNoSplit ? split : -1;
        g_tree.split_mask = mask;
        g_tree_of = b;
    }
    __builtin_amdgcn_wave_barrier();
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
}

// Before, a batch was one launch pair per run of consecutive equal shapes, each a dependent chain of
// tasks with most of the chip idle: 64 trees of 22 shapes, V = 128256, SpecInfer 3.6 ms, now 0.092 ms;
// 256 trees of 162 shapes, V = 151936, Traversal 22.2 ms, now 0.51 ms.
//
// Parent arrays travel to the device as kernel arguments (a byte per node): no copy that could
// synchronise, no host memory that has to outlive the call, and a captured graph holds them.
constexpr int kShapeChunkBytes = 3584;               // (kernel arguments: 4 KB in all)
struct ShapeChunk { unsigned char parent[kShapeChunkBytes]; };

// The tables of the trees [first, first + gridDim.x) from their parent arrays: one wave per tree, lane n
// looks after node n; the two loops over the nodes are scalar steps over the wave's registers (about 2 us
// for 41 nodes).  The host has checked the arrays (0 <= parent[n] < n, depth, number of children).
__global__ __launch_bounds__(kWave) void shape_kernel(ShapeChunk chunk, unsigned long long* shapes, int first, int N, int split) {
    __shared__ int sh_child[MPV_MAX_NODES], sh_post[MPV_MAX_NODES];
    const int lane = threadIdx.x;
    const bool live = lane < N;
    const int par = (live && lane > 0) ? chunk.parent[blockIdx.x * N + lane] : 0;
    unsigned long long sub = live ? 1ull << lane : 0ull, kids = 0ull;
    for (int m = N - 1; m > 0; --m) {                  // descendants and children, as masks of nodes
        const int p = __builtin_amdgcn_readlane(par, m);
        const unsigned long long of_m = (static_cast<unsigned long long>(static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(sub >> 32), m))) << 32)
                                      | static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(sub), m));
        if (lane == p) { sub |= of_m; kids |= 1ull << m; }
    }
    const int nchild = __popcll(kids), size = __popcll(sub);
    const int off = wave_inclusive_scan_i32(nchild) - nchild;
    int depth = 0, start = 0, next = 0;                // start: postorder position of the subtree's first node
    for (int m = 1; m < N; ++m) {
        const int p = __builtin_amdgcn_readlane(par, m);
        const int at = __builtin_amdgcn_readlane(next, p), d = __builtin_amdgcn_readlane(depth, p);
        const int sz = __builtin_amdgcn_readlane(size, m);
        if (lane == p) next += sz;
        if (lane == m) { start = at; next = at; depth = d + 1; }
    }
    const int rank = start + size - 1;
    const unsigned long long siblings = __shfl(kids, par, kWave);
    const int par_off = __shfl(off, par, kWave);
    if (lane == 0) sh_child[N - 1] = 0;                // (N - 1 entries: the root is nobody's child)
    __builtin_amdgcn_wave_barrier();
    if (live) {
        if (lane > 0) sh_child[par_off + __popcll(siblings & ((1ull << lane) - 1ull))] = lane;
        sh_post[rank] = lane;
    }
    __syncthreads();
    // the first node from the root down that does not have exactly one child
    int branch = 0;
    while (__builtin_amdgcn_readlane(nchild, branch) == 1) branch = sh_child[__builtin_amdgcn_readlane(off, branch)];
    branch = uniform_i32(branch);
    const int branch_depth = __builtin_amdgcn_readlane(depth, branch), branch_kids = __builtin_amdgcn_readlane(nchild, branch);
    int split_node = kShapeNoSplit;
    if (split && branch_kids >= 2) {
        const int c0 = uniform_i32(sh_child[__builtin_amdgcn_readlane(off, branch)]);
        if (__builtin_amdgcn_readlane(nchild, c0) > 0) split_node = branch;
    }
    auto field = [](int v, int at) { return static_cast<unsigned long long>(v) << at; };
    if (live)
        shapes[static_cast<size_t>(first + static_cast<int>(blockIdx.x)) * N + lane] =
            field(par, kShapeParent) | field(nchild, kShapeNChild) | field(off, kShapeChildOff) |
            field(sh_child[lane], kShapeChildList) | field(depth, kShapeDepth) | field(sh_post[lane], kShapePostorder) |
            field(rank, kShapeRank) | field(start, kShapeSubLo) | field(depth <= branch_depth ? 0 : 1, kShapeCls) |
            field(split_node, kShapeSplit);
}

// ------------------------------------------------------------------ init

// Grid: x covers the trees (and the few per-launch words), y the nodes, so that every table
// lookup by node has a workgroup-uniform index.
//
// Latency only: every word is written once and nothing is read but the arguments, so what counts is
// that no thread does one thing after another.  The launch block goes over a word per lane, straight
// from the argument segment (a structure passed by value and indexed by the lane would first be
// copied to private memory; a word per workgroup, through scalar loads, was a chain of 40 loads on a
// small tree), and only the words of the teams that are launched are cleared.
// Median of this kernel 7.2 -> 5.4 us; with the tree tables next to the launch block, so that the kernel
// that follows asks for both at once, a call on one tree of 7 nodes takes 35.6 us (41.3).
__global__ __launch_bounds__(kInitBlock) void init_kernel(LaunchBlock block) {
    const QueuePlan& q = block.l.q;
    const Workspace& ws = block.l.ws;
    const Args& a = block.l.a;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;      // tree, or word number
    const int n = blockIdx.y;
    const int stride = gridDim.x * gridDim.y * blockDim.x;
    const int me = (blockIdx.y * gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
    {   // the launch block of the next kernel (the only argument: it starts the argument segment)
        const auto* src = (const __attribute__((address_space(4))) int*)__builtin_amdgcn_kernarg_segment_ptr();
        int* dst = reinterpret_cast<int*>(ws.launch);
        for (int w = me; w < static_cast<int>(sizeof(LaunchBlock) / sizeof(int)); w += stride) dst[w] = src[w];
    }
    {   // team words: no exchange has been written (their numbers are above 0), nobody has arrived
        const int exch_words = q.teams * q.team_size * 2 * kExchWords;
        for (int w = me; w < exch_words; w += stride) ws.exch[w] = 0ull;
        for (int w = me; w < kMaxTeams * 2; w += stride) ws.team_task[w] = 0ull;
        for (int w = me; w < q.teams; w += stride) ws.mailbox[w * q.box_step] = kMailboxAbsent;
    }
    if (n == 0) {
        if (i < MPV_COUNTER_COUNT && !a.keep_counters) a.counters[i] = 0u;
        if (i < kCtlWords) ws.qctl[i] = i == 0 ? q.init_total : 0;
        if (i < a.B) {
            // the root is never tested: it counts as accepted from the start
            ws.known[i] = 1ull << (a.N - 1);
            ws.acc[i] = 1ull << (a.N - 1);
            ws.decided[i] = 0;
            ws.cur[i] = 0;
            if (a.dbg_edge) {
                a.dbg_edge[static_cast<size_t>(i) * a.N * 2] = 1.f;
                a.dbg_edge[static_cast<size_t>(i) * a.N * 2 + 1] = 1.f;
            }
        }
    }
    if (i >= a.B) return;
    const int b = i;
    const size_t bn = static_cast<size_t>(b) * a.N + n;
    reinterpret_cast<unsigned long long*>(ws.a0)[bn] = kNotReady;
    if (a.alpha) a.alpha[bn] = 0.f;                          // leaves have no acceptance rate
    // a node no task ever reaches is tested with probability 0
    ws.atest[bn] = (n == 0) ? 1.0 : 0.0;
    ws.cfin[bn] = 0.0;
    const int at = n * a.B + b;                               // this thread's share of the queue words: "not written yet"
    if (at < q.off[q.nclass]) ws.queue[at] = -1;
}

// ------------------------------------------------------------------ task queue
//
// node_task_kernel is launched with three workgroups per compute unit at most, grouped in teams;
// each team runs tasks until told to exit.  A team takes part only once every member has
// started (the last to arrive counts off its first task), so a task is only ever handed to
// workgroups that are running, whatever else occupies the device.  A task is appended only when
// everything it needs has been published, so every queued task can run at once, on any team.
//   first:    the tasks that can run from the start are counted off by the teams (one atomic add each,
//             see claim_first), asked for ahead of time like the others.  Only what follows from them is
//             queued, and only a team for which no first task is left turns to the dispatcher.
//             (Through the dispatcher, as all tasks were before, a single team had its first task 5.6 us
//             after the start of the kernel and 768 workgroups theirs after 7 to 20; now 2.0 and 2.8.  The
//             counts of a team's arrivals and its first announcement are in a line of their own: next to
//             other teams' they took 9.6 us.)
//   append:   appended++, then slot = tail++ of the class, then the entry is written.
//   request:  mailbox[team] = "soon" when a team asks ahead, before the last sweep of its
//             current task (the answer is then usually there when it is done), "waiting" once
//             it has nothing to do.  Idle teams are served before those that asked ahead.
//   dispatch: a leader that has nothing to do takes the dispatcher lock if it is free and,
//             with its first wave, hands queued tasks to waiting teams (its own included)
//             in priority order (class, then age), until it has a task of its own; then it
//             passes the lock to a team that is still waiting, or releases it.  Those that find the
//             lock taken poll their own mailbox and nothing else (the lock and the exit flag only
//             now and then, should the holder have left at the moment they began to wait): when every
//             idle team looked at them all the time, their line, which the busy teams need for their
//             counts, was the bottleneck (200 trees of V = 1500 on 512 teams, Traversal: 338 us, then 273).
//             If every team is busy nobody dispatches, and nobody needs to.  Node tasks of trees
//             whose outcome is settled are dropped here when only what is needed is computed.
//   end:      whoever finishes the last tree (acceptance rates: the last task) sets the exit flag, see tree_done; what
//             is still queued then belongs to settled trees.  As a fallback, for a launch in which something went wrong,
//             the dispatcher looks in every 16th round without a queued task whether completed == appended, with
//             appended read before and after completed and unchanged: no task is queued, handed out or running, so
//             nothing can be appended any more.  A task's appends are performed before its completed++.
// A team may also run a task it has produced itself straight away (counted in appended,
// never queued).  Every wait is bounded.  Only the leader (member 0) of a team talks to the queue.

__device__ __forceinline__ int ld_relaxed(const int32_t* p) {
    return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long ld_relaxed(const unsigned long long* p) {
    return __hip_atomic_load(as_global(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(int32_t* p, int v) {
    __hip_atomic_store(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_relaxed(unsigned long long* p, unsigned long long v) {
    __hip_atomic_store(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The read-modify-write operations of the task kernels (relaxed, device scope, like HIP's own of
// these names, which they hide inside this namespace) on pointers known to be global.
__device__ __forceinline__ int atomicAdd(int* p, int v) {
    return __hip_atomic_fetch_add(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned atomicAdd(unsigned* p, unsigned v) {
    return __hip_atomic_fetch_add(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long atomicOr(unsigned long long* p, unsigned long long v) {
    return __hip_atomic_fetch_or(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned long long atomicAdd(unsigned long long* p, unsigned long long v) {
    return __hip_atomic_fetch_add(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int atomicCAS(int* p, int expected, int desired) {
    __hip_atomic_compare_exchange_strong(as_global(p), &expected, desired, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                         __HIP_MEMORY_SCOPE_AGENT);
    return expected;
}
// all loads, stores and atomics issued so far by this lane have been performed
__device__ __forceinline__ void wait_memory() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Append one task to class c (one lane).  What the task needs and this lane has stored before
// is performed before the task can be handed out (the wait below covers it).
__device__ __forceinline__ void append_task(const TreeDesc& tree, const Workspace& ws, int c, int entry) {
    (void)atomicAdd(&ws.qctl[0], 1);
    wait_memory();                                    // counted before it can be handed out (and finished)
    const int slot = atomicAdd(&ws.qctl[4 + c], 1);
    const int first = tree.class_off[c], end = tree.class_off[c + 1];
    if (slot < end - first) st_relaxed(&ws.queue[first + slot], entry);
}

// First task number h, or kTaskNone when there are not that many.
__device__ __forceinline__ int first_task(const QueuePlan& q, const Args& a, int h) {
    if (h >= q.init_total) return kTaskNone;
    if (q.root_is_leaf) return a.B * a.N + h;
    int trees = uniform_i32(a.B);                     // (its reciprocal is not kept across tasks)
    asm volatile("" : "+s"(trees));
    return (h % trees) * a.N + q.init_node[h / trees];
}
// Counts off one first task (one lane).  The address is made a lane's own: for one that is the same in every lane the
// compiler adds the lanes up first and waits for the result at once; here it is waited for where it is used.
__device__ __forceinline__ int claim_first(const Workspace& ws) {
    unsigned long long at = reinterpret_cast<unsigned long long>(&ws.qctl[kCtlFirst]);
    asm volatile("" : "+v"(at));
    return atomicAdd(reinterpret_cast<int32_t*>(at), 1);
}

// A tree's outputs are written (one lane): with the last one the launch is over, whatever is still
// queued belongs to settled trees (returns whether it was the last).
__device__ __forceinline__ bool tree_done(const Workspace& ws, const Args& a) {
    const bool last = atomicAdd(&ws.qctl[kCtlTreesDone], 1) + 1 == a.B;
    if (last) st_relaxed(&ws.qctl[2], 1);
    return last;
}

// What the holder of the dispatcher's lock keeps from round to round.
struct Dispatcher {
    int head;             // lane c: head of class c
    unsigned left;        // which of the lane's teams (lane, lane + 64, ...: a bit each) are still waiting
    int hint;             // what kCtlIdle says
    unsigned quiet;       // rounds in which nothing was queued
    int own;              // the task its own team was given (-1: none)
    int previous;         // the task it took from its mailbox last
};

// One round of dispatching, by a whole wave that holds the lock, for team `team`.  Returns true when everything is finished
// (the exit flag has been set).
//
// Latency only: queued tasks wait for it.  Numbers that are the same in every lane are scalars, a lane's place among the
// waiting ones is a count of bits; all queue entries are asked for before the first is looked at, then all flags (two
// round trips to memory, not two for every 64 teams).
__device__ __forceinline__ bool dispatch_round(const QueuePlan& q, const TreeDesc& tree, const Workspace& ws, const Args& a, bool drop_settled,
                               int team, Dispatcher& d, long long t_begin) {
    const int lane = threadIdx.x;
    const int workers = uniform_i32(q.teams);
    // who is waiting, what is queued
    int box[kWorkerSlots];
#pragma unroll
    for (int sl = 0; sl < kWorkerSlots; ++sl) {
        box[sl] = kMailboxAbsent;
        if (sl * kWave < workers && lane + kWave * sl < workers) box[sl] = ld_relaxed(&ws.mailbox[(lane + kWave * sl) * q.box_step]);
    }
    const int tail = (lane <= kMaxClasses) ? ld_relaxed(&ws.qctl[lane < kMaxClasses ? 4 + lane : 2]) : 0;
    unsigned waiting = 0u, soon = 0u;
    int idle_others = 0, n_soon = 0;
    const int self_bit = team / kWave;
    const bool self_lane = (team & (kWave - 1)) == lane;
#pragma unroll
    for (int sl = 0; sl < kWorkerSlots; ++sl) {
        if (sl * kWave >= workers) continue;
        if (box[sl] == kMailboxWaiting) waiting |= 1u << sl;
        if (box[sl] == kMailboxSoon) soon |= 1u << sl;
        idle_others += __popcll(__ballot(box[sl] == kMailboxWaiting));
        n_soon += __popcll(__ballot(box[sl] == kMailboxSoon));
    }
    d.left = waiting;
    {   // the holder before may have handed this team a task that it had not seen when it took the lock
        int in_box = -1;
#pragma unroll
        for (int sl = 0; sl < kWorkerSlots; ++sl)
            if (self_lane && sl == self_bit) in_box = box[sl];
        in_box = __builtin_amdgcn_readlane(in_box, team & (kWave - 1));
        if (in_box >= 0 && in_box != d.previous) {
            d.own = in_box;
            return false;
        }
    }
    if (__builtin_amdgcn_readlane(tail, kMaxClasses) != 0) return true;               // (the exit flag)
    // the dispatcher's own team comes last of the idle ones: it goes on dispatching while there are others
    const bool mine_waits = self_lane && ((waiting >> self_bit) & 1u);
    const int self = __ballot(mine_waits) != 0ull ? 1 : 0;
    if (mine_waits) waiting &= ~(1u << self_bit);
    idle_others -= self;
    const int total_idle = idle_others + self, total_waiting = total_idle + n_soon;
    int first[kMaxClasses], before[kMaxClasses], total_avail = 0;      // class c: where its first entry is, number of that entry
#pragma unroll
    for (int c = 0; c < kMaxClasses; ++c) {
        const int head = __builtin_amdgcn_readlane(d.head, c);
        first[c] = uniform_i32(tree.class_off[c]) + head;
        before[c] = total_avail;
        if (c < q.nclass) total_avail += __builtin_amdgcn_readlane(tail, c) - head;
    }
    if (total_avail == 0 && (++d.quiet & 15u) == 0u) {
        // (the last tree ends the launch, see tree_done: this is for a launch in which something went wrong)
        int done = 0;
        if (lane == 0) {
            const int a1 = ld_relaxed(&ws.qctl[0]);
            wait_memory();
            const int co = ld_relaxed(&ws.qctl[1]);
            wait_memory();
            const int a2 = ld_relaxed(&ws.qctl[0]);
            done = (co == a1 && a1 == a2) ? 1 : 0;
            // a queue entry that never arrives, a task that never ends: give up after 2 s (must never happen)
            if (!done && wall_clock64() - t_begin > kLaunchTimeoutTicks) {
                atomicAdd(&a.counters[MPV_COUNTER_DEPENDENCY_TIMEOUT], 1u);
                done = 1;
            }
            if (done) {
                st_relaxed(&ws.qctl[2], 1);
                wait_memory();
            }
        }
        if (__builtin_amdgcn_readfirstlane(done)) return true;
    }
    // how many will still be waiting after this round: tasks look at it to decide whether work
    // that may turn out useless is worth queueing
    const int still_idle = max(0, total_idle - total_avail);
    if (lane == 0 && still_idle != d.hint) st_relaxed(&ws.qctl[kCtlIdle], still_idle);
    d.hint = still_idle;
    if (total_avail == 0 || total_waiting == 0) {
        __builtin_amdgcn_s_sleep(4);
        return false;
    }
    // Requester number r gets queued task number r (in class, age order); the idle teams
    // come first, then those that asked ahead.
    int entry[kWorkerSlots];
    unsigned served = 0u;
    {
        int r_idle = 0, r_soon = total_idle;
        const unsigned long long below = (1ull << lane) - 1ull;
#pragma unroll
        for (int sl = 0; sl < kWorkerSlots; ++sl) {
            entry[sl] = 0;
            if (sl * kWave >= workers) continue;
            const bool w = (waiting >> sl) & 1u, s = (soon >> sl) & 1u;
            const unsigned long long w_mask = __ballot(w), s_mask = __ballot(s);
            int mine = total_avail;
            if (w) mine = r_idle + __popcll(w_mask & below);
            if (s) mine = r_soon + __popcll(s_mask & below);
            if (mine_waits && sl == self_bit) mine = idle_others;
            r_idle += __popcll(w_mask);
            r_soon += __popcll(s_mask);
            if (mine < total_avail) {
                int at = first[0] + mine;
#pragma unroll
                for (int c = 1; c < kMaxClasses; ++c)
                    if (c < q.nclass && mine >= before[c]) at = first[c] + (mine - before[c]);
                entry[sl] = ld_relaxed(&ws.queue[at]);
                box[sl] = at;
                served |= 1u << sl;
            }
        }
    }
#pragma unroll
    for (int sl = 0; sl < kWorkerSlots; ++sl) {
        if (sl * kWave >= workers || !((served >> sl) & 1u)) continue;
        for (int spin = 0; spin < kMaxSpins && entry[sl] < 0; ++spin) {          // the entry follows its tail count closely
            __builtin_amdgcn_s_sleep(2);
            entry[sl] = ld_relaxed(&ws.queue[box[sl]]);
        }
    }
    int settled[kWorkerSlots], own = -1;
#pragma unroll
    for (int sl = 0; sl < kWorkerSlots; ++sl) {
        settled[sl] = 0;
        if (drop_settled && sl * kWave < workers && ((served >> sl) & 1u) && entry[sl] >= 0 && entry[sl] < a.B * a.N)
            settled[sl] = ld_relaxed(&ws.decided[entry[sl] / a.N]);
    }
#pragma unroll
    for (int sl = 0; sl < kWorkerSlots; ++sl) {
        if (sl * kWave >= workers || !((served >> sl) & 1u)) continue;
        if (entry[sl] < 0) {                          // must never happen: counted as finished, nobody runs it
            atomicAdd(&a.counters[MPV_COUNTER_DEPENDENCY_TIMEOUT], 1u);
            atomicAdd(&ws.qctl[1], 1);
        } else if (settled[sl] != 0) {
            atomicAdd(&a.counters[MPV_COUNTER_NODE_TASKS_CANCELLED], 1u);
            atomicAdd(&ws.qctl[1], 1);
        } else {
            st_relaxed(&ws.mailbox[(lane + kWave * sl) * q.box_step], entry[sl]);
            d.left &= ~(1u << sl);
            if (mine_waits && sl == self_bit) own = entry[sl];
        }
    }
    d.own = __builtin_amdgcn_readlane(own, team & (kWave - 1));
#pragma unroll
    for (int c = 0; c < kMaxClasses; ++c) {
        const int avail = (c + 1 < kMaxClasses ? before[c + 1] : total_avail) - before[c];
        if (lane == c) d.head += max(0, min(avail, total_waiting - before[c]));
    }
    wait_memory();
    return false;
}

// The next task of this team, or kTaskExit; called by every lane of the leader's first wave, returns
// the same value in each.  The team has asked (its mailbox says "waiting" or already holds
// the answer).  `previous` is the task it took from the mailbox last: until the request has
// reached memory the mailbox may still show it (no entry is ever handed out twice, so the
// value is unambiguous).
__device__ __attribute__((noinline)) int acquire_task(int team_in, int previous_in, bool drop_settled_in, long long t_start) {
    const Args& a = lds_launch().a;
    const Workspace& ws = lds_launch().ws;
    const QueuePlan& q = lds_launch().q;
    const TreeDesc& tree = g_tree;
    const int team = uniform_i32(team_in), previous = uniform_i32(previous_in);
    const bool drop_settled = uniform_i32(drop_settled_in ? 1 : 0) != 0;
    const int lane = threadIdx.x;
    int32_t* const box = &ws.mailbox[team * q.box_step];
    for (int spin = 0; spin < 8 * kMaxSpins; ++spin) {        // (the time limit below comes first)
        int t = 0, ex = 0, lk = 1;
        if (lane == 0) {
            // nothing to do any more: from "soon" to "waiting" (unless the answer has arrived)
            t = (spin == 0) ? static_cast<int>(atomicCAS(box, kMailboxSoon, kMailboxWaiting)) : ld_relaxed(box);
            if ((spin & 15) == 0) {
                ex = ld_relaxed(&ws.qctl[2]);
                lk = ld_relaxed(&ws.qctl[3]);
            }
        }
        t = __builtin_amdgcn_readfirstlane(t);
        if (t >= 0 && t != previous) return t;
        if (t == kMailboxExit || __builtin_amdgcn_readfirstlane(ex)) return kTaskExit;
        int got = 0;
        if (t == kMailboxDispatch) {
            if (lane == 0) st_relaxed(box, kMailboxWaiting);
            wait_memory();
            got = 1;
        } else if (lane == 0 && lk == 0 && t != kMailboxAbsent) {
            // (a team whose mailbox is still "absent" cannot be handed anything: it does not dispatch either)
            got = (atomicCAS(&ws.qctl[3], 0, 1) == 0) ? 1 : 0;
        }
        if (__builtin_amdgcn_readfirstlane(got)) {
            // the previous holder wrote the heads before it passed the lock on
            Dispatcher d;
            d.head = (lane < q.nclass) ? ld_relaxed(&ws.qctl[4 + kMaxClasses + lane]) : 0;
            d.left = d.quiet = 0u;
            d.hint = d.own = -1;
            d.previous = previous;
            int result = kTaskExit;
            for (;;) {
                if (dispatch_round(q, tree, ws, a, drop_settled, team, d, t_start)) break;
                if (d.own >= 0) { result = d.own; break; }
            }
            if (lane < q.nclass) st_relaxed(&ws.qctl[4 + kMaxClasses + lane], d.head);
            wait_memory();
            if (result == kTaskExit) {                 // (later ones see the flag)
                for (int sl = 0; sl < kWorkerSlots; ++sl)
                    if ((d.left >> sl) & 1u) st_relaxed(&ws.mailbox[(lane + kWave * sl) * q.box_step], kMailboxExit);
                return result;
            }
            const unsigned long long lanes = __ballot(d.left != 0u);
            if (lanes == 0ull) {
                if (lane == 0) st_relaxed(&ws.qctl[3], 0);
            } else if (lane == __ffsll(static_cast<long long>(lanes)) - 1) {
                st_relaxed(&ws.mailbox[(lane + kWave * (__ffs(static_cast<int>(d.left)) - 1)) * q.box_step], kMailboxDispatch);
            }
            return result;
        }
        if (wall_clock64() - t_start > kLaunchTimeoutTicks) break;
        __builtin_amdgcn_s_sleep(8);
    }
    if (lane == 0) atomicAdd(&a.counters[MPV_COUNTER_DEPENDENCY_TIMEOUT], 1u);     // must never happen
    return kTaskExit;
}

// Results one task leaves for another task of the same launch (which may run on another
// chiplet, behind another L2 cache): written through and read past the caches with relaxed
// device-scope atomics.  Order between them is the writer's business: it waits for its stores
// to be acknowledged (s_waitcnt vmcnt(0)) before the atomic that lets the reader start.
__device__ __forceinline__ void st_shared_f64(double* p, double v) {
    __hip_atomic_store(as_global(reinterpret_cast<unsigned long long*>(p)),
                       static_cast<unsigned long long>(__double_as_longlong(v)), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double ld_shared_f64(const double* p) {
    return __longlong_as_double(static_cast<long long>(__hip_atomic_load(
        as_global(reinterpret_cast<const unsigned long long*>(p)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)));
}

// ------------------------------------------------------------------ teams
//
// The G members of a team run the same task in lockstep on different vocabulary ranges: they
// execute the same scalar code on the same numbers (exchanged sums are added in the same order
// by every member, so they are bitwise equal everywhere) and therefore take the same branches;
// side effects (results, queue, counters) are the leader's (member 0).  What the leader alone
// can know (the task, whether teams are idle, a starting weight) travels with the task word or
// with the first exchange of the task.
// An exchange: every member writes up to kExchWords words into its own 64-byte line of the
// team's area, each word tagged with the number of the exchange, and polls the other lines until
// every word carries that number.  Two areas alternate: a member can be at most one exchange
// ahead of the slowest (it needs everybody's words of exchange s to finish s, see exchange_waits),
// so the words of exchange s are never overwritten before everybody has read them.

struct Team {
    int id, member, size;
    unsigned seq;                    // number of the last exchange; whether the team runs on one chiplet (before_first_exchange)
    unsigned tseq;                   // task words seen
    unsigned long long* area;        // [2][size][kExchWords]
    unsigned long long* task_word;   // [2]
    long long t_start;               // wall clock at the start of the launch
    int dead;                        // a partner never answered: results are invalid, every wait is skipped
};

// What the members of a team tell each other.  Loads of device scope are served by the chiplet's L2, past the first-level
// caches; so where every member runs on one chiplet (checked as they arrive, by the hardware's own number: teams are laid
// out for it, but nothing promises where a workgroup runs) the words need not go any further than that L2 either, which
// a store of workgroup scope says.  A store of device scope writes through to memory and takes the line out of
// the L2, and every reader waits for memory: an exchange between 2 / 6 / 12 / 16 workgroups with nothing else to do took
// 0.68 / 0.70 / 0.84 / 1.02 us with it and takes 0.35 / 0.40 / 0.43 / 0.44.  (64 trees of V = 128256, Traversal, 139 -> 133 us a
// call; 32 of V = 262144 on teams of 16, SpecInfer, 79 -> 73; 256 of V = 151936, Traversal, 447 -> 433.)
// (uniform_i32, and the rare side of an exchange's wait marked as rare: the choice is one scalar branch then, not a masked
// one.  The code of a task is longer than the instruction cache, so that calls of single-member teams, which exchange
// nothing, paid for it: 35 trees of V = 1216, block efficiency, Traversal, 206 us before there was a choice, 211, now 207; 104 of
// V = 1152 170, 177, 170; 5 of V = 2737, a call, 48.6, 49.7, 49.2.)
__device__ __forceinline__ void st_team(const Team& t, unsigned long long* p, unsigned long long v) {
    if (on_one_chiplet(static_cast<unsigned>(uniform_i32(static_cast<int>(t.seq))))) __hip_atomic_store(as_global(p), v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    else st_relaxed(p, v);
}
static_assert(kMaxTeam < (1 << kArrivedBits), "the counts of a team's arrivals fit their fields");
__device__ __forceinline__ int chiplet_here() { return __builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15; }      // (HW_REG_XCC_ID, 4 bits)

// What a workgroup carries from task to task, kept in LDS: the functions that run the tasks are
// not inlined, and state handed to them by reference would live in each lane's private memory.
// Written by the first lane of the first wave only (between two barriers of the task loop);
// whoever needs it takes a copy into registers.
struct LoopState {
    Team team;
    int asked;            // the leader has asked for its next task (mailbox says waiting or soon, or it has one: claimed)
    int own_task;         // leader: a task the team produced for itself, already announced (-1: none);
                          // member: the task it has already heard of (kNothingHeard: none)
    int own_flags;
    int previous_task;    // last task taken from the mailbox
    int claims;           // leader: there may be first tasks left to count off
    int claimed;          // leader: the first task the team has counted off ahead of time (kTaskNone: none)
    int finished;         // leader: the team has finished the last tree
    int kept_task;        // the node task this workgroup finished last (-1: none), its statistics and final state
    double kept_At, kept_Ad, kept_c;
    int want_claim;       // leader: the second wave is to count off a first task while the team samples
};
__shared__ LoopState g_loop;
constexpr int kNothingHeard = -4;
constexpr int kNotStarted = -5;           // own_task, every member: the team's first announcement is still to come

// The lane number, for numbers derived from it that are not worth keeping: computed where they are used, from nothing
// that would have to be kept, instead of ahead of the task loop (there they took so many registers that others went to
// private memory, and a reload waits for every row in flight).  With this in estimate_wave and in the words of the task's
// announcement too, and two more numbers computed where they are used (first_task, the children's exponent), the node
// tasks' loop has no private-memory access: 256 trees of 41 nodes, V = 151936, Traversal 452 -> 441 us, 64 trees of 15
// nodes, V = 128256, SpecInfer 83 -> 80, one tree of V = 1500, Traversal 61 -> 56.
__device__ __forceinline__ int lane_here() {
    int lane;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(lane));
    return lane;
}

// The node task's exchanges (first wave only) stay in registers: lane 16 r + m looks after member m, so that
// the members' numbers meet in reductions along a row of 16 lanes, and a member's own numbers do not travel.
// The sampling task's go the same way.  (Through LDS, one member after the other, the statistics of a team of 8 took
// 1.15 us from the last word's arrival to the logarithms, now 0.3.)
static_assert(kMaxTeam <= kTeamRow, "a row of lanes holds a team");

// Lane l < count sends word l; the lanes of the first ROWS rows, and those with `also` set, receive the words at[] of member
// lane & 15 into got[] (a member's own are there already).  Returns whether a partner failed to answer.
template <int ROWS, int COUNT>
__device__ __forceinline__ int swap_words(const Team& t, unsigned mine, int count, const int (&at)[COUNT], unsigned (&got)[COUNT], bool also = false) {
    const int lane = lane_here();
    unsigned long long* const base = t.area + static_cast<size_t>(exchange_area(t.seq)) * t.size * kExchWords;
    if (lane < count) st_team(t, base + t.member * kExchWords + lane, (static_cast<unsigned long long>(t.seq) << 32) | mine);
    int dead = t.dead;
    if (exchange_waits<ROWS>(lane, t.size, also) && (lane & 15) != t.member) {
        const unsigned long long* const line = base + (lane & 15) * kExchWords;
        for (unsigned spin = 1; !dead; ++spin) {
            unsigned long long v[COUNT];
            bool there = true;
#pragma unroll
            for (int i = 0; i < COUNT; ++i) v[i] = ld_relaxed(line + at[i]);
#pragma unroll
            for (int i = 0; i < COUNT; ++i) {
                there = there && static_cast<unsigned>(v[i] >> 32) == t.seq;
                got[i] = static_cast<unsigned>(v[i]);
            }
            if (there) break;
            if (__builtin_expect((spin & 31u) == 0u, 0) && wall_clock64() - t.t_start > kLaunchTimeoutTicks) dead = 1;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    return __ballot(dead != 0) != 0ull;
}

// a partner has not answered: counted once, and everybody leaves at the next occasion
__device__ __forceinline__ void note_dead(Team& t, int dead) {
    if (dead && !t.dead && threadIdx.x == 0) {
        atomicAdd(&lds_launch().a.counters[MPV_COUNTER_DEPENDENCY_TIMEOUT], 1u);
        st_relaxed(&lds_launch().ws.qctl[2], 1);
    }
    t.dead = dead;
}

// reductions along the rows of 16 lanes (every lane gets its row's result, in a fixed order)
__device__ __forceinline__ float row_max(float v) {
    v = fmaxf(v, dpp_f32<0xB1>(v));
    v = fmaxf(v, dpp_f32<0x4E>(v));
    v = fmaxf(v, dpp_f32<0x124>(v));
    return fmaxf(v, dpp_f32<0x128>(v));
}
__device__ __forceinline__ double row_sum(double v) {
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    v += dpp_f64<0x124>(v);
    return v + dpp_f64<0x128>(v);
}

__device__ __forceinline__ unsigned half_of(double v, int hi) {
    return static_cast<unsigned>(hi ? __double2hiint(v) : __double2loint(v));
}
// task word flags (leader -> members)
constexpr int kFlagIdle = 1;          // teams were idle after the last round of dispatching
constexpr int kFlagOneChiplet = 2;    // the first announcement: every member runs on one chiplet
constexpr int kFlagStopShift = 8;     // a sampling task: the node where the walk stopped, plus one (0: not known)

// The leader tells the others which task it has taken.  Every task announced this way contains at
// least one exchange, so the leader cannot announce the next before everybody has read this one.
__device__ __forceinline__ void team_announce(Team& t, int task, int flags) {
    t.tseq++;
    if (t.size == 1) return;
    if (const int half = lane_here(); half < 2) {
        const unsigned long long tag = static_cast<unsigned long long>(t.tseq) << 32;
        st_team(t, t.task_word + half, tag | static_cast<unsigned>(half == 0 ? task : flags));
    }
}
// The others wait for it (first wave; returns the same in every lane).  kTaskExit on a timeout.
// first: the team's first task, which its last member to arrive announces to all of them; a team that
// is still incomplete when the launch ends leaves by the exit flag (it has no task).
template <bool FIRST = false>
__device__ __forceinline__ int team_listen(Team& t, int& flags, const Workspace& ws) {
    t.tseq++;
    unsigned long long v = 0ull;
    int ok = 1;
    if (const int half = lane_here(); half < 2) {
        const unsigned long long* const word = (FIRST ? t.area + 1 : t.task_word) + half;
        for (unsigned spin = 1;; ++spin) {
            // (the exit flag is looked at rarely: its line is the one that the first tasks are counted on)
            const int leave = FIRST && (spin & 31u) == 0u ? ld_relaxed(&ws.qctl[2]) : 0;
            v = ld_relaxed(word);
            if ((v >> 32) == t.tseq) break;
            if (leave != 0 || wall_clock64() - t.t_start > kLaunchTimeoutTicks) { ok = 0; break; }
            __builtin_amdgcn_s_sleep(FIRST ? 1 : 2);
        }
    }
    const int all_ok = __ballot(!ok) == 0ull;
    const int task = __builtin_amdgcn_readlane(static_cast<int>(static_cast<unsigned>(v)), 0);
    flags = __builtin_amdgcn_readlane(static_cast<int>(static_cast<unsigned>(v)), 1);
    if (FIRST) {
        t.seq = before_first_exchange(all_ok && (flags & kFlagOneChiplet) != 0);
        flags &= ~kFlagOneChiplet;
    }
    return all_ok ? task : kTaskExit;
}

// ------------------------------------------------------------------ node task

// Double-precision scalar steps between the sweeps, as calls: their registers are then theirs alone
// and the part of the row pair a task keeps in registers stays where it is.
__device__ __forceinline__ double cold_exp2(double x) { return exp2(x); }
// 2^x for a probability (x <= a few): the whole part of x goes into the exponent, the rest through
// the hardware's float 2^f (relative error about 1e-7, far inside what a test probability needs):
// a dozen instructions on the first wave's path instead of the library routine's hundred.
__device__ __forceinline__ double probability_exp2(double x) {
    if (!(x > -1000.0)) return 0.0;                    // (also -inf and NaN)
    const double n = rint(x);
    const float f = static_cast<float>(x - n);         // [-0.5, 0.5]
    return ldexp(static_cast<double>(fast_exp2(f)), static_cast<int>(n));
}
__device__ __forceinline__ double cold_log2(double x) { return log2(x); }
__device__ __forceinline__ ResidualConsts cold_residual_consts(double At, double Ad, double c) { return residual_consts(At, Ad, c); }
// a comparison of numbers that are the same in every lane: a scalar branch, not a masked one
__device__ __forceinline__ bool all_alike(bool x) { return __builtin_amdgcn_ballot_w64(x) != 0ull; }
// The constants that a draw weighs a pair with.  c = 0 (nothing has been taken away from p): the draft row is left out, as
// one that is masked throughout has no partition, and 0 times one of its terms would be no number.
__device__ __forceinline__ ResidualConsts draw_consts(double At, double Ad, double c) {
    const bool use_d = all_alike(c > 0.0);
    ResidualConsts r = residual_consts(At, use_d ? Ad : 0.0, use_d ? c : 0.0);
    if (!use_d) r.nAd = -INFINITY;
    return r;
}
// x^k for a small whole k
__device__ __forceinline__ double int_power(double x, int k) {
    double r = 1.0;
    for (int i = 0; i < k; ++i) r *= x;
    return r;
}


// (defined below) walk and bonus token of tree b, or one draw of a token-following walk, by the
// whole team; returns the task that follows from it (-1: none; the same in every lane of every member)
template <class E, int METHOD>
__device__ __attribute__((noinline)) int sample_task(int b_in, int stop_in);

// (defined below) draws of a top-down walk of tree b, from node n on; returns the task that follows (-1: none)
template <class E>
__device__ __attribute__((noinline)) int draw_walk(int b_in, int n_in, int row_in, int there_in);

// (defined below) expected block efficiency of tree b from the per-node results, by the first wave
template <int METHOD>
__device__ __forceinline__ void estimate_wave(const TreeDesc& tree, const Workspace& ws, const Args& a, int b);

// One node task (or the resumed task of the node where the tree branches), by every member of the
// team.  A function of its own, not inlined: what it keeps in registers (its part of the row pair)
// then competes only with its own scalar steps for registers, not with the dispatcher or the sampler.
//
// Inside a workgroup the four waves split the work in another way as well: all four sweep their
// share of the part, but everything scalar (statistics, weights, the child loop, the exchange with
// the other members, what follows from the task) is the first wave's alone.  The other waves wait
// at a barrier for the next sweep's constants: they issue no instruction meanwhile, which leaves
// the compute unit to the sweeps of the other workgroups that live on it.
//   first wave:   ... scalar step ... | write command | barrier B | sweep | partial | barrier A | read partials ...
//   other waves:                                      | barrier B | sweep | partial | barrier A | (loop)
// asked / own_task / own_flags: the leader's notes for the task loop (has the team asked for its
// next task; the task it is to run next, already announced to the team, and its flags); only the
// first wave's copies matter.

// The barrier between the waves of a workgroup inside a node task.  What the waves hand each other
// there goes through LDS only (the command, partial sums, the children's scalars), so the barrier
// waits for this wave's LDS operations and nothing else: __syncthreads() would also wait for every
// global load in flight, i.e. for the rows of the next task that have just been asked for.
__device__ __forceinline__ void task_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

constexpr int kCmdTask = 5;
constexpr int kCmdDone = 0;          // the task is over
constexpr int kCmdMass = 1;          // sum (p - rho q)_+
constexpr int kCmdMassSlope = 2;     // the same and sum_{p > rho q} rho q       (SpecTr's root search)
constexpr int kCmdAcceptance = 3;    // the NSS / Naive acceptance-rate sum      (acceptance rates only)
constexpr int kCmdTiles = 6;         // a draw from the pair on chip comes next: the masses of its tiles (top-down rules)

struct SweepCmd {
    int kind;
    float nAt, nAd, rho;             // constants of the residual sweeps
    float sp, sq;                    // acceptance sweep: scale factors of p and q
    int m, naive;                    // acceptance sweep: exponent, which formula (kCmdTask: m = the task)
    int claim;                       // a sweep: the second wave counts off a first task meanwhile (g_claim_number)
    int b, n;                        // kCmdTask: its tree and node;  a sweep: n = the node of `next`, in the same tree
    int ahead, ahead_row;            // kCmdTask: the node of this tree whose rows are asked for when its first sweep is over
                                     // (ahead_row: only the target's, for a draw), by the waves that then wait (short_part_kernel)
    int next;                        // a sweep: the task this team goes on with when the sweep was the
                                     // current task's last (-1: not known); each wave asks for its share
                                     // of that task's rows as soon as it is done with its share of the sweep
};
__shared__ SweepCmd g_cmd;
__shared__ int g_claim_number;
// A draw (see draw_walk).
struct DrawShared {
    float tile[kDrawTiles];          // the masses of this member's tiles, in units of 2^(g_sh.partf of the wave)
    float nAt, nAd, rho;             // a pair: the constants they were weighed with
    int there;                       // the row lies in LDS already (RetainedPart::ask_ahead)
    int pending, b, n, row;          // the node task that has just ended has come to this draw: tree, node, from a target row alone
    int owner, in_tile, token, next;
    double rem, total;               // of the tile that holds the target: mass to cover inside it; the whole row's, in the same unit
};
__shared__ DrawShared g_draw;

// One sweep over the part on chip as the command says; the wave's partial sums go to g_sh.part.
template <class E, int KIND, class PAIR>
__device__ __forceinline__ void run_sweep(PAIR& pair, const SweepCmd& cmd, float k32, int wave, int lane) {
    constexpr bool ACCEPT = KIND == kKindAcceptance;
    constexpr bool SLOPE = method_of(KIND) != MPV_METHOD_TRAVERSAL;      // SpecTr's search exists in the top-down kernels only
    double s0 = 0.0, s1 = 0.0;
    if (SLOPE && cmd.kind == kCmdMassSlope) {
        ResidualMassSlopeRawF<E> f;
        f.init();
        f.k32 = k32; f.nAt = cmd.nAt; f.nAd = cmd.nAd; f.rho = cmd.rho;
        pair.replay(f);
        s0 = static_cast<double>(f.acc0) + static_cast<double>(f.acc1);
        s1 = static_cast<double>(f.q0) + static_cast<double>(f.q1);
    } else if (ACCEPT && cmd.kind == kCmdAcceptance) {
        AcceptanceF<E> f;
        f.init(k32, cmd.nAt, cmd.nAd, cmd.sp, cmd.sq, cmd.m, cmd.naive != 0);
        pair.replay(f);
        s0 = static_cast<double>(f.acc0) + static_cast<double>(f.acc1);
    } else {
        ResidualMassRawF<E, ACCEPT> f;
        f.init(k32, cmd.nAt, cmd.nAd, cmd.rho);
        pair.replay(f);
        s0 = f.total();
    }
    s0 = wave_sum(s0);
    if (SLOPE) s1 = wave_sum(s1);
    if (lane == 0) { g_sh.part[wave][0] = s0; g_sh.part[wave][1] = s1; }
}

// First wave, after barrier A: the workgroup's sums of the last sweep (one or two), exchanged and added
// over the team.  Every lane of the first wave of every member gets the same bits.
template <bool TWO>
__device__ __forceinline__ void collect_sums(Team& t, double& s0, double& s1) {
    const int lane = lane_here(), row = lane >> 4, m = lane & 15;
    t.seq++;
    // row 0 of the lanes looks after the first sum, row 1 after the second; each quad adds up the four waves
    double v = g_sh.part[lane & 3][TWO ? row & 1 : 0];
    v += dpp_f64<0xB1>(v);
    v += dpp_f64<0x4E>(v);
    if (t.size > 1) {
        const double other = TWO ? lane_f64(v, 16) : 0.0, one = TWO ? lane_f64(v, 0) : v;
        const unsigned mine = half_of(TWO && (lane & 2) ? other : one, lane & 1);
        unsigned got[2] = {half_of(v, 0), half_of(v, 1)};
        const int at[2] = {2 * row, 2 * row + 1};
        note_dead(t, swap_words<TWO ? 2 : 1>(t, mine, TWO ? 4 : 2, at, got));
        v = row_sum(m < t.size && !t.dead ? __hiloint2double(static_cast<int>(got[1]), static_cast<int>(got[0])) : 0.0);
    }
    s0 = lane_f64(v, 0);
    s1 = TWO ? lane_f64(v, 16) : 0.0;
}

// First wave, after barrier A of the statistics sweep: the waves' partials (g_sh.part, partf) become the log2-partitions of the
// two rows; a0 is the leader's starting weight (WEIGHT; what the other members bring is ignored).
template <bool WEIGHT>
__device__ __forceinline__ void collect_stats(Team& t, double& a0, double& At, double& Ad) {
    const int lane = lane_here(), row = lane >> 4, m = lane & 15;
    t.seq++;
    // row 0: target, row 1: draft; each quad brings the four waves to the largest reference
    const float Mw = g_sh.partf[lane & 3][row & 1];
    double s = g_sh.part[lane & 3][row & 1];
    float M = fmaxf(Mw, dpp_f32<0xB1>(Mw));
    M = fmaxf(M, dpp_f32<0x4E>(M));
    s *= static_cast<double>(fast_exp2(Mw - M));
    s += dpp_f64<0xB1>(s);
    s += dpp_f64<0x4E>(s);
    if (t.size > 1) {
        // words: the two references, the two sums, the weight
        const float Mt = lane_f32(M, 0), Md = lane_f32(M, 16);
        const double st = lane_f64(s, 0), sd = lane_f64(s, 16);
        const double of_pair = lane < 4 ? st : lane < 6 ? sd : a0;
        unsigned mine = half_of(of_pair, lane & 1);
        if (lane < 2) mine = __float_as_uint(lane ? Md : Mt);
        unsigned got[3] = {half_of(s, 0), __float_as_uint(M), half_of(s, 1)};
        if (WEIGHT && row == 2) { got[0] = half_of(a0, 0); got[2] = half_of(a0, 1); }
        const int at[3] = {2 * row + 2, row < 2 ? row : 6, 2 * row + 3};
        note_dead(t, swap_words<2>(t, mine, WEIGHT ? 8 : 6, at, got, WEIGHT && lane == 32));
        const bool live = m < t.size && !t.dead;
        const float Mm = live ? __uint_as_float(got[1]) : OnlineLse::kFloor;
        M = row_max(Mm);
        s = row_sum(live ? __hiloint2double(static_cast<int>(got[2]), static_cast<int>(got[0])) * static_cast<double>(fast_exp2(Mm - M)) : 0.0);
        if (WEIGHT) a0 = __hiloint2double(__builtin_amdgcn_readlane(static_cast<int>(got[2]), 32), __builtin_amdgcn_readlane(static_cast<int>(got[0]), 32));
    }
    const double A = static_cast<double>(M) + cold_log2(s);          // both logarithms in one go, a row of lanes each
    At = lane_f64(A, 0);
    Ad = lane_f64(A, 16);
}

// the wave that has tile t of a draw (see PartDraw; the elements at the row's ends are the first wave's)
__device__ __forceinline__ int draw_wave(int t) { return t == 0 ? 0 : (t - 1) % kTaskWaves; }

template <class E> using TaskPart = RetainedPart<E, kTaskBlock, kRegVecs, kLdsVecs>;
template <class E> using TaskDraw = PartDraw<E, kTaskBlock, kRegVecs, kLdsVecs>;

template <class E, int KIND>
__device__ __attribute__((noinline)) void run_node_task(int task_in, int flags_in) {
    using T = typename E::T;
    constexpr bool ACCEPT = KIND == kKindAcceptance, SHORT = KIND == kKindShort, STAGED = SHORT || KIND == kKindShortAll;
    constexpr int METHOD = method_of(KIND);
    // Trees with shapes of their own: a task of another tree has its tables loaded here (Traversal), or it goes back to the
    // task loop, which loads them.  The top-down rules run this function through its whole length for SpecTr, and the loads
    // within it made plain batches of many trees slower (Naive, 204 trees of V = 7872: 246 us, 237 without); Traversal
    // has no such cost, and going back would make 256 trees of V = 151936 slower (538 us, 531).
    constexpr bool kShapeInTask = !ACCEPT && METHOD == MPV_METHOD_TRAVERSAL;
    constexpr bool DRAWS = KIND == kKindWalk || SHORT;
    const Args& a = lds_launch().a;
    const Workspace& ws = lds_launch().ws;
    const QueuePlan& q = lds_launch().q;
    const TreeDesc& tree = g_tree;
    // (what arrives as an argument arrives in vector registers: back to scalar ones)
    int task = uniform_i32(task_in), flags = uniform_i32(flags_in);
    const int wave = uniform_i32(static_cast<int>(threadIdx.x) / kWave), lane = threadIdx.x & (kWave - 1);
    uint4* const lds_t = g_rows;
    uint4* const lds_d = g_rows + kLdsVecs * kTaskBlock;
    const int B = uniform_i32(a.B), N = uniform_i32(a.N), V = uniform_i32(a.V);
    const float k32 = uniform_f32(a.k32);
    const int member = uniform_i32(g_loop.team.member), team_size = uniform_i32(g_loop.team.size);

    // what a task number stands for (tree, node: made scalar explicitly, so that the table lookups
    // that follow have uniform addresses)
    const T* const zt0 = uniform_ptr(static_cast<const T*>(a.zt));
    const T* const zd0 = uniform_ptr(static_cast<const T*>(a.zd));
    const int part_vecs = uniform_i32(q.part_vecs);
    struct NodeView { int b, n; bool resumed; size_t bn; const T* zt; const T* zd; };
    auto view_at = [&](int b, int n, bool resumed) __attribute__((always_inline)) -> NodeView {
        NodeView v;
        v.resumed = resumed;
        v.b = uniform_i32(b);
        v.n = uniform_i32(n);
        v.bn = static_cast<size_t>(v.b) * N + v.n;
        v.zt = zt0 + v.bn * V;
        v.zd = zd0 + v.bn * V;
        return v;
    };
    auto view_of = [&](int t) __attribute__((always_inline)) -> NodeView {
        if (t >= B * N + B) return view_at(t - (B * N + B), tree.split_node, true);
        int nodes_per_tree = N;                           // (its reciprocal is not kept across tasks)
        asm volatile("" : "+s"(nodes_per_tree));
        return view_at(t / nodes_per_tree, t % nodes_per_tree, false);
    };

    auto tree_of = [&](int t) __attribute__((always_inline)) -> int {
        int nodes_per_tree = N;
        asm volatile("" : "+s"(nodes_per_tree));
        return tree_of_task(t, B, nodes_per_tree);
    };

    // ---- the part of the pair this member keeps on chip while a task runs
    RetainedPart<E, kTaskBlock, kRegVecs, kLdsVecs, STAGED> pair;
    auto weigh_tiles = [&](float nAt, float nAd, float rho) __attribute__((always_inline)) {
        PartDraw<E, kTaskBlock, kRegVecs, kLdsVecs, STAGED> d(pair);
        d.f.init(k32, nAt, nAd, rho);
        d.weigh_pair(g_draw.tile, wave, lane);
        if (lane == 0) g_sh.partf[wave][0] = 0.f;
    };

    if (wave != 0) {
        // ---- a sweeping wave does what the first wave commands: it takes up a task (loads its
        //      share of the pair and runs the statistics sweep) or sweeps once more
        int asked_for = -1;                               // the task whose rows this wave has asked for already
        int ahead = -1;                                   // the task whose rows are in LDS
        auto take_up = [&](int t, const NodeView& nv) __attribute__((always_inline)) {
            int tid_l = threadIdx.x;
            asm volatile("" : "+v"(tid_l));     // per-task copy: nothing derived from it is kept across tasks
            pair.setup(nv.zt, nv.zd, V, lds_t, lds_d, tid_l, member, team_size, part_vecs);
            if (!SHORT || t != ahead) pair.issue_loads();
            ahead = -1;
            asked_for = t;
        };
        for (;;) {
            task_barrier();                                // B: the command is there
            const SweepCmd cmd = g_cmd;
            const int kind = uniform_i32(cmd.kind);
            if (kind == kCmdDone) {
                if (SHORT || asked_for >= 0) wait_memory();        // (asked for in vain, or for the draw: nothing may land in LDS after this)
                return;
            }
            if (kind == kCmdTask) {
                const int t = uniform_i32(cmd.m);
                if (SHORT) {                              // what has been asked for ahead is there, or at least out of the way:
                    wait_memory();                        // each wave waits for its own, then all of them for each other
                    task_barrier();                       // C
                }
                if (asked_for != t) take_up(t, view_at(cmd.b, cmd.n, false));
                asked_for = -1;
                PairStatsRawF<E, ACCEPT> f;
                f.t.init(); f.d.init(); f.k32 = k32;
                pair.first_pass(f);
                f.t.finish(); f.d.finish();
                const float Mt_w = wave_max(f.t.mk), Md_w = wave_max(f.d.mk);
                const double st_w = wave_sum((f.t.s > 0.f) ? static_cast<double>(f.t.s * fast_exp2(f.t.mk - Mt_w)) : 0.0);
                const double sd_w = wave_sum((f.d.s > 0.f) ? static_cast<double>(f.d.s * fast_exp2(f.d.mk - Md_w)) : 0.0);
                if (lane == 0) {
                    g_sh.partf[wave][0] = Mt_w; g_sh.partf[wave][1] = Md_w;
                    g_sh.part[wave][0] = st_w; g_sh.part[wave][1] = sd_w;
                }
            } else if (DRAWS && kind == kCmdTiles) {
                weigh_tiles(uniform_f32(cmd.nAt), uniform_f32(cmd.nAd), uniform_f32(cmd.rho));
            } else {
                const bool claims_now = wave == 1 && uniform_i32(cmd.claim) != 0;
                int claim_number = 0;
                if (claims_now && lane == 0) claim_number = claim_first(ws);
                run_sweep<E, KIND>(pair, cmd, k32, wave, lane);
                if (claims_now && lane == 0) g_claim_number = claim_number;
                const int nx = uniform_i32(cmd.next);       // (Traversal only)
                if (nx >= 0) take_up(nx, view_at(cmd.b, cmd.n, false));     // this wave's slots are free again: the next task's rows
            }
            task_barrier();                                // A: this wave's partial sums are there
            if (SHORT && kind == kCmdTask) {
                // every wave has its vectors in registers: the LDS is free
                const NodeView nx = view_at(cmd.b, cmd.ahead, false);
                TaskPart<E> then;
                then.setup(nx.zt, nx.zd, V, lds_t, lds_d, threadIdx.x, member, team_size, part_vecs);
                const bool row = uniform_i32(cmd.ahead_row) != 0;
                then.ask_ahead(wave - 1, kTaskWaves - 1, !row);
                ahead = row ? -1 : uniform_i32(cmd.b) * N + uniform_i32(cmd.ahead);
            }
        }
    }

    // ================================================================ the first wave
    Team team = uniform_struct(g_loop.team);           // in registers while the tasks run
    bool asked = uniform_i32(g_loop.asked) != 0, claims = uniform_i32(g_loop.claims) != 0;
    int claimed = uniform_i32(g_loop.claimed);
    // a first task to be counted off, or being counted off by the second wave while it sweeps
    bool claim_wanted = false, claim_pending = false;
    int own_task = -1, own_flags = 0;
    const bool leader = team.member == 0;
    const bool lead = leader && lane == 0;            // the one lane that talks to the rest of the launch
    // The leader asks for the team's next task ahead of time: a first task, while there are any, else
    // the dispatcher.
    auto ask_ahead = [&]() __attribute__((always_inline)) {
        if (claims) {
            claim_wanted = true;
        } else if (lane == 0) {
            st_relaxed(&ws.mailbox[team.id * q.box_step], kMailboxSoon);
        }
        asked = true;
    };
    auto settle_claim = [&]() __attribute__((always_inline)) {
        if (!claim_wanted && !claim_pending) return;
        int number = 0;
        if (claim_pending) number = g_claim_number;
        else if (lane == 0) number = claim_first(ws);
        claim_wanted = claim_pending = false;
        claimed = first_task(q, a, uniform_i32(number));
        if (claimed == kTaskNone) {
            claims = false;
            if (lane == 0) st_relaxed(&ws.mailbox[team.id * q.box_step], kMailboxSoon);
        }
    };
    // the task that was asked for, if it is there (-1); it is the team's then
    auto answer = [&]() __attribute__((always_inline)) -> int {
        settle_claim();
        int t = claimed;
        if (t == kTaskNone) {
            if (claims) return -1;
            const int previous = uniform_i32(g_loop.previous_task);
            if (lane == 0) t = ld_relaxed(&ws.mailbox[team.id * q.box_step]);
            t = uniform_i32(t);
            if (t < 0 || t == previous) return -1;
            if (lane == 0) g_loop.previous_task = t;
        }
        claimed = kTaskNone;
        asked = false;
        return t;
    };
    // What the scalar steps look up is kept in registers, a node (or a child) per lane: read from LDS or memory
    // one after the other, when needed, it was most of the time between the sweeps.
    const int lazy = DRAWS ? 1 : uniform_i32(a.lazy), walk = uniform_i32(a.walk);
    auto estimate = [&]() __attribute__((always_inline)) { return !DRAWS && a.estimate != 0; };
    unsigned nodes = 0u;                              // the tree's tables, lane n: see below
    int tokens = -1;                                  // lane n: token and uniform of node n
    float uniforms = 2.f;
    int tree_in_regs = -1;                            // the tree they belong to
    unsigned children = 0u;                           // lane j (and 32 + j): node word of child j of the task's node, its number instead of the list entry
    unsigned long long token_ok = 0ull;               // bit j: child j's token is in range
    T logits = 0;                                     // lane j: child j's target logit, lane 32 + j: draft logit
    constexpr int kOff = 5, kEntry = 11, kRank = 17, kLow = 23, kClass = 29;      // nchild: bits 0..4
    auto field = [](unsigned word, int at, unsigned mask) __attribute__((always_inline)) { return static_cast<int>((word >> at) & mask); };
    auto node_word = [&](int node) __attribute__((always_inline)) { return static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(nodes), node)); };
    auto n_children = [&](int node) __attribute__((always_inline)) { return field(node_word(node), 0, 31u); };
    auto load_tables = [&]() __attribute__((always_inline)) {
        nodes = 0u;
        const int own = lane_here();
        if (own < N)
            nodes = static_cast<unsigned>(tree.nchild[own]) | static_cast<unsigned>(tree.child_off[own]) << kOff |
                    static_cast<unsigned>(tree.child_list[own]) << kEntry | static_cast<unsigned>(tree.rank[own]) << kRank |
                    static_cast<unsigned>(tree.sub_lo[own]) << kLow | static_cast<unsigned>(tree.cls[own]) << kClass;
    };
    load_tables();
    auto gather = [&](int from_lane, int v) __attribute__((always_inline)) { return __builtin_amdgcn_ds_bpermute(from_lane << 2, v); };
    // Walks draw their tokens in draw_walk, which is called next; a pair's tiles are weighed here, where it is on chip.
    // (On long parts, what the compiler knows makes paths of their own, which take dozens of registers to private memory.)
    auto draw_here = [&]() __attribute__((always_inline)) {
        if constexpr (!DRAWS || SHORT) return DRAWS;
        int x = 1;
        asm volatile("" : "+s"(x));
        return x != 0;
    };
    // The rows asked for ahead (see start_task): their node, -1: none; only a leaf's target row; the task they belong to.
    int ahead_node = -1, ahead_task = -1;
    bool ahead_row = false, there = false;            // (there: of the task under way: its rows were there when it was taken up)
    // Takes a task up: the other waves are told, this wave's share of the pair is asked for, then the children's logits
    // (tokens and uniforms once per tree, so that nothing waits for a load that depends on a load).
    auto start_task = [&](const NodeView& v, int t) __attribute__((always_inline)) {
        const bool ready = SHORT && t == ahead_task;
        if (SHORT) {
            // What comes next if it is accepted: the first child (its rows, or a leaf's target row).
            ahead_node = field(node_word(field(node_word(v.n), kOff, 63u)), kEntry, 63u);
            ahead_row = n_children(ahead_node) == 0;
            ahead_task = !ahead_row ? v.b * N + ahead_node : -1;
            if (lane == 0) { g_cmd.ahead = ahead_node; g_cmd.ahead_row = ahead_row ? 1 : 0; }
        }
        if (lane == 0) { g_cmd.kind = kCmdTask; g_cmd.m = t; g_cmd.b = v.b; g_cmd.n = v.n; }
        task_barrier();                                    // B: the other waves take the task up
        if (SHORT) task_barrier();                         // C: the LDS is theirs to write
        int tid_l = threadIdx.x;
        asm volatile("" : "+v"(tid_l));     // per-task copy: nothing derived from it is kept across tasks
        pair.setup(v.zt, v.zd, V, lds_t, lds_d, tid_l, member, team_size, part_vecs);
        if (ACCEPT) {
            pair.issue_loads();
            return;
        }
        const bool new_tree = tree_in_regs != v.b;
        tree_in_regs = v.b;
        if (new_tree) {
            const size_t at = static_cast<size_t>(v.b) * N + min(lane_here(), N - 1);
            tokens = as_global(a.tokens)[at];
            if (!estimate()) uniforms = as_global(a.uniforms)[at];
        }
        there = ready;
        if (!ready) pair.issue_loads();
        // (lanes read each other's registers here, not LDS: the compiler would wait for the loads that go there)
        const int own = lane_here(), j = own & 31, k = n_children(v.n);
        const int child = field(static_cast<unsigned>(gather(field(node_word(v.n), kOff, 63u) + j, static_cast<int>(nodes))), kEntry, 63u);
        children = (static_cast<unsigned>(gather(child, static_cast<int>(nodes))) & ~(63u << kEntry)) | static_cast<unsigned>(child) << kEntry;
        const int x = gather(child, tokens);
        const bool ok = j < k && x >= 0 && x < V;
        token_ok = __ballot(ok);
        logits = as_global(own < 32 ? v.zt : v.zd)[ok ? x : 0];
    };
    // A task taken up before it was certain (the task this team is most likely to run next,
    // started while the leader still settles what follows from the last one), -1: none.
    int started = -1;
    // Outcomes settled by tasks that handed on to a child's task directly (see the end of the
    // task): published by the first task that goes the long way.  And the weight such a child
    // starts with (Traversal), known here without asking memory; negative: not known.
    unsigned long long chain_settled = 0ull, chain_accepted = 0ull;
    double a0_known = -1.0;
    int chained = -1;                                 // the node of the task handed on to (same tree)
    // One node task after the other, for as long as the team knows its next one itself (the task
    // a node task hands to its own team: a child's, or the rest of the node where the tree
    // branches): no way back through the task loop, no queue in between.
    for (;;) {
    {
    // (a task that is under way already belongs to the tree of the task before)
    if (kShapeInTask && started != task && uniform_i32(a.per_tree)) {
        load_shape(reinterpret_cast<const unsigned long long*>(ws.aux), N, tree_of(task));
        load_tables();
    }
    const NodeView nv = chained >= 0 ? view_at(tree_in_regs, chained, false) : view_of(task);
    chained = -1;
    const bool resumed = nv.resumed;
    const int b = nv.b, n = nv.n, k = n_children(n), off = field(node_word(n), kOff, 63u);
    auto child_of = [&](int j) __attribute__((always_inline)) { return field(node_word(off + j), kEntry, 63u); };
    (void)child_of;
    const size_t bn = nv.bn;
    const T* const zt = nv.zt;
    const T* const zd = nv.zd;
    (void)zt; (void)zd;
    own_task = -1; own_flags = 0;
    if (started != task) start_task(nv, task);            // (else: under way since the end of the task before)
    started = -1;
    double At_ = 0.0, Ad_ = 0.0, wa = 1.0;            // log2-partitions of the two rows; the node's weight
    int next_hint_node = 0;
    int next_hint = -1;                               // goes out with a sweep command (SweepCmd::next)
    // one more sweep by all four waves; the team's sums come back
    auto sweep = [&](int kind, const ResidualConsts& rc, float sp, float sq, int m, int naive, double& s0, double& s1) __attribute__((always_inline)) {
        if (lane == 0) {
            g_cmd.kind = kind; g_cmd.nAt = rc.nAt; g_cmd.nAd = rc.nAd; g_cmd.rho = rc.rho;
            g_cmd.sp = sp; g_cmd.sq = sq; g_cmd.m = m; g_cmd.naive = naive; g_cmd.next = next_hint;
            g_cmd.b = b; g_cmd.n = next_hint_node;
            g_cmd.claim = claim_wanted ? 1 : 0;
        }
        claim_pending = claim_pending || claim_wanted;
        claim_wanted = false;
        task_barrier();                                    // B
        SweepCmd cmd;
        cmd.kind = kind; cmd.nAt = uniform_f32(rc.nAt); cmd.nAd = uniform_f32(rc.nAd); cmd.rho = uniform_f32(rc.rho);
        cmd.sp = sp; cmd.sq = sq; cmd.m = m; cmd.naive = naive; cmd.next = -1;
        run_sweep<E, KIND>(pair, cmd, k32, 0, lane);
        task_barrier();                                    // A
        if (kind == kCmdMassSlope) collect_sums<true>(team, s0, s1);
        else collect_sums<false>(team, s0, s1);
    };
    // W(c) for one c
    auto residual_mass = [&](double cc) __attribute__((always_inline)) -> double {
        const ResidualConsts rc = cold_residual_consts(At_, Ad_, cc);
        double s0, s1;
        sweep(kCmdMass, rc, 0.f, 0.f, 0, 0, s0, s1);
        return uniform_f64(uniform_f64(rc.scale) * s0);
    };

    if (lead) atomicAdd(&a.counters[resumed ? MPV_COUNTER_NODE_TASKS_RESUMED : MPV_COUNTER_NODE_TASKS_RUN], 1u);
    // are teams idle?  Asked now, needed when this task hands on to the next (the leader's business)
    int idle_now = 0;
    if (lead) idle_now = ld_relaxed(&ws.qctl[kCtlIdle]);
    const bool split_here = METHOD == MPV_METHOD_TRAVERSAL && lazy && !resumed && n == uniform_i32(tree.split_node);
    const bool idle_seen = (flags & kFlagIdle) != 0;

    // Traversal, only what is needed, and idle teams about: an only child's task is queued
    // now, ahead of its starting weight.  It reads its rows while this task reads its own and
    // then finds the weight published (or waits a moment for it), so that a chain of nodes
    // takes little more than one task's time.  If the weight turns out to be 0 it gives up.
    bool child_ahead = false;
    if (METHOD == MPV_METHOD_TRAVERSAL && lazy && k == 1 && !split_here && idle_seen) {
        const int cn = child_of(0);
        if (n_children(cn) > 0) {
            child_ahead = true;
            if (lead) append_task(tree, ws, field(node_word(cn), kClass, 1u), b * N + cn);
        }
    }

    // ---- softmax statistics of both rows: the one read of the pair from memory
    float un = 2.f;                                   // the node's own uniform
    {
        // Traversal: the starting weight comes from the parent's task, which published it
        // before it queued this task (or publishes it shortly, if this task was queued ahead).
        // The leader fetches it and passes it on with the statistics.  Value and "ready" flag
        // are one 64-bit word (a weight is never NaN), read and written with relaxed
        // device-scope atomics: no fence, no cache invalidation.  Asked for before the sweep:
        // the answer is there when the sweep is over.
        const bool wants_a0 = lead && METHOD == MPV_METHOD_TRAVERSAL && n != 0 && !(a0_known >= 0.0);
        unsigned long long bits = kNotReady;
        if (wants_a0) bits = ld_relaxed(reinterpret_cast<const unsigned long long*>(&ws.a0[bn]));
        PairStatsRawF<E, ACCEPT> f;
        f.t.init(); f.d.init(); f.k32 = k32;
        pair.first_pass(f, there);
        f.t.finish(); f.d.finish();
        double a0 = 1.0;
        if (wants_a0) {
            for (int spin = 0; spin < kMaxSpins && bits == kNotReady; ++spin) {
                if (wall_clock64() - team.t_start > kLaunchTimeoutTicks) break;
                __builtin_amdgcn_s_sleep(8);
                bits = ld_relaxed(reinterpret_cast<const unsigned long long*>(&ws.a0[bn]));
            }
            if (bits != kNotReady) {
                a0 = __longlong_as_double(static_cast<long long>(bits));
            } else {            // the parent's task never published it (must never happen): the subtree is written off
                a0 = 0.0;
                atomicAdd(&a.counters[MPV_COUNTER_DEPENDENCY_TIMEOUT], 1u);
            }
        }
        a0 = lane_f64(a0, 0);
        if (all_alike(a0_known >= 0.0)) a0 = a0_known;
        a0_known = -1.0;
        // lanes to their wave's largest reference, waves to the workgroup's, members to the team's
        const float Mt_w = wave_max(f.t.mk), Md_w = wave_max(f.d.mk);
        const double st_w = wave_sum((f.t.s > 0.f) ? static_cast<double>(f.t.s * fast_exp2(f.t.mk - Mt_w)) : 0.0);
        const double sd_w = wave_sum((f.d.s > 0.f) ? static_cast<double>(f.d.s * fast_exp2(f.d.mk - Md_w)) : 0.0);
        if (lane == 0) {
            g_sh.partf[0][0] = Mt_w; g_sh.partf[0][1] = Md_w;
            g_sh.part[0][0] = st_w; g_sh.part[0][1] = sd_w;
        }
        task_barrier();                                    // A: every wave's partials are there
        un = lane_f32(uniforms, n);
        collect_stats<METHOD == MPV_METHOD_TRAVERSAL>(team, a0, At_, Ad_);
        if (METHOD == MPV_METHOD_TRAVERSAL) wa = a0;
    }
    RowStat rt, rd;
    rt.A = At_; rd.A = Ad_; rt.m = 0.f; rd.m = 0.f;

    // ---- per-child scalars and one residual-mass reduction per child
    if (METHOD == MPV_METHOD_TRAVERSAL && lazy && n != 0 && !all_alike(wa > 0.0) && chain_settled == 0ull) {
        // queued ahead of its weight, which is 0: the parent has written off the whole subtree.
        // Nothing to do but to pass the news on to an only child queued ahead in turn.
        if (lead) {
            if (child_ahead) {
                const size_t bc = static_cast<size_t>(b) * N + child_of(0);
                st_relaxed(reinterpret_cast<unsigned long long*>(&ws.a0[bc]), static_cast<unsigned long long>(__double_as_longlong(0.0)));
            }
            wait_memory();
            atomicAdd(&ws.qctl[1], 1);
        }
        goto task_end;
    }
    double c = 0.0, W = 1.0;
    const double kd = static_cast<double>(k32);
    // p(x) and q(x) of every child's token at once: lane j has the target's, lane 32 + j the draft's
    static_assert(MPV_MAX_CHILDREN <= 32, "one lane per child and row");
    double pq_all;
    {
        float k_here = k32;                           // (widened here: as a double it is not kept across tasks)
        asm volatile("" : "+s"(k_here));
        pq_all = probability_exp2(static_cast<double>(E::load_one(&logits)) * static_cast<double>(k_here) - (lane_here() >= 32 ? Ad_ : At_));
    }
    // test outcomes this task settles, one bit per node at its position in postorder
    unsigned long long settled_bits = 0ull, accepted_bits = 0ull;
    int next_node = -1;                               // SpecInfer, only what is needed: the accepted child
    double own_w = 0.0;                               // ... and the weight it starts with
    int own_child = -1;                               // Traversal: index of the first child whose task is to be run
    bool paused = false;
    bool own_given = false;                           // that child's task was queued after all (some team is idle)
    // SpecTr (App. B, Alg. 3): the division factor rho* is the root of
    //   f(rho) = p_acc(rho) - rho beta(rho),  p_acc = 1 - (1 - beta)^k,  beta(rho) = sum_v min(p_v/rho, q_v)
    // on [1, k]; f decreases, f(1) >= 0 >= f(k).  Written with the sums of positive terms
    //   W(rho) = sum_v (p_v - rho q_v)_+   and   D(rho) = sum_v (q_v - p_v/rho)_+ = (W + rho - 1)/rho = 1 - beta,
    // f = W - D^k: no cancellation, so the sign of f is right even where |f| is far below the
    // rounding error of beta itself (p close to q, where f is nearly flat to the right of the root).
    // Each W is one sweep over the pair on chip, the same reduction the other rules use.  At the
    // root p_acc/beta = rho*, so the vector the token is drawn from, (p - gamma min(p/rho*, q))_+,
    // is (p - rho* q)_+ : the node's final state is simply c = rho*.
    // The paper's binary search is replaced by Newton's method from rho = 1, kept inside the
    // bracket [last rho with f > 0, first rho with f < 0] (a step that leaves it is replaced by the
    // midpoint); the sweep returns the slope with the value: W'(rho) = -sum_{p > rho q} q, and
    // D' = (W' + 1 - D)/rho.  Once a step is shorter than the tolerance the next point is put
    // just across, to close the bracket.  The same root in about seven sweeps instead of thirty
    // (f has a kink where the largest token switches sides and can be nearly flat beyond it:
    // there it takes more).
    double sp_rho = 1.0, sp_W = 1.0;
    if (METHOD == MPV_METHOD_SPECINFER && walk == 3) {
        constexpr double kTol = 3e-8;                 // relative width of the final bracket
        double lo = 1.0, hi = static_cast<double>(k);
        double x = 1.0, fx = 0.0, dfx = 0.0;
        const int evals = (k > 1) ? 64 : 1;
        for (int it = 0; it < evals; ++it) {
            if (it > 0) {
                double cand = 0.0;                    // outside the bracket: "no candidate"
                if (all_alike(dfx < 0.0)) {
                    const double step = -fx / dfx;
                    cand = x + step;
                    if (fabs(step) <= 0.5 * kTol * x) cand = fx > 0.0 ? x * (1.0 + kTol) : x * (1.0 - kTol);
                }
                if (!(cand > lo && cand < hi)) cand = 0.5 * (lo + hi);
                x = uniform_f64(cand);
            }
            const ResidualConsts rc = cold_residual_consts(rt.A, rd.A, x);
            double sum_w, sum_q;
            sweep(kCmdMassSlope, rc, 0.f, 0.f, 0, 0, sum_w, sum_q);
            const double scale = uniform_f64(rc.scale);
            const double Wx = uniform_f64(scale * sum_w);
            const double dWx = -uniform_f64(scale * sum_q) / x;       // the sweep added up rho q over {p > rho q}
            const double Dx = fmin(fmax((Wx + x - 1.0) / x, 0.0), 1.0);
            const double dDx = (dWx + 1.0 - Dx) / x;
            const double kk = static_cast<double>(k);
            fx = Wx - int_power(Dx, k);
            dfx = dWx - kk * int_power(Dx, k - 1) * dDx;
            sp_rho = x;
            sp_W = Wx;
            if (team.dead) break;
            if (it == 0) {
                if (!all_alike(fx > 0.0)) break;               // the root is 1 (also when k = 1)
            } else {
                if (all_alike(fx > 0.0)) lo = x;
                else if (all_alike(fx < 0.0)) hi = x;
                else break;
                if (all_alike(hi - lo <= kTol * hi)) break;
            }
        }
    }
    if (ACCEPT) {
        // Acceptance rate of this node (App. C): the chance that the solver's output is one of k draft
        // tokens drawn i.i.d. from q.  For SpecInfer and SpecTr the part of App. C's formulas that
        // covers a hit by the token drawn from the final residual is zero (the residual has no mass
        // where a draft token can have been rejected), which leaves 1 - (mass of that residual):
        //   SpecInfer  1 - W(c_{k+1}),  c_1 = 0, c_{i+1} = c_i + W(c_i)      (k sweeps)
        //   SpecTr     p_acc = 1 - (1 - beta(rho*))^k                          (the search above)
        //   NSS        sum_t p (1 - (1-q)^k)                                    (one sweep)
        //   Naive      sum_t min(p,q) + sum_t (p-q)_+ (1 - (1-q)^(k-1))         (one sweep)
        // (nothing follows from such a task: the team asks for its next one right away)
        if (leader && !asked) ask_ahead();
        double alpha;
        if (a.walk == 3) {
            const double D = fmin(fmax((sp_W + sp_rho - 1.0) / sp_rho, 0.0), 1.0);
            alpha = 1.0 - int_power(D, k);
        } else if (a.walk == 0) {
            double cc = 0.0, Wc = 1.0;
            for (int j = 0; j < k && all_alike(Wc > 0.0) && !team.dead; ++j) {
                cc = uniform_f64(cc + Wc);
                Wc = residual_mass(cc);
            }
            alpha = 1.0 - Wc;
        } else {
            const float At_hi = static_cast<float>(rt.A), Ad_hi = static_cast<float>(rd.A);
            ResidualConsts rc;
            rc.nAt = -At_hi; rc.nAd = -Ad_hi; rc.rho = 0.f; rc.scale = 1.0;
            double s0, s1;
            sweep(kCmdAcceptance, rc, static_cast<float>(cold_exp2(static_cast<double>(At_hi) - rt.A)),
                  static_cast<float>(cold_exp2(static_cast<double>(Ad_hi) - rd.A)), a.walk == 1 ? k : k - 1, a.walk == 2 ? 1 : 0, s0, s1);
            alpha = s0;
        }
        // the answer may be there already: then the team goes straight on (see the end of the other tasks)
        if (leader && asked && !team.dead) {
            const int t = answer();
            if (t >= 0) {
                team_announce(team, t, 0);
                if (!(t >= B * N && t < B * N + B)) {
                    start_task(view_of(t), t);
                    started = t;
                }
                own_task = t;                              // (announced; counted when it was queued)
            }
        }
        if (lead) {
            as_global(a.alpha)[bn] = static_cast<float>(fmin(fmax(alpha, 0.0), 1.0));
            // (the team that finishes the last task has found no further first task)
            if (claims) (void)atomicAdd(&ws.qctl[1], 1);
            else if (atomicAdd(&ws.qctl[1], 1) + 1 == q.init_total) st_relaxed(&ws.qctl[2], 1);
        }
        goto task_end;
    }
    for (int j = 0; j < k; ++j) {
        // a resumed task repeats the arithmetic of the first child (whose task has long run)
        // to get at the residual that follows its rejection
        const bool redone = resumed && j == 0;
        const unsigned child = static_cast<unsigned>(__builtin_amdgcn_readlane(static_cast<int>(children), j));
        const int cn = field(child, kEntry, 63u);
        const bool inner_child = field(child, 0, 31u) > 0;
        const size_t bc = static_cast<size_t>(b) * N + cn;
        double px = 0.0, qx = 0.0;
        const bool tok_ok = ((token_ok >> j) & 1ull) != 0ull;
        if (tok_ok) {
            px = lane_f64(pq_all, j);
            qx = lane_f64(pq_all, 32 + j);
        } else if (lead) {
            atomicAdd(&a.counters[MPV_COUNTER_BAD_TOKEN], 1u);
        }
        const double rest = fmax(px - c * qx, 0.0);       // current distribution at x, times W
        double w_child;
        if (METHOD == MPV_METHOD_TRAVERSAL) {
            // block-verification weight recursion (Sec. 3.1) with the current a and P
            if (!all_alike(wa > 0.0 && rest > 0.0)) w_child = 0.0;
            else if (all_alike(qx > 0.0)) w_child = fmin(1.0, wa * rest / (W * qx));
            else w_child = 1.0;
        } else if (walk == 1) {
            // NSS tests nothing (App. B Alg. 1); the estimate wants p(x): the chance that Y ~ p is x
            w_child = px;
        } else if (walk == 3) {
            // App. B Alg. 3: accept x if rho* U <= p(x)/q(x)
            if (all_alike(qx > 0.0)) w_child = fmin(1.0, px / (sp_rho * qx));
            else w_child = (px > 0.0) ? 1.0 : 0.0;
        } else {
            // App. B Alg. 4: accept x with min(1, p(x)/q(x))
            if (all_alike(qx > 0.0)) w_child = fmin(1.0, rest / (W * qx));
            else w_child = (rest > 0.0) ? 1.0 : 0.0;
        }
        // the same comparison the walk makes
        const double u_child = static_cast<double>(lane_f32(uniforms, cn));
        // (top-down: as a mask; a scalar branch here makes the compiler copy the loop's end, which costs registers)
        const bool child_accepted = METHOD == MPV_METHOD_TRAVERSAL ? all_alike(u_child < w_child) : u_child < w_child, child_weight = all_alike(w_child > 0.0);
        const unsigned long long child_bit = 1ull << field(child, kRank, 63u);
        if (redone) {
        } else if (METHOD == MPV_METHOD_SPECINFER) {
            settled_bits |= child_bit;
        } else if (!inner_child) {
            settled_bits |= child_bit;
            if (child_accepted) accepted_bits |= child_bit;
        } else if (lazy && !child_weight) {
            // A child of weight 0 can never be accepted, passes weight 0 to its whole subtree
            // and never provides a bonus distribution: its task (and its subtree's) is not
            // queued, its rows are never read; the whole subtree counts as rejected.
            const int hi = field(child, kRank, 63u), lo = field(child, kLow, 63u);
            const unsigned long long upto = (hi >= 63) ? ~0ull : ((1ull << (hi + 1)) - 1ull);
            settled_bits |= upto & ~((1ull << lo) - 1ull);
        }
        // Traversal: the child's own task is needed unless its weight is 0 (see above)
        const bool run_child = METHOD == MPV_METHOD_TRAVERSAL && !redone && inner_child && (child_weight || !lazy);
        const bool first_to_run = run_child && own_child < 0;
        if (first_to_run) {
            // kept for this team if it is the last thing this task finds out and nobody is idle
            own_child = j;
            own_w = w_child;
            own_given = (idle_seen || j < k - 1 || child_ahead) && !(split_here && j == 0);
        }
        // One more sweep to go at most: time to ask for the next task, unless this team
        // already knows what it will run next (a child's task).
        if (leader && j == k - 1 && !asked && (own_child < 0 || own_given) &&
            !(METHOD == MPV_METHOD_SPECINFER && lazy && child_accepted && inner_child))
            ask_ahead();
        if (lead && !redone) {
            if (METHOD == MPV_METHOD_TRAVERSAL) {
                if (!inner_child) {
                    st_shared_f64(&ws.atest[bc], w_child);           // leaves are tested as they are
                } else {
                    st_relaxed(reinterpret_cast<unsigned long long*>(&ws.a0[bc]), static_cast<unsigned long long>(__double_as_longlong(w_child)));
                    // The first child that needs a task is kept for this team (run next,
                    // no queue) unless some team is idle; every other one is queued now,
                    // while this task goes on with the sweeps that follow.
                    if (run_child && (!first_to_run || own_given) && !child_ahead)
                        append_task(tree, ws, field(child, kClass, 1u), b * N + cn);      // (waits for the weight's store with its own count)
                }
            } else if (!draw_here()) {
                st_shared_f64(&ws.atest[bc], w_child);
                if (estimate() && walk == 3) {
                    // App. D, SpecTr Branching: p_res(x), p_res = norm (p - rho* q)_+ (see the search above)
                    const double r = fmax(px - sp_rho * qx, 0.0);
                    st_shared_f64(&ws.aux[bc], sp_W > 0.0 ? fmin(r / sp_W, 1.0) : px);
                }
            }
            if (a.dbg_edge) {
                as_global(a.dbg_edge)[bc * 2] = static_cast<float>(px);
                as_global(a.dbg_edge)[bc * 2 + 1] = static_cast<float>(qx);
            }
        }

        // Where the tree branches and no team is to spare, the first child's subtree is
        // explored first: most walks end there, and then nothing else of this node is needed.
        if (split_here && j == 0 && run_child) {
            paused = true;
            break;
        }

        if (METHOD == MPV_METHOD_SPECINFER && (walk >= 2 || draw_here()) && !estimate() && lead && fabs(w_child - u_child) < 1e-6)
            atomicAdd(&a.counters[MPV_COUNTER_NEAR_TIE_ACCEPT], 1u);     // (else these are counted by the walk)
        // SpecInfer moves into the first child it accepts: later children and this node's
        // residual are not needed (the same in every lane: no lane is left behind)
        if (METHOD == MPV_METHOD_SPECINFER && lazy && child_accepted) {
            next_node = cn;
            if (a.context_node) {
                // the walk goes on at the node of the accepted entry's context (anything else than a node
                // number is ignored)
                const int stands_for = uniform_i32(as_global(a.context_node)[static_cast<size_t>(b) * N + cn]);
                if (stands_for >= 0 && stands_for < N) next_node = stands_for;
            }
            break;
        }
        // NSS: nothing else to find out here
        if (METHOD == MPV_METHOD_SPECINFER && walk == 1) continue;
        // Naive (App. B, Alg. 2) tests the first child only; the token then drawn comes from (p - q)_+
        if (METHOD == MPV_METHOD_SPECINFER && walk == 2 && !estimate()) {
            c = 1.0;
            break;
        }
        // SpecTr tests every child against the same p; its residual is formed once, by the draw
        if (METHOD == MPV_METHOD_SPECINFER && walk == 3) {
            c = sp_rho;
            continue;
        }

        // ---- the child (SpecInfer) or its whole subtree (Traversal) is rejected:
        //      P <- norm (a P - q)_+ ,  i.e.  c <- c + W/a ,  W <- W(c)
        if (METHOD == MPV_METHOD_TRAVERSAL && !all_alike(wa > 0.0)) continue;   // (0*P - q)_+ = 0: nothing changes
        if (team.dead) break;
        const double c2 = uniform_f64(c + W / wa);
        // the task's last sweep, and the team goes on with a child's task: the other waves may ask for its rows
        if (METHOD == MPV_METHOD_TRAVERSAL && j == k - 1 && own_child >= 0 && !own_given) {
            next_hint_node = child_of(own_child);
            next_hint = b * N + next_hint_node;
        }
        const double W2 = residual_mass(c2);
        next_hint = -1;
        if (all_alike(W2 > 0.0)) {
            if (METHOD == MPV_METHOD_TRAVERSAL) {
                const double S = (wa / W) * W2;
                wa = uniform_f64(S / (S + (1.0 - wa)));
            }
            c = c2;
            W = W2;
        } else {
            if (METHOD == MPV_METHOD_TRAVERSAL) wa = all_alike(wa >= 1.0) ? 1.0 : 0.0;
            if (lead) atomicAdd(&a.counters[MPV_COUNTER_ZERO_MASS], 1u);
        }
        if (METHOD == MPV_METHOD_SPECINFER && walk == 2) {
            // Naive, estimate (App. D, Naive Branching): p_res(x_i) for every child, p_res = norm (p - q)_+
            // (now c = 1 and W = its mass; p itself if the mass was zero: c = 0, W = 1)
            for (int i = 0; i < k; ++i) {
                const int ci = child_of(i);
                double r = 0.0;
                if ((token_ok >> i) & 1ull)
                    r = fmax(lane_f64(pq_all, i) - c * lane_f64(pq_all, 32 + i), 0.0) / W;
                else if (i > 0 && lead)
                    atomicAdd(&a.counters[MPV_COUNTER_BAD_TOKEN], 1u);
                if (lead) {
                    st_shared_f64(&ws.aux[static_cast<size_t>(b) * N + ci], r);
                    if (i > 0) st_shared_f64(&ws.atest[static_cast<size_t>(b) * N + ci], 0.0);   // never tested
                }
                settled_bits |= 1ull << field(node_word(ci), kRank, 63u);
            }
            break;
        }
    }

    // ---- The sweeps are over and the part on chip is no longer needed.  What this team will
    //      most likely run next (every member works it out by itself, from the same numbers) is
    //      taken up at once: its rows travel while the leader settles what follows from this
    //      task, and while the others wait to hear of it.
    next_node = uniform_i32(next_node);
    if (DRAWS && draw_here() && (next_node < 0 || n_children(next_node) == 0)) {
        // The walk has come to its draw, at this node or at the accepted leaf: every member knows, nothing is announced.
        const bool row = next_node >= 0;
        if (!row) {
            const ResidualConsts rc = draw_consts(At_, Ad_, c);
            if (lane == 0) { g_cmd.kind = kCmdTiles; g_cmd.nAt = rc.nAt; g_cmd.nAd = rc.nAd; g_cmd.rho = rc.rho; }
            task_barrier();                                // B
            weigh_tiles(uniform_f32(rc.nAt), uniform_f32(rc.nAd), uniform_f32(rc.rho));
            if (lane == 0) { g_draw.nAt = rc.nAt; g_draw.nAd = rc.nAd; g_draw.rho = rc.rho; }
            task_barrier();                                // A
        }
        settle_claim();
        bool want_claim = false;
        if (leader && !asked) {
            want_claim = claims;
            if (!claims && lane == 0) st_relaxed(&ws.mailbox[team.id * q.box_step], kMailboxSoon);
            asked = true;
        }
        if (lane == 0) {
            g_draw.pending = 1;
            g_draw.b = b;
            g_draw.n = row ? next_node : n;
            g_draw.row = row ? 1 : 0;
            g_draw.there = row && ahead_row && ahead_node == next_node ? 1 : 0;
            g_loop.want_claim = want_claim ? 1 : 0;
        }
        own_task = -1; own_flags = 0;
        goto task_end;
    }
    int likely_node = -1;
    if (!team.dead) {
        if (METHOD == MPV_METHOD_TRAVERSAL) {
            if (paused) likely_node = child_of(0);
            else if (own_child >= 0 && !own_given) likely_node = child_of(own_child);
        } else if (lazy && next_node >= 0 && n_children(next_node) > 0) {
            likely_node = next_node;
        }
    }
    const int likely = likely_node >= 0 ? b * N + likely_node : -1;
    // The team has asked for its next task ahead of time; if the answer is in the mailbox already
    // (and nothing of this task's own can come first) the team is told now and takes the task
    // up, while the leader settles what follows from this one: whatever that produces then goes
    // to the queue instead of being run by this team.  (Not with the token-following rules: a
    // tree can need several draws, the queue has room for one.)
    int taken = -1;
    if (leader && likely < 0 && !paused && asked && !team.dead && walk == 0) {
        taken = answer();
        if (taken >= 0) team_announce(team, taken, uniform_i32(idle_now) != 0 ? kFlagIdle : 0);
    }
    {
        // (trees of different shapes: the tables in LDS are still this tree's)
        const int start_now = likely >= 0 ? likely
                            : ((taken >= 0 && !(taken >= B * N && taken < B * N + B) && (!a.per_tree || tree_of(taken) == b)) ? taken : -1);
        if (start_now >= 0) {
            start_task(likely >= 0 ? view_at(b, likely_node, false) : view_of(start_now), start_now);
            started = start_now;
        }
        if (likely >= 0) {
            // Where that task is a child's and nothing else follows from this one (a chain), the
            // team simply goes on with it: every member knows the task and what it starts with,
            // so nothing is announced, nothing waited for, and the outcomes settled here are
            // noted for the first task that goes the long way to publish.  (If another branch
            // settles the tree meanwhile, the chain runs on in vain until it ends.)
            if (METHOD == MPV_METHOD_TRAVERSAL || walk == 0 || draw_here()) {
                if (!draw_here() && !(METHOD == MPV_METHOD_TRAVERSAL && paused)) {
                    if (lead) {
                        st_shared_f64(&ws.At[bn], rt.A);
                        st_shared_f64(&ws.Ad[bn], rd.A);
                        st_shared_f64(&ws.cfin[bn], c);
                        if (METHOD == MPV_METHOD_TRAVERSAL && n != 0) st_shared_f64(&ws.atest[bn], wa);
                    }
                    chain_settled |= settled_bits;
                    chain_accepted |= accepted_bits;
                    if (METHOD == MPV_METHOD_TRAVERSAL && n != 0) {
                        const unsigned long long own = 1ull << field(node_word(n), kRank, 63u);
                        chain_settled |= own;
                        if (all_alike(static_cast<double>(un) < wa)) chain_accepted |= own;
                    }
                }
                if (METHOD == MPV_METHOD_TRAVERSAL) a0_known = own_w;
                chained = likely_node;
                task = likely;                            // (flags: as they are)
                continue;
            }
        }
    }
    settled_bits |= chain_settled;
    accepted_bits |= chain_accepted;
    chain_settled = 0ull;
    chain_accepted = 0ull;

    if (!paused && lane == 0) {                       // (a sampling task of this node by this team need not ask memory)
        g_loop.kept_task = b * N + n;
        g_loop.kept_At = rt.A; g_loop.kept_Ad = rd.A; g_loop.kept_c = c;
    }
    // ---- what follows from this task: the leader's business (its first wave's)
    if (!leader) goto task_end;
    own_flags = uniform_i32(idle_now) != 0 ? kFlagIdle : 0;
    if (METHOD == MPV_METHOD_SPECINFER && lazy && walk == 0 && likely < 0 && taken < 0) {
        // The walk ends here or in the accepted leaf: the sampling follows at once, by this team, as a part of this task
        // (nothing is counted, nothing of this node's has to reach memory first: every member has it).
        own_task = B * N + b;
        own_flags |= ((next_node >= 0 ? next_node : n) + 1) << kFlagStopShift;
        team_announce(team, own_task, own_flags);
        goto task_end;
    }
    if (paused) {
        // nothing is settled yet; the first child's task is run next by this team
        own_task = b * N + child_of(0);
        team_announce(team, own_task, own_flags);
        if (lane == 0) {
            (void)atomicAdd(&ws.qctl[0], 1);
            wait_memory();                            // counted (and the child's weight written) before this task counts as finished
            atomicAdd(&ws.qctl[1], 1);
        }
        goto task_end;
    }
    int push_sample_i = 0, settled_i = 0, resume_i = 0, accepted_at = -1;
    if (lane == 0) {
        st_shared_f64(&ws.At[bn], rt.A);
        st_shared_f64(&ws.Ad[bn], rd.A);
        st_shared_f64(&ws.cfin[bn], c);
        if (METHOD == MPV_METHOD_TRAVERSAL && n != 0) st_shared_f64(&ws.atest[bn], wa);
        bool push_sample, settled_tree = false, resume = false;
        if (METHOD == MPV_METHOD_SPECINFER && lazy) {
            // the walk ends here (no child accepted) or in the accepted leaf
            push_sample = next_node < 0 || n_children(next_node) == 0;
            if (walk) st_relaxed(&ws.cur[b], next_node >= 0 ? next_node : n);     // where the next token is drawn
            wait_memory();                            // results written through before anything else is started
        } else {
            // Announce the outcomes settled here, then see whether the tree's outcome is settled:
            //   only what is needed: in postorder, the first node that is not known to be
            //     rejected is known (then it is the accepted one: the walk stops there);
            //   everything: every node is known.
            // `acc` is written before `known`, so the acc bits of known nodes are final.  Of
            // the tasks that see a settled tree, the first to flip `decided` starts the sampling.
            if (METHOD == MPV_METHOD_TRAVERSAL && n != 0) {
                const unsigned long long own = 1ull << field(node_word(n), kRank, 63u);
                settled_bits |= own;
                if (static_cast<double>(un) < wa) accepted_bits |= own;
            }
            if (accepted_bits) (void)atomicOr(&ws.acc[b], accepted_bits);
            wait_memory();                            // results written through before they are announced
            const unsigned long long known_before = atomicOr(&ws.known[b], settled_bits);
            const unsigned long long known = known_before | settled_bits;
            wait_memory();
            const unsigned long long acc = ld_relaxed(&ws.acc[b]);
            const int decided_before = ld_relaxed(&ws.decided[b]);      // issued with the load above: one round trip
            bool settled;
            if (lazy) {
                const unsigned long long open = ~(known & ~acc);          // not known to be rejected
                const int first = __ffsll(static_cast<long long>(open)) - 1;   // the root's bit is always set
                settled = ((known >> first) & 1ull) != 0ull;
                accepted_at = first;
            } else {
                const unsigned long long all = (N >= 64) ? ~0ull : ((1ull << N) - 1ull);
                settled = known == all;
            }
            push_sample = settled && decided_before == 0 && atomicCAS(&ws.decided[b], 0, 1) == 0;
            // only what is needed: once a tree is settled (here or by another task) the rest of
            // its node tasks are pointless
            settled_tree = lazy && (settled || decided_before != 0);
            // The subtree that was explored first has just turned out to be rejected as a whole
            // (this task supplied its last missing outcome): time for the rest of the node
            // where the tree branches.
            if (METHOD == MPV_METHOD_TRAVERSAL && lazy && tree.split_node >= 0 && !settled_tree &&
                ((tree.split_mask >> field(node_word(n), kRank, 63u)) & 1ull) != 0ull) {          // this node lies in that subtree
                const unsigned long long m = tree.split_mask;
                resume = (known & m) == m && (known_before & m) != m && (acc & m) == 0ull;
            }
        }
        push_sample_i = push_sample ? 1 : 0;
        settled_i = settled_tree ? 1 : 0;
        resume_i = resume ? 1 : 0;
    }
    push_sample_i = uniform_i32(push_sample_i);
    settled_i = uniform_i32(settled_i);
    resume_i = uniform_i32(resume_i);
    // What follows from this task.  One task is run by this team itself, next (no queue,
    // no waiting): the sampling if this task settled the tree, else the first child that needs
    // its own task (Traversal) or the accepted child (SpecInfer).  The other children are queued.
    if (push_sample_i) {
        if (!ACCEPT && estimate()) {
            // the expected block efficiency instead of a walk: scalar work over the tree's
            // per-node results, done here and now by this wave (there are no uniforms to walk with)
            estimate_wave<METHOD>(tree, ws, a, b);
            if (lane == 0) tree_done(ws, a);
        } else if (taken >= 0) {
            if (lane == 0) append_task(tree, ws, 0, B * N + b);      // (the results were waited for above)
        } else {
            own_task = B * N + b;
            // (only what is needed: the outcome is known here, the team need not look it up)
            int stop = next_node >= 0 ? next_node : n;
            if (METHOD == MPV_METHOD_TRAVERSAL)
                stop = __ffsll(static_cast<long long>(__ballot(lane < N && field(nodes, kRank, 63u) == uniform_i32(accepted_at)))) - 1;
            if (lazy && walk == 0) own_flags |= (stop + 1) << kFlagStopShift;
        }
    } else if (resume_i) {
        // Queued, not run at once: while there are trees that have not been begun, beginning them comes
        // first (class 0), so that the long trees, whose branching node is resumed, share the teams evenly
        // at the end instead of running on by themselves (benchmark batch: 5 % less time).
        if (lane == 0) append_task(tree, ws, 1, B * N + B + b);
    } else if (taken >= 0) {
        // (nothing else can follow from a task that has no child of its own to run)
    } else if (METHOD == MPV_METHOD_TRAVERSAL) {
        if (own_child >= 0 && !own_given && !settled_i) own_task = b * N + child_of(own_child);
    } else if (lazy && next_node >= 0 && n_children(next_node) > 0) {
        own_task = b * N + next_node;
    }
    // the others hear of it at once (they are waiting for the next task by now)
    if (own_task >= 0) team_announce(team, own_task, own_flags);
    if (lane == 0) {
        if (own_task >= 0) {
            (void)atomicAdd(&ws.qctl[0], 1);
            wait_memory();
        }
        // (cannot happen: a task that settles the tree or completes a subtree has no child left to run)
        if (METHOD == MPV_METHOD_TRAVERSAL && own_child >= 0 && !own_given && !settled_i && (push_sample_i || resume_i)) {
            const int cn = child_of(own_child);
            append_task(tree, ws, field(node_word(cn), kClass, 1u), b * N + cn);
        }
        wait_memory();                                // every new task has been counted
        atomicAdd(&ws.qctl[1], 1);
    }
    if (taken >= 0) own_task = taken;                 // (announced above; counted when it was queued)
    }   // (the task's own scope)
task_end:
    // The task that follows: the leader knows (and has told the others, who hear of it here).
    int next, next_flags = 0;
    if (leader) {
        next = own_task;
        next_flags = own_flags;
    } else if (DRAWS && draw_here()) {
        next = kNothingHeard;                              // (a draw comes next, what follows it is announced in the task loop)
    } else {
        next = team_listen(team, next_flags, ws);
    }
    bool node_next = next >= 0 && !(next >= B * N && next < B * N + B) && !team.dead;
    if constexpr (!kShapeInTask && !ACCEPT) node_next = node_next && (!a.per_tree || tree_of(next) == uniform_i32(g_tree_of));
    if (started >= 0 && (!node_next || next != started)) {
        // taken up in vain (the tree was settled meanwhile, or the task went elsewhere): the other
        // waves finish their sweep, this wave's loads land, and the slots are free again
        task_barrier();                                    // A
        wait_memory();
        started = -1;
    }
    if (!node_next) {
        settle_claim();
        // (before the others leave: with a draw to come the second wave counts off a first task for the leader then)
        if (lane == 0) {
            g_cmd.kind = kCmdDone;
            g_loop.team = team;
            g_loop.asked = asked ? 1 : 0;
            g_loop.claims = claims ? 1 : 0;
            g_loop.claimed = claimed;
            g_loop.own_task = next;                       // (already announced to, or heard by, the team)
            g_loop.own_flags = next_flags;
        }
        task_barrier();                                    // B: the other waves leave
        return;
    }
    task = next;
    flags = next_flags;
    }   // node tasks
}


template <class E, int KIND>
__device__ __forceinline__ void run_tasks(const LaunchBlock* __restrict__ launch) {
    // KIND: MPV_METHOD_TRAVERSAL; the top-down rules: MPV_METHOD_SPECINFER, kKindWalk, kKindShort, kKindShortAll; or kKindAcceptance: the
    // top-down kernel reduced to what the acceptance rates need (an instantiation of its own, so that
    // its extra sweeps do not weigh on the register allocation of the verification kernels)
    constexpr bool ACCEPT = KIND == kKindAcceptance, DRAWS = KIND == kKindWalk || KIND == kKindShort;
    constexpr int METHOD = method_of(KIND);
    __shared__ int sh_task, sh_flags;
    // The launch parameters and the tree tables are read from LDS, copied there from the
    // workspace (init_kernel put them there): as kernel arguments, handed on by reference or
    // indexed with a value the compiler keeps in a vector register, they were copied, whole,
    // into every lane's private memory.
    for (int w = threadIdx.x; w < static_cast<int>(sizeof(Launch) / sizeof(int)); w += kTaskBlock)
        g_launch_words[w] = reinterpret_cast<const int*>(launch)[w];
    for (int w = threadIdx.x; w < static_cast<int>(sizeof(TreeDesc) / sizeof(int)); w += kTaskBlock)
        reinterpret_cast<int*>(&g_tree)[w] = reinterpret_cast<const int*>(&launch->tree)[w];
    __syncthreads();
    const QueuePlan& q = lds_launch().q;
    const Workspace& ws = lds_launch().ws;
    const Args& a = lds_launch().a;
    const TreeDesc& tree = g_tree;                // the task loop starts with a barrier

    // ---- this workgroup's place in its team
    const bool drop_settled = METHOD == MPV_METHOD_TRAVERSAL && a.lazy != 0;
    const int wave = uniform_i32(static_cast<int>(threadIdx.x) / kWave);
    bool leader;
    {
        Team team;
        team.size = q.team_size;
        const int i = static_cast<int>(blockIdx.x);
        if (q.same_xcd) {                         // workgroup i runs on chiplet i % 8: keep a team on one
            const int r = i / 8;
            team.id = (i % 8) + 8 * (r / team.size);
            team.member = r % team.size;
        } else {
            team.id = i / team.size;
            team.member = i % team.size;
        }
        team.seq = before_first_exchange(false); team.tseq = 0u; team.dead = 0;
        team.area = ws.exch + static_cast<size_t>(team.id) * 2 * team.size * kExchWords;
        // (a line holds the words of eight teams: of one chiplet, like everything that stays in its L2)
        team.task_word = ws.team_task + static_cast<size_t>(q.same_xcd ? (team.id % 8) * (kMaxTeams / 8) + team.id / 8 : team.id) * 2;
        team.t_start = wall_clock64();
        leader = team.member == 0;
        if (wave == 0) {
            const int lane = threadIdx.x;
            // The last member to arrive counts off the team's first task and tells the others; if there is
            // none left it opens the team's mailbox: from then on the dispatcher may hand it tasks.
            const int flags = q.spare ? kFlagIdle : 0;
            int task = kNotStarted, n_arrived = 1, n_here = 0;
            if (team.size > 1) {
                const int on = chiplet_here();
                unsigned long long so_far = arrival_of(on);
                if (lane == 0) so_far += atomicAdd(team.area, so_far);
                n_arrived = uniform_i32(arrived(so_far));
                n_here = uniform_i32(arrived_on(so_far, on));
            }
            if (n_arrived == team.size) {
                int number = 0;
                if (lane == 0) number = claim_first(ws);
                const int t = first_task(q, a, uniform_i32(number));
                if (t == kTaskNone && lane == 0) st_relaxed(&ws.mailbox[team.id * q.box_step], kMailboxWaiting);
                if (team.size == 1) task = t == kTaskNone ? -1 : t;
                else if (lane < 2) st_relaxed(team.area + 1 + lane, (1ull << 32) | static_cast<unsigned>(lane == 0 ? t : flags | (n_here == team.size ? kFlagOneChiplet : 0)));
            }
            if (lane == 0) {
                g_loop.team = team;
                g_loop.own_task = task;
                g_loop.own_flags = flags;
                g_loop.asked = task == -1;
                g_loop.claims = task != -1;
                g_loop.claimed = kTaskNone;
                g_loop.previous_task = -4;            // none yet
                g_loop.finished = 0;
                g_loop.kept_task = -1;
                g_draw.pending = 0;
                g_tree_of = -1;
            }
        }
    }
    // The first wave's scalar steps are the critical path of every task and few in number: they
    // go first when the compute unit's waves compete for issue slots.
    // (Not for the acceptance rates: there every team has its next task at once, the vector units decide, and a first wave that
    // goes ahead only holds up the sweeps: 64 trees of 33 inner nodes, V = 151936: 413 us with, 398 without.)
    if (wave == 0 && !ACCEPT) __builtin_amdgcn_s_setprio(3);
    for (;;) {
    __syncthreads();                                  // the previous task is done with LDS; g_loop is as it left it
    if (wave == 0) {
        // the task loop's own state: taken from g_loop, put back before the barrier below
        Team team = uniform_struct(g_loop.team);
        bool asked = uniform_i32(g_loop.asked) != 0;
        int own_task = uniform_i32(g_loop.own_task), own_flags = uniform_i32(g_loop.own_flags);
        int previous_task = uniform_i32(g_loop.previous_task);
        bool claims = uniform_i32(g_loop.claims) != 0;
        int claimed = uniform_i32(g_loop.claimed);
        int task = kTaskExit, flags = 0;
        if (team.dead) {
            task = kTaskExit;
        } else if (leader && uniform_i32(g_loop.finished) != 0) {
            team_announce(team, task, 0);
        } else if (leader) {
            for (;;) {
                if (own_task == kNotStarted) {
                    own_task = -1;
                    task = team_listen<true>(team, flags, ws);
                    if (task == kTaskExit) team_announce(team, task, 0);      // (for one that heard "none" just before)
                    if (task != kTaskNone) break;
                    claims = false;
                    asked = true;
                }
                if (own_task >= 0) {
                    task = own_task;
                    flags = own_flags;
                    own_task = -1;
                    break;
                }
                if (claims && claimed == kTaskNone) {
                    int number = 0;
                    if (threadIdx.x == 0) number = claim_first(ws);
                    claimed = first_task(q, a, uniform_i32(number));
                    if (claimed == kTaskNone) claims = false;
                }
                if (claimed != kTaskNone) {
                    task = claimed;
                    claimed = kTaskNone;
                } else {
                    if (!asked) {
                        if (threadIdx.x == 0) st_relaxed(&ws.mailbox[team.id * q.box_step], kMailboxWaiting);
                        wait_memory();
                    }
                    task = acquire_task(team.id, previous_task, drop_settled, team.t_start);
                    previous_task = task;
                }
                // are teams idle (as of the last round of dispatching)?
                flags = uniform_i32(ld_relaxed(&ws.qctl[kCtlIdle])) != 0 ? kFlagIdle : 0;
                asked = false;
                // tasks without any V-wide work are the leader's alone; everything else is announced
                const bool solo = task != kTaskExit && task >= a.B * a.N && task < a.B * a.N + a.B && (ACCEPT || a.estimate);
                if (solo) {
                    if (!ACCEPT) estimate_wave<METHOD>(tree, ws, a, task - a.B * a.N);
                    if (threadIdx.x == 0) {
                        wait_memory();
                        tree_done(ws, a);
                        atomicAdd(&ws.qctl[1], 1);
                    }
                    continue;
                }
                team_announce(team, task, flags);
                break;
            }
        } else if (own_task >= 0 || own_task == kTaskExit) {
            task = own_task;
            flags = own_flags;
            own_task = kNothingHeard;
        } else {
            task = kTaskNone;
            if (own_task == kNotStarted) task = team_listen<true>(team, flags, ws);
            if (task == kTaskNone) task = team_listen(team, flags, ws);
            own_task = kNothingHeard;
        }
        const bool samples = task != kTaskExit && task >= a.B * a.N && task < a.B * a.N + a.B && !(ACCEPT || a.estimate);
        if (!ACCEPT && a.per_tree && task != kTaskExit) load_shape(reinterpret_cast<const unsigned long long*>(ws.aux), a.N, tree_of_task(task, a.B, a.N));
        bool want_claim = false;
        if (samples && leader && !asked) {
            // the walk and the bonus token come next: one sweep or two, then the team is free
            want_claim = claims;
            if (!claims && threadIdx.x == 0) st_relaxed(&ws.mailbox[team.id * q.box_step], kMailboxSoon);
            asked = true;
        }
        if (threadIdx.x == 0) {
            g_loop.team = team;
            g_loop.claims = claims ? 1 : 0;
            g_loop.claimed = claimed;
            g_loop.want_claim = want_claim ? 1 : 0;
            g_loop.asked = asked ? 1 : 0;
            g_loop.own_task = own_task;
            g_loop.own_flags = own_flags;
            g_loop.previous_task = previous_task;
            sh_task = task; sh_flags = flags;
        }
    }
    __syncthreads();
    const int task = uniform_i32(sh_task), flags = uniform_i32(sh_flags);
    if (task == kTaskExit) break;
    const bool sampling = task >= a.B * a.N && task < a.B * a.N + a.B;
    // the leader's second wave, when the first is busy with a walk's end
    auto claim_ahead = [&]() __attribute__((always_inline)) {
        if (leader && threadIdx.x == kWave && g_loop.want_claim) {
            g_loop.claimed = first_task(q, a, claim_first(ws));
            if (g_loop.claimed == kTaskNone) {
                g_loop.claims = 0;
                st_relaxed(&ws.mailbox[g_loop.team.id * q.box_step], kMailboxSoon);
            }
        }
    };
    // A walk is over.  The count of trees is waited for by the second wave, or, if there is nothing to go on with, by the
    // first, which then knows whether the launch is over.
    auto count_tree = [&]() __attribute__((always_inline)) {
        const bool by_first = g_loop.claims == 0 && g_loop.claimed == kTaskNone;
        if (threadIdx.x == (by_first ? 0 : kWave)) {
            const bool last = tree_done(ws, a);
            if (by_first && last) g_loop.finished = 1;
            atomicAdd(&ws.qctl[1], 1);
        }
    };
    if (!DRAWS && sampling) {
        if (ACCEPT || a.estimate) {
            // no walk in these modes (there are no uniforms): scalar work of the leader's first
            // wave alone, whichever way the task came
            if (wave == 0 && leader) {
                if (!ACCEPT) estimate_wave<METHOD>(tree, ws, a, task - a.B * a.N);
                if (threadIdx.x == 0) {
                    wait_memory();
                    tree_done(ws, a);
                    atomicAdd(&ws.qctl[1], 1);
                }
            }
            continue;
        }
        claim_ahead();
        // the tree's outcome is settled: walk and bonus token
        const int next = sample_task<E, METHOD>(task - a.B * a.N, (flags >> kFlagStopShift) - 1);
        if (next < 0 && leader) count_tree();
        if (next >= 0 && wave == 0 && leader) {
            {                                         // a token-following walk goes on
                Team team = uniform_struct(g_loop.team);          // (as sample_task left it)
                wait_memory();                        // the walk's position, which every member reads when it hears of the task
                team_announce(team, next, flags);
                if (threadIdx.x == 0) {
                    g_loop.team = team;
                    g_loop.own_task = next;
                    g_loop.own_flags = flags;
                }
            }
            if (threadIdx.x == 0) {
                (void)atomicAdd(&ws.qctl[0], 1);
                wait_memory();                        // counted before this one is
                atomicAdd(&ws.qctl[1], 1);
            }
        }
        continue;
    }
    if (!sampling) run_node_task<E, KIND>(task, flags);
    if constexpr (DRAWS) {
        if (!sampling && uniform_i32(g_draw.pending) == 0) continue;
        // the walk has come to a draw: the node task's that has just ended, or its first step
        claim_ahead();
        const int next = draw_walk<E>(sampling ? task - a.B * a.N : g_draw.b, sampling ? 0 : g_draw.n, sampling ? 1 : g_draw.row, sampling ? 0 : g_draw.there);
        if (next < 0 && leader) count_tree();
        if (threadIdx.x == 0) {
            g_draw.pending = 0;
            if (next >= 0) { g_loop.own_task = next; g_loop.own_flags = 0; }          // every member knows: it is not announced
        }
    }
    }   // task loop
}

// (disable_tail_calls: a call marked as a possible tail call makes the compiler treat the callee
// as one that must preserve registers for its caller, and the task functions, which use nearly
// all of them, would save and restore dozens per call in private memory)
template <class E, int KIND>
__global__ __launch_bounds__(kTaskBlock) __attribute__((amdgpu_waves_per_eu(3, 3))) __attribute__((disable_tail_calls))
void node_task_kernel(const LaunchBlock* __restrict__ launch) { run_tasks<E, KIND>(launch); }

// The top-down rules where walks draw their tokens themselves (draw_walk) and nothing but the walks runs: neither estimates nor
// debug outputs.  Kernels apart: with the draws, which it never uses, in its code and a question for them at every step
// node_task_kernel took 22.5 us for the block efficiency of one tree of V = 6784 in float32 (NSS) and 65 for 41 trees of V = 4480
// (Naive), without 21.2 and 60; and what a walk never uses taken out here, 32 trees of V = 262144, SpecInfer, take 66.2 us (67.8
// before), 241 of V = 6295 63 (64.8), 200 of V = 136256, SpecTr, 168.5 (170.4).
template <class E>
__global__ __launch_bounds__(kTaskBlock) __attribute__((amdgpu_waves_per_eu(3, 3))) __attribute__((disable_tail_calls))
void walk_kernel(const LaunchBlock* __restrict__ launch) { run_tasks<E, kKindWalk>(launch); }

// The same on parts that the registers hold (six vectors of a row per lane).  Their rows come through the LDS, and
// as soon as the first sweep has taken them from there the second to fourth wave ask for the rows of the first child,
// which is where the walk goes on if it is accepted (for a leaf, the target row, for the draw): they travel while the
// first wave exchanges sums and works out whether it is.  Without slots in LDS and beyond them the task function is
// little more than half as long (65 KB, 108 in bf16; the instruction cache of two compute units has 64).  64 trees of V = 128256,
// SpecInfer: a link of the chain 9.2 -> 8.3 us; calls: 37 trees of V = 50001, SpecTr, 79 -> 73 us, 2 of V = 1143 74 -> 64, 186 of V = 1974, Naive,
// 61 -> 54, 26 of V = 5093, SpecInfer, 48 -> 46.  Traversal gained nothing by it (94 trees of V = 8515: 151 us, 157 with).
template <class E>
__global__ __launch_bounds__(kTaskBlock) __attribute__((amdgpu_waves_per_eu(3, 3))) __attribute__((disable_tail_calls))
void short_part_kernel(const LaunchBlock* __restrict__ launch) { run_tasks<E, kKindShort>(launch); }

// Estimates and debug outputs of the top-down rules on such parts: nothing is asked for ahead, and the shorter function alone is
// worth it (block efficiency of 212 trees of V = 1474, NSS: 156 us by node_task_kernel, 145 by this; 178 of V = 2475, SpecInfer: 122, 114).
template <class E>
__global__ __launch_bounds__(kTaskBlock) __attribute__((amdgpu_waves_per_eu(3, 3))) __attribute__((disable_tail_calls))
void staged_part_kernel(const LaunchBlock* __restrict__ launch) { run_tasks<E, kKindShortAll>(launch); }

// ------------------------------------------------------------------ walk
//
// The uniform-dependent part of SpecInfer and Traversal.  Where the task says in which node the walk stopped, only the
// leader's third wave does it, to record the path; else every wave of the sampling team does (they all need the stopping
// node; the leader's first records the path).  Lane n compares u[n] with the probability node n is tested with
// (which does not depend on the uniforms), the 64 outcomes become a bit mask, and
// the walk itself is a few scalar steps over that mask.
//   SpecInfer (Sec. 3.2 walk + App. B Alg. 4): from the root, move to the first
//     accepted child in list order; stop where no child is accepted.
//   Traversal: nodes are tested in depth-first post-order; the first accepted one
//     wins, the root is accepted unconditionally.
// Returns the stopping node (the same value in every lane) and writes the path.
// accepted length and path of a walk that ended in `stop` (one lane)
__device__ __forceinline__ void write_path(const TreeDesc& tree, const Args& a, int b, int stop) {
    const size_t base = static_cast<size_t>(b) * a.N;
    const int len = tree.depth[stop];
    as_global(a.accept_len)[b] = len;
    int32_t* pn = a.path_nodes + static_cast<size_t>(b) * a.max_depth;
    int32_t* pt = a.path_tokens + static_cast<size_t>(b) * a.max_depth;
    for (int i = len; i < a.max_depth; ++i) { pn[i] = -1; pt[i] = -1; }
    for (int n = stop, i = len - 1; n > 0; n = tree.parent[n], --i) {
        pn[i] = n;
        pt[i] = as_global(a.tokens)[base + n];
    }
}

template <int METHOD>
__device__ __forceinline__ int walk_wave(const TreeDesc& tree, const Workspace& ws, const Args& a, int b, bool record) {
    const int lane = threadIdx.x & (kWave - 1);
    const size_t base = static_cast<size_t>(b) * a.N;
    bool acc = false, near = false;
    if (lane > 0 && lane < a.N) {
        const double at = ld_shared_f64(&ws.atest[base + lane]);
        const double uu = static_cast<double>(as_global(a.uniforms)[base + lane]);
        acc = uu < at;
        near = fabs(at - uu) < 1e-6;
        if (a.dbg_accept && record) as_global(a.dbg_accept)[base + lane] = static_cast<float>(at);
    }
    if (lane == 0 && a.dbg_accept && record) as_global(a.dbg_accept)[base] = 1.f;
    const unsigned long long accm = __ballot(acc);
    const unsigned long long nearm = __ballot(near);
    unsigned long long tested = 0ull;
    int stop = 0;
    if (METHOD == MPV_METHOD_SPECINFER) {
        int n = 0;
        for (;;) {
            int next = -1;
            const int k = tree.nchild[n], off = tree.child_off[n];
            for (int j = 0; j < k; ++j) {
                const int cn = tree.child_list[off + j];
                tested |= 1ull << cn;
                if ((accm >> cn) & 1ull) { next = cn; break; }
            }
            if (next < 0) break;
            n = next;
        }
        stop = n;
    } else {
        for (int i = 0; i + 1 < a.N; ++i) {
            const int n = tree.postorder[i];
            tested |= 1ull << n;
            if ((accm >> n) & 1ull) { stop = n; break; }
        }
    }
    if (lane == 0 && record) {
        write_path(tree, a, b, stop);
        const int nn = __popcll(nearm & tested);
        if (nn) atomicAdd(&a.counters[MPV_COUNTER_NEAR_TIE_ACCEPT], static_cast<unsigned>(nn));
    }
    return stop;
}

// ------------------------------------------------------------------ expected block efficiency
//
// Sec. 5, Eq. 1-3: E[tau + 1 | tree] = sum over nodes of P(the node lies on the accepted path).
// Lane n looks after node n.  Top-down rules: the probability of moving from a node to its
// child is put together from the per-child results the node tasks left (App. D):
//   SpecInfer  a_j prod_{l<j} (1 - a_l), a_l the probability sibling l is tested with;
//   NSS        p(x_j) if no earlier sibling carries the same token (a drawn token leads to the
//              first sibling that carries it), else 0;
//   Naive      [j = 1] a_1 + (1 - a_1) p_res(x_j) [first carrier of x_j];
//   SpecTr     a_j prod_{l<j} (1 - a_l) + p_res(x_j) prod_l (1 - a_l) [first carrier of x_j];
// and a node's reach probability is the product along its path from the root.  Traversal: nodes
// are tested in postorder, each after everything before it was rejected, so the node at position
// r is the accepted one with a_r prod_{r'<r} (1 - a_r'), and a node is on the accepted path iff
// the accepted node is in its subtree.
template <int METHOD>
__device__ __forceinline__ void estimate_wave(const TreeDesc& tree, const Workspace& ws, const Args& a, int b) {
    __shared__ double sh_v[MPV_MAX_NODES], sh_w[MPV_MAX_NODES];
    const int n = lane_here();
    const size_t base = static_cast<size_t>(b) * a.N;
    const bool live = n < a.N;
    double reach = 0.0;
    if (METHOD == MPV_METHOD_TRAVERSAL) {
        // sh_v[r]: test probability of the node at postorder position r (the root, last, is accepted)
        if (live) {
            const int node = tree.postorder[n];
            sh_v[n] = (node == 0) ? 1.0 : ld_shared_f64(&ws.atest[base + node]);
        }
        __builtin_amdgcn_wave_barrier();
        if (live) {
            double none_before = 1.0;
            for (int r = 0; r < n; ++r) none_before *= 1.0 - sh_v[r];
            sh_w[n] = sh_v[n] * none_before;          // the node at position n is the accepted one
        }
        __builtin_amdgcn_wave_barrier();
        if (live) {
            if (n == 0) reach = 1.0;
            else for (int r = tree.sub_lo[n]; r <= tree.rank[n]; ++r) reach += sh_w[r];
        }
    } else {
        if (live) {
            sh_v[n] = (n == 0) ? 1.0 : ld_shared_f64(&ws.atest[base + n]);
            sh_w[n] = (n == 0 || a.walk < 2) ? 0.0 : ld_shared_f64(&ws.aux[base + n]);
        }
        __builtin_amdgcn_wave_barrier();
        double step = 1.0;                            // from the parent to this node
        if (live && n > 0) {
            const int par = tree.parent[n], off = tree.child_off[par], k = tree.nchild[par];
            const int x = as_global(a.tokens)[base + n];
            double none_before = 1.0, none_at_all = 1.0;
            bool first_carrier = true;
            int j = 0;
            // trees of distinct contexts, SpecTr: an accepted entry leads to the node it stands for, so a
            // node collects the acceptances of every entry that stands for it and a repeat collects nothing
            const bool aliased = a.walk == 3 && a.context_node != nullptr;
            double through_entries = 0.0;
            for (int l = 0; l < k; ++l) {
                const int sib = tree.child_list[off + l];
                if (sib == n) j = l;
                if (sib < n) {                        // list order is node order
                    none_before *= 1.0 - sh_v[sib];
                    if (as_global(a.tokens)[base + sib] == x) first_carrier = false;
                }
                if (aliased && as_global(a.context_node)[base + sib] == n) through_entries += sh_v[sib] * none_at_all;
                none_at_all *= 1.0 - sh_v[sib];
            }
            if (a.walk == 0) step = sh_v[n] * none_before;
            else if (a.walk == 1) step = first_carrier ? sh_v[n] : 0.0;
            else if (a.walk == 2) {
                const double a1 = sh_v[tree.child_list[off]];
                step = (j == 0 ? a1 : 0.0) + (first_carrier ? (1.0 - a1) * sh_w[n] : 0.0);
            } else if (aliased) {
                step = through_entries + (first_carrier ? sh_w[n] * none_at_all : 0.0);
            } else {
                step = sh_v[n] * none_before + (first_carrier ? sh_w[n] * none_at_all : 0.0);
            }
        }
        __builtin_amdgcn_wave_barrier();              // everybody has read sh_v / sh_w
        if (live) sh_v[n] = step;
        __builtin_amdgcn_wave_barrier();
        if (live) {
            reach = 1.0;
            for (int m = n; m > 0; m = tree.parent[m]) reach *= sh_v[m];
        }
    }
    if (live && a.reach_prob) as_global(a.reach_prob)[base + n] = static_cast<float>(reach);
    const double total = wave_sum(live ? reach : 0.0);
    if (n == 0 && a.expected) as_global(a.expected)[b] = static_cast<float>(total);
}

// ------------------------------------------------------------------ bonus sample

// The member whose share of a row contains u times the mass of all, lane m < team.size holding member m's mass (the others
// 0): the first whose running total exceeds it and that has mass; rounding only: the last one that has mass.  into: how far
// the target lies into that member's share.
__device__ __forceinline__ int member_at(const Team& team, double mass, float u, double& into, double& total) {
    double upto = mass;                                // sums along the row of lanes: member m and those before it
    upto += dpp_f64<0x111>(upto);
    upto += dpp_f64<0x112>(upto);
    upto += dpp_f64<0x114>(upto);
    upto += dpp_f64<0x118>(upto);
    total = lane_f64(upto, team.size - 1);
    const double target = static_cast<double>(u) * total;
    const unsigned long long hit = __ballot(mass > 0.0 && upto > target), any = __ballot(mass > 0.0);
    const int owner = hit ? __ffsll(static_cast<long long>(hit)) - 1 : any ? 63 - __clzll(static_cast<long long>(any)) : 0;
    into = target - lane_f64(dpp_f64<0x111>(upto), owner);
    return owner;
}

// The vocabulary is split among the members in runs of whole wave tiles (64 vectors of 16 bytes, counted from the aligned
// address at or before the row's start, so that rows of any offset are read with vector loads), in member order; tile i of
// a member's run belongs to wave i % 4.  Each member adds up the masses r_v = (p_v - c q_v)_+ of its tiles (up to the common
// factor 2^-At_lo), one exchange gives everybody every member's total, and the member whose run contains u * R finds the token.
// Everything it reads from the workspace was written by node tasks of this launch (see st_shared_f64) before the task
// that started this one was announced.
//
// Latency only (a few microseconds of every tree, or of every step of a token-following walk): the rows are asked for at once
// and stay in registers (kKeep tiles per wave and row; longer runs are read again), so that a leaf's statistics, the masses
// and the search for the token share one read; whoever started the task says where the walk stopped (and the team that has just
// finished that node has its state); the path is recorded by the third wave at the end, and the second adds the tiles up while
// the first exchanges.  64 trees, V = 128256, an inner node: 7.5 us (12.3 with the rows read up to three times and the walk and
// the scan in front).  (Whole and partial vectors told apart per lane instead of per tile: half the code, but 36 registers in
// scratch memory and 3 % slower calls.)
//
// stop_in: the node where the walk stopped, -1: not known here (it is worked out from the tests' outcomes).
template <class E, int METHOD>
__device__ __attribute__((noinline)) int sample_task(int b_in, int stop_in) {
    using T = typename E::T;
    constexpr int NW = kTaskWaves, VEC = E::VEC, TILE = kWave * VEC, kKeep = 13;
    const Args& a = lds_launch().a;
    const Workspace& ws = lds_launch().ws;
    const TreeDesc& tree = g_tree;
    const int b = uniform_i32(b_in), known_stop = uniform_i32(stop_in), walk = uniform_i32(a.walk);
    const int lane = threadIdx.x & (kWave - 1), wave = uniform_i32(static_cast<int>(threadIdx.x) / kWave);
    float* const tile_sum = reinterpret_cast<float*>(g_rows);
    Team team = uniform_struct(g_loop.team);           // every wave its copy; the first wave's counts exchanges
    const bool leader = team.member == 0;
    __shared__ double sh_At, sh_before, sh_target, sh_total;
    __shared__ int sh_owner, sh_tile, sh_tok, sh_next;

    // where the token is drawn: the node the rule stops in, or the node a token-following walk has reached
    const bool told = walk == 0 && known_stop >= 0;
    int n = known_stop;
    if (walk) n = ld_relaxed(&ws.cur[b]);
    else if (!told) n = walk_wave<METHOD>(tree, ws, a, b, leader && wave == 0);
    n = uniform_i32(n);
    const size_t bn = static_cast<size_t>(b) * a.N + n;
    const int V = uniform_i32(a.V);
    const T* const zt = uniform_ptr(static_cast<const T*>(a.zt)) + bn * V;
    const T* const zd = uniform_ptr(static_cast<const T*>(a.zd)) + bn * V;
    const float k32 = uniform_f32(a.k32);
    // from p itself: a leaf (its target row has not been touched yet) or an NSS draw
    const bool from_p = uniform_i32(tree.nchild[n]) == 0 || walk == 1;
    double At = 0.0, Ad = 0.0, c = 0.0;
    if (!from_p && uniform_i32(g_loop.kept_task) == b * a.N + n) {
        At = g_loop.kept_At; Ad = g_loop.kept_Ad; c = g_loop.kept_c;
    } else if (!from_p) {
        At = ld_shared_f64(&ws.At[bn]);
        Ad = ld_shared_f64(&ws.Ad[bn]);
        c = ld_shared_f64(&ws.cfin[bn]);
    }
    const float u_draw = wave == 0 ? (walk ? as_global(a.draw_uniforms)[bn] : as_global(a.uniforms)[static_cast<size_t>(b) * a.N]) : 0.f;
    const int k = walk ? uniform_i32(tree.nchild[n]) : 0;
    int child_token = -1, child = 0;                   // lane j < k: child j
    if (wave == 0 && lane < k) {
        child = tree.child_list[tree.child_off[n] + lane];
        child_token = as_global(a.tokens)[static_cast<size_t>(b) * a.N + child];
    }

    const int mis = static_cast<int>((reinterpret_cast<uintptr_t>(zt) & 15u) / sizeof(T));      // the same for both rows
    const int ntiles = (mis + V + TILE - 1) / TILE;
    const int per = (ntiles + team.size - 1) / team.size;
    const int t_lo = min(team.member * per, ntiles), t_hi = min(t_lo + per, ntiles);
    const int my_tiles = t_hi - t_lo;
    const int cnt = (my_tiles - wave + NW - 1) / NW;   // this wave's tiles: t_lo + wave + NW i
    uint4 qt[kKeep], qd[kKeep];
    // 16 bytes of a row; elements before its start and after its end count as masked ones
    auto load_vec = [&](const T* row, int tile) __attribute__((always_inline)) -> uint4 {
        const int first = tile * TILE - mis;
        if (first >= 0 && first + TILE <= V) return load_raw(row + first + lane * VEC);
        struct alignas(16) { T x[VEC]; } part;
        const uint4 masked = NegInfVec<E>::v();
        __builtin_memcpy(&part, &masked, 16);
#pragma unroll
        for (int i = 0; i < VEC; ++i) {
            const int e = first + lane * VEC + i;
            if (e >= 0 && e < V) part.x[i] = as_global(row)[e];
        }
        return __builtin_bit_cast(uint4, part);
    };
    auto load_tiles = [&](int i0) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < kKeep; ++j) {
            if (i0 + j >= cnt) continue;                // (the same in every lane)
            qt[j] = load_vec(zt, t_lo + wave + NW * (i0 + j));
            if (!from_p) qd[j] = load_vec(zd, t_lo + wave + NW * (i0 + j));
        }
    };
    load_tiles(0);

    if (from_p) {
        // ---- the row's statistics first
        WaveLse<> s;
        s.init();
        for (int i0 = 0; i0 < cnt; i0 += kKeep) {
            if (i0 > 0) load_tiles(i0);
#pragma unroll
            for (int j = 0; j < kKeep; ++j) {
                if (i0 + j >= cnt) continue;
                float x[VEC];
                E::unpack(qt[j], x);
                s.vec(x, k32);
            }
        }
        const double sum = wave_sum(static_cast<double>(s.s));
        if (lane == 0) {                               // (the second row of collect_stats is not used)
            g_sh.partf[wave][0] = s.mk; g_sh.partf[wave][1] = 0.f;
            g_sh.part[wave][0] = sum; g_sh.part[wave][1] = 1.0;
        }
        task_barrier();
        if (wave == 0) {
            double none = 0.0, unused;
            collect_stats<false>(team, none, At, unused);
            if (lane == 0) sh_At = At;
        }
        task_barrier();
        At = sh_At;
        if (cnt > kKeep) load_tiles(0);
    }

    float nAt = -static_cast<float>(At), nAd = 0.f, rho = 0.f;
    const bool use_d = all_alike(c > 0.0);
    if (use_d) {
        const ResidualConsts rc = residual_consts(At, Ad, c);
        nAt = rc.nAt; nAd = rc.nAd; rho = rc.rho;
    }
    nAt = uniform_f32(nAt); nAd = uniform_f32(nAd); rho = uniform_f32(rho);
    // the masses of a lane's vector
    auto masses = [&](const uint4& vt, const uint4& vd, float (&r)[VEC]) __attribute__((always_inline)) {
        float x[VEC];
        E::unpack(vt, x);
        if (use_d) {
            float y[VEC];
            E::unpack(vd, y);
#pragma unroll
            for (int i = 0; i < VEC; ++i) r[i] = fmaxf(fmaf(-rho, fast_exp2(fmaf(y[i], k32, nAd)), fast_exp2(fmaf(x[i], k32, nAt))), 0.f);
        } else {
#pragma unroll
            for (int i = 0; i < VEC; ++i) r[i] = fast_exp2(fmaf(x[i], k32, nAt));
        }
    };
    auto lane_sum = [&](const float (&r)[VEC]) __attribute__((always_inline)) -> float {
        float s = 0.f;
#pragma unroll
        for (int i = 0; i < VEC; ++i) s += r[i];
        return s;
    };

    // ---- the mass of every tile of this member's run, in vocabulary order
    double wave_total = 0.0;
    for (int i0 = 0; i0 < cnt; i0 += kKeep) {
        if (i0 > 0) load_tiles(i0);
        float s[kKeep];
#pragma unroll
        for (int j = 0; j < kKeep; ++j) {
            s[j] = 0.f;
            if (i0 + j >= cnt) continue;
            float r[VEC];
            masses(qt[j], qd[j], r);
            s[j] = lane_sum(r);
        }
#pragma unroll
        for (int j = 0; j < kKeep; ++j) s[j] = wave_sum_f32(s[j]);              // (side by side)
#pragma unroll
        for (int j = 0; j < kKeep; ++j) {
            if (lane == 0 && i0 + j < cnt) tile_sum[wave + NW * (i0 + j)] = s[j];
            wave_total += static_cast<double>(s[j]);
        }
    }
    if (lane == 0) g_sh.part[wave][0] = wave_total;
    if (wave == 0) wait_memory();                      // (the node tasks' outcomes, for the path)
    task_barrier();

    // ---- everybody's totals (first wave), and meanwhile where this member's tiles lie (second wave: each lane a run of them)
    const int per_lane_tiles = (my_tiles + kWave - 1) / kWave;
    const int l0 = min(lane * per_lane_tiles, my_tiles), l1 = min(l0 + per_lane_tiles, my_tiles);
    double run = 0.0, incl = 0.0;
    if (wave == 0) {
        team.seq++;
        double v = g_sh.part[lane & 3][0];
        v += dpp_f64<0xB1>(v);
        v += dpp_f64<0x4E>(v);
        unsigned got[2] = {half_of(v, 0), half_of(v, 1)};
        if (team.size > 1) {
            const int at[2] = {0, 1};
            note_dead(team, swap_words<1>(team, half_of(v, lane & 1), 2, at, got));
        }
        const double mass = lane < team.size && !team.dead ? __hiloint2double(static_cast<int>(got[1]), static_cast<int>(got[0])) : 0.0;
        double in_run, total;
        const int owner = member_at(team, mass, u_draw, in_run, total);
        if (lane == 0) {
            sh_owner = owner;
            sh_target = in_run;
            sh_total = total;
        }
    } else if (wave == 1) {
        for (int t = l0; t < l1; ++t) run += tile_sum[t];
        incl = wave_inclusive_scan(run);
    }
    task_barrier();
    const int owner = uniform_i32(sh_owner);
    const bool mine_it = owner == team.member;
    if (mine_it) {
        const double local_target = sh_target;
        // ---- the tile that contains the target ...
        if (wave == 1) {
            const unsigned long long hit = __ballot(incl > local_target && run > 0.0);
            int lane_owner = hit ? (__ffsll(static_cast<long long>(hit)) - 1) : -1;
            if (lane_owner < 0) {           // rounding only: last lane that has mass
                const unsigned long long any = __ballot(run > 0.0);
                lane_owner = any ? (63 - __clzll(static_cast<long long>(any))) : 0;
            }
            if (lane == lane_owner) {
                double acc = incl - run;
                int found = -1, last = l0;
                double bef = acc;
                for (int t = l0; t < l1; ++t) {
                    const double ts = tile_sum[t];
                    if (ts > 0.0) last = t;
                    if (found < 0 && acc + ts > local_target && ts > 0.0) { found = t; bef = acc; }
                    acc += ts;
                }
                if (found < 0) {       // rounding only: last tile of the run that has mass
                    found = last;
                    bef = incl - run;
                    for (int t = l0; t < last; ++t) bef += tile_sum[t];
                }
                sh_tile = found;
                sh_before = bef;
            }
        }
        task_barrier();
        // ---- ... and the token inside that tile, by the wave that has it
        const int tile = uniform_i32(sh_tile);
        if (wave == tile % NW) {
            const double rem = local_target - sh_before;       // mass to cover inside the tile
            const int slot = tile / NW;
            uint4 vt = qt[0], vd = qd[0];
            if (cnt > kKeep) {
                vt = load_vec(zt, t_lo + tile);
                if (!from_p) vd = load_vec(zd, t_lo + tile);
            } else {
#pragma unroll
                for (int j = 1; j < kKeep; ++j)
                    if (slot == j) { vt = qt[j]; vd = qd[j]; }
            }
            float r[VEC];
            masses(vt, vd, r);
            bool near = false;
            const int found = element_at(r, lane_sum(r), lane, rem, sh_total, near);
            if (found >= 0) {
                const int tk = min(max((t_lo + tile) * TILE - mis + lane * VEC + found, 0), V - 1);
                if (k == 0) as_global(a.bonus)[b] = tk;          // (once in a walk, see draw_find)
                sh_tok = tk;
                if (near) atomicAdd(&a.counters[MPV_COUNTER_NEAR_TIE_BONUS], 1u);
            }
        }
    }
    if (told && leader && wave == 2) (void)walk_wave<METHOD>(tree, ws, a, b, true);       // the path
    int next = -1;
    if (walk) {
        // Sec. 3.2: if the drawn token is a child's token the walk moves to that child (the
        // first such child in list order), otherwise it ends here.  Everybody needs the token (the owner's word; the
        // others' say only that they have come this far).
        task_barrier();
        if (wave == 0) {
            unsigned got[1] = {static_cast<unsigned>(sh_tok)};
            if (team.size > 1) {
                team.seq++;
                const int at[1] = {0};
                note_dead(team, swap_words<1>(team, got[0], 1, at, got));
            }
            const int tok = __builtin_amdgcn_readlane(static_cast<int>(got[0]), owner);
            const unsigned long long m = __ballot(lane < k && child_token == tok);
            int to_task = -1;
            if (m) {
                const int to = __builtin_amdgcn_readlane(child, __ffsll(static_cast<long long>(m)) - 1);
                if (leader && lane == 0) st_relaxed(&ws.cur[b], to);
                // Naive and SpecTr test children of an inner node before they draw there; NSS and leaves draw at once
                to_task = (walk >= 2 && tree.nchild[to] > 0) ? b * a.N + to : a.B * a.N + b;
            } else if (leader) {
                if (lane == 0) {
                    as_global(a.bonus)[b] = tok;
                    write_path(tree, a, b, n);
                }
                if (a.dbg_accept && lane < a.N)
                    as_global(a.dbg_accept)[static_cast<size_t>(b) * a.N + lane] =
                        lane == 0 ? 1.f : static_cast<float>(ld_shared_f64(&ws.atest[static_cast<size_t>(b) * a.N + lane]));
            }
            if (lane == 0) sh_next = to_task;
        }
        task_barrier();
        next = uniform_i32(sh_next);
    }

    // ---- optional: the normalised distribution itself (of the walk's last draw; a member's share of it differs from row to row)
    if (a.dbg_resid && next < 0) {
        const double inv = 1.0 / sh_total;
        float* out = a.dbg_resid + static_cast<size_t>(b) * V;
        for (int i = 0; i < cnt; ++i) {
            const int tile = t_lo + wave + NW * i;
            const uint4 vt = load_vec(zt, tile);
            uint4 vd = vt;
            if (!from_p) vd = load_vec(zd, tile);
            float r[VEC];
            masses(vt, vd, r);
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const int e = tile * TILE - mis + lane * VEC + v;
                if (e >= 0 && e < V) out[e] = static_cast<float>(static_cast<double>(r[v]) * inv);
            }
        }
    }
    if (threadIdx.x == 0) g_loop.team = team;          // (the task loop reads it after its barrier)
    return next;
}

// ------------------------------------------------------------------ draws of the top-down rules
//
// The end of every top-down walk, and every step of a token-following one, by the whole team.  Either the node task that has
// just ended has weighed the tiles of its pair, which it had on chip (the walk stops at its node), or the token comes from p at
// a leaf (NSS: at any node): then the target row is asked for here, once, straight into LDS, and every wave weighs its
// tiles against its own largest logit, so that the row's sum and the members' shares of it are one exchange, not two, and no
// logarithm.  The member whose part holds the target finds the tile, and the wave that has it the token; a pair's tile is
// read again for that (2 KB: the registers that held it are gone, and keeping them took others from the sweeps).
//
// Latency only.  Before, a walk that had come to its end left the node task, was sent back through the task loop to
// sample_task, which read the rows once more, and for a leaf had two exchanges: 64 trees of V = 128256 on teams of 12,
// from the last test to the token 12 us (an inner node) and 16 (a leaf), now 6 and 7 (call: 88 -> 82 us; 32 of V = 262144:
// 73 -> 63; 37 of V = 50001, SpecTr: 87 -> 79; 186 of V = 1974, Naive: 96 -> 58).  sample_task stays for Traversal, whose walk
// stops at a node that another team may have had, for parts of more slots than are kept, and for the debug outputs.
//
// Returns the task that follows (-1: the walk is over; the same in every lane of every member).

// The token inside the tile that holds the target, by the wave that has it.  last: the walk ends with this draw.  (The bonus
// token is written once in a walk: several members' stores to one word, from different chiplets or with nothing that
// orders them, can leave any of them there.)
template <class E>
__device__ __forceinline__ void draw_find(const TaskDraw<E>& d, bool row, bool last, int b, int wave, int lane) {
    const Args& a = lds_launch().a;
    bool near = false;
    const int tok = d.find(uniform_i32(g_draw.in_tile), row, lane, g_draw.rem, g_draw.total, near);
    if (tok >= 0) {
        if (last) as_global(a.bonus)[b] = tok;
        g_draw.token = tok;
        if (near) atomicAdd(&a.counters[MPV_COUNTER_NEAR_TIE_BONUS], 1u);
    }
}

// 2^(from - to) of two whole numbers, exactly
__device__ __forceinline__ double unit_ratio(float from, float to) { return ldexp(1.0, static_cast<int>(fmaxf(from - to, -4096.f))); }

// First wave, when every wave has weighed its tiles: who has the target (u times the mass of the whole row), and in which tile.
__device__ __forceinline__ void draw_owner(Team& team, int slots, float u) {
    const int lane = lane_here();
    // this workgroup's tiles, lane t that of tile t, in units of 2^unit
    const float unit = fmaxf(fmaxf(g_sh.partf[0][0], g_sh.partf[1][0]), fmaxf(g_sh.partf[2][0], g_sh.partf[3][0]));
    const double of_wave = unit_ratio(g_sh.partf[draw_wave(lane)][0], unit);
    const double in_tile = lane < 2 + kTaskWaves * slots ? static_cast<double>(g_draw.tile[lane]) * of_wave : 0.0;
    const double incl = wave_inclusive_scan(in_tile), own = lane_f64(incl, kWave - 1);
    unsigned got[3] = {half_of(own, 0), half_of(own, 1), __float_as_uint(unit)};
    team.seq++;
    if (team.size > 1) {
        const int at[3] = {0, 1, 2};
        note_dead(team, swap_words<1>(team, lane < 2 ? half_of(own, lane & 1) : __float_as_uint(unit), 3, at, got));
    }
    const bool live = lane < team.size && !team.dead;
    const float of_m = live ? __uint_as_float(got[2]) : OnlineLse::kFloor, team_unit = lane_f32(row_max(of_m), 0);
    const double mass = live ? __hiloint2double(static_cast<int>(got[1]), static_cast<int>(got[0])) * unit_ratio(of_m, team_unit) : 0.0;
    double in_part, total;
    const int owner = member_at(team, mass, u, in_part, total);
    if (lane == 0) g_draw.owner = owner;
    if (owner != team.member) return;
    const double scale = unit_ratio(unit, team_unit);          // (this member has mass, or nobody has)
    const double here = in_part / scale;
    const unsigned long long hit_t = __ballot(in_tile > 0.0 && incl > here), any_t = __ballot(in_tile > 0.0);
    // (no mass anywhere: token 0, as in sample_task)
    const int tile = hit_t ? __ffsll(static_cast<long long>(hit_t)) - 1 : any_t ? 63 - __clzll(static_cast<long long>(any_t)) : 0;
    if (lane == tile) {
        g_draw.in_tile = tile;
        g_draw.rem = (here - (incl - in_tile)) / of_wave;
        g_draw.total = total / scale / of_wave;
    }
}

template <class E>
__device__ __attribute__((noinline)) int draw_walk(int b_in, int n_in, int row_in, int there_in) {
    using T = typename E::T;
    const Args& a = lds_launch().a;
    const Workspace& ws = lds_launch().ws;
    const TreeDesc& tree = g_tree;
    (void)ws;
    const int b = uniform_i32(b_in), walk = uniform_i32(a.walk), N = uniform_i32(a.N), V = uniform_i32(a.V);
    const int lane = threadIdx.x & (kWave - 1), wave = uniform_i32(static_cast<int>(threadIdx.x) / kWave);
    const int part_vecs = uniform_i32(lds_launch().q.part_vecs);
    int n = uniform_i32(n_in);
    bool row = uniform_i32(row_in) != 0, there = uniform_i32(there_in) != 0;
    Team team = uniform_struct(g_loop.team);           // every wave its copy; the first wave's counts exchanges
    const bool leader = team.member == 0;
    const size_t at = static_cast<size_t>(b) * N;
    const T* const zt0 = uniform_ptr(static_cast<const T*>(a.zt)) + at * V;
    const T* const zd0 = uniform_ptr(static_cast<const T*>(a.zd)) + at * V;
    TaskPart<E> part;
    TaskDraw<E> d(part);
    d.k32 = uniform_f32(a.k32);
    int next = -1;
    task_barrier();                                    // (every wave has waited for what it had asked for ahead)
    for (;;) {
        const size_t off = static_cast<size_t>(n) * V;
        part.setup(zt0 + off, zd0 + off, V, g_rows, g_rows + kLdsVecs * kTaskBlock, threadIdx.x, team.member, team.size, part_vecs);
        const int k = walk ? uniform_i32(tree.nchild[n]) : 0;
        float u = 0.f;
        int child = 0, child_token = -1;               // lane j < k: child j
        if (wave == 0) {                               // (asked for ahead of the row)
            u = walk ? as_global(a.draw_uniforms)[at + n] : as_global(a.uniforms)[at];
            if (lane < k) {
                child = tree.child_list[tree.child_off[n] + lane];
                child_token = as_global(a.tokens)[at + child];
            }
        }
        if (row) {
            d.weigh_row(g_draw.tile, wave, lane, there);
            if (lane == 0) g_sh.partf[wave][0] = d.mk;
        } else {
            d.f.init(d.k32, uniform_f32(g_draw.nAt), uniform_f32(g_draw.nAd), uniform_f32(g_draw.rho));
        }
        task_barrier();
        if (wave == 0) draw_owner(team, part.nslots, u);
        else if (wave == 2 && leader && k == 0) write_path(tree, a, b, n);          // (the walk ends here)
        task_barrier();
        if (uniform_i32(g_draw.owner) == team.member && wave == draw_wave(uniform_i32(g_draw.in_tile))) draw_find<E>(d, row, k == 0, b, wave, lane);
        if (k == 0) break;
        // Sec. 3.2: if the drawn token is a child's token the walk moves to that child (the first such child in list order),
        // otherwise it ends here.  Everybody needs the token (the owner's word; the others' say only that they have come
        // this far).
        task_barrier();
        if (wave == 0) {
            unsigned got[1] = {static_cast<unsigned>(g_draw.token)};
            team.seq++;
            if (team.size > 1) {
                const int word[1] = {0};
                note_dead(team, swap_words<1>(team, got[0], 1, word, got));
            }
            const int tok = __builtin_amdgcn_readlane(static_cast<int>(got[0]), uniform_i32(g_draw.owner));
            const unsigned long long m = __ballot(lane < k && child_token == tok);
            int to = -1;
            if (m != 0ull && !team.dead) to = __builtin_amdgcn_readlane(child, __ffsll(static_cast<long long>(m)) - 1);
            else if (leader && lane == 0) {
                as_global(a.bonus)[b] = tok;
                write_path(tree, a, b, n);
            }
            if (lane == 0) g_draw.next = to;
        }
        task_barrier();
        n = uniform_i32(g_draw.next);
        if (n < 0) break;
        // Naive and SpecTr test children of an inner node before they draw there; NSS and leaves draw at once
        if (walk >= 2 && uniform_i32(tree.nchild[n]) > 0) {
            next = b * N + n;
            break;
        }
        row = true;
        there = false;
    }
    if (threadIdx.x == 0) g_loop.team = team;          // (the task loop reads it after its barrier)
    return next;
}

// ------------------------------------------------------------------ stand-alone row statistics

template <class E>
__global__ __launch_bounds__(kTaskBlock) void row_stats_kernel(const typename E::T* z, int64_t rows, int V,
                                                              float k32, float* out) {
    __shared__ double scratch[2 * (kTaskBlock / kWave)];
    const int64_t r = blockIdx.x;
    RowStatsF<E> f;
    f.t.init(); f.k32 = k32;
    sweep_row<E, kTaskBlock, kTaskUnroll>(z + r * V, V, f);
    OnlineLse none; none.init();
    RowStat rt, rd;
    finish_stats2<kTaskBlock>(f.t, none, rt, rd, scratch);
    if (threadIdx.x == 0) {
        out[2 * r] = rt.m;
        // ln sum exp((z-m)/T) = ln2 * (A - m*k32)
        out[2 * r + 1] = static_cast<float>(0.6931471805599453 * (rt.A - static_cast<double>(rt.m) * static_cast<double>(k32)));
    }
}

// Debug statistics [B,N,4] from the workspace (internal nodes, stopping leaves) --
// rows the path never touched are computed here.
template <class E>
__global__ __launch_bounds__(kTaskBlock) void debug_stats_kernel(TreeDesc tree, Args a) {
    using T = typename E::T;
    __shared__ double scratch[2 * (kTaskBlock / kWave)];
    const int64_t bn = blockIdx.x;
    const int n = static_cast<int>(bn % a.N);
    const T* zt = static_cast<const T*>(a.zt) + bn * a.V;
    const T* zd = static_cast<const T*>(a.zd) + bn * a.V;
    const bool leaf = tree.nchild[n] == 0;
    RowStat rt, rd;
    if (leaf) {
        RowStatsF<E> f;
        f.t.init(); f.k32 = a.k32;
        sweep_row<E, kTaskBlock, kTaskUnroll>(zt, a.V, f);
        OnlineLse none; none.init();
        finish_stats2<kTaskBlock>(f.t, none, rt, rd, scratch);
    } else {
        PairStatsF<E, kTaskBlock, kTaskUnroll> f;
        f.t.init(); f.d.init(); f.k32 = a.k32;
        sweep_pair<E, kTaskBlock, kTaskUnroll>(zt, zd, a.V, f);
        finish_stats2<kTaskBlock>(f.t, f.d, rt, rd, scratch);
    }
    if (threadIdx.x == 0) {
        const double kd = static_cast<double>(a.k32);
        float* o = a.dbg_stats + bn * 4;
        o[0] = rt.m;
        o[1] = static_cast<float>(0.6931471805599453 * (rt.A - static_cast<double>(rt.m) * kd));
        o[2] = leaf ? NAN : rd.m;
        o[3] = leaf ? NAN : static_cast<float>(0.6931471805599453 * (rd.A - static_cast<double>(rd.m) * kd));
    }
}

// ------------------------------------------------------------------ uniforms

__global__ void fill_uniforms_kernel(uint64_t seed, int64_t count, float* out) {
    const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= count) return;
    uint64_t z = seed + static_cast<uint64_t>(i + 1) * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z = z ^ (z >> 31);
    out[i] = static_cast<float>(z >> 40) * (1.0f / 16777216.0f);
}

// ------------------------------------------------------------------ host side

thread_local int g_last_hip_error = 0;

static bool hip_ok(hipError_t e) {
    if (e == hipSuccess) return true;
    g_last_hip_error = static_cast<int>(e);
    return false;
}

// Optional per-launch timing: when enabled, every kernel launched by mpv_verify carries a pair
// of hipEvents that the runtime stamps with the start and the end of that dispatch itself
// (hipExtLaunchKernelGGL): no extra packet goes into the stream, the launches stay back to back.
struct LaunchTimer {
    bool enabled = false;
    int capacity = 0, used = 0;
    hipEvent_t* start = nullptr;
    hipEvent_t* stop = nullptr;
    int32_t* kernel = nullptr;
};
static LaunchTimer g_timer;

template <typename... Params, typename... Args>
static void launch(int kernel_id, void (*kernel)(Params...), dim3 grid, dim3 block, hipStream_t s, Args... args) {
    if (g_timer.enabled && g_timer.used < g_timer.capacity) {
        const int slot = g_timer.used++;
        g_timer.kernel[slot] = kernel_id;
        hipExtLaunchKernelGGL(kernel, grid, block, 0, s, g_timer.start[slot], g_timer.stop[slot], 0,
                              static_cast<Params>(args)...);
    } else {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, static_cast<Params>(args)...);
    }
}

struct Plan {
    TreeDesc tree;
    int max_tree_depth;
    int n_internal;
    int nclass;
    int64_t class_tasks[kMaxClasses];      // tasks a class can ever hold, over the batch
    const int32_t* shapes;                 // HOST [B,N]: a parent array per tree, checked; null: every tree is `tree`
    bool teams_apart = false;              // tests only (mpv_test_verify_teams_apart)
};

// What the checks of one parent array find out.
struct TreeScan {
    int nch[MPV_MAX_NODES], depth[MPV_MAX_NODES];
    int max_depth, internal, trunk;        // trunk: internal nodes from the root down to the first that branches
    bool branches;
};

static int scan_tree(const int32_t* parent, int N, int max_depth, TreeScan* t) {
    if (parent[0] != -1) return MPV_ERR_BAD_TREE;
    memset(t->nch, 0, sizeof(int) * static_cast<size_t>(N));
    t->depth[0] = 0;
    for (int n = 1; n < N; ++n) {
        const int par = parent[n];
        if (par < 0 || par >= n) return MPV_ERR_BAD_TREE;
        t->depth[n] = t->depth[par] + 1;
        ++t->nch[par];
    }
    t->max_depth = t->internal = t->trunk = 0;
    for (int n = 0; n < N; ++n) {
        if (t->nch[n] > MPV_MAX_CHILDREN) return MPV_ERR_UNSUPPORTED;
        if (t->depth[n] > t->max_depth) t->max_depth = t->depth[n];
        if (t->nch[n]) ++t->internal;
    }
    // (the nodes of a trunk come in ascending order, each the only one of its depth)
    int branch = 0;
    for (int n = 1; n < N && t->nch[branch] == 1; ++n)
        if (parent[n] == branch) branch = n;
    t->branches = t->nch[branch] > 0;
    t->trunk = t->depth[branch] + (t->branches ? 1 : 0);
    return t->max_depth > max_depth ? MPV_ERR_BAD_SHAPE : MPV_OK;
}

// Queue space: class 0 holds the trunk's tasks and the sampling task, class 1 the other nodes' and the resumed one.
static void count_tasks(const TreeScan& t, int64_t trees, Plan* plan) {
    plan->class_tasks[0] += trees * (t.trunk + 1);
    if (t.branches) plan->class_tasks[1] += trees * (t.internal - t.trunk + 1);
    if (t.branches) plan->nclass = 2;
}

static int validate(const mpv_problem* p, Plan* plan) {
    if (!p) return MPV_ERR_NULL;
    if (p->B < 0 || p->N < 1 || p->V < 1) return MPV_ERR_BAD_SHAPE;
    if (p->N > MPV_MAX_NODES || p->V > MPV_MAX_VOCAB) return MPV_ERR_UNSUPPORTED;
    // task numbers (tree * N + node, and two more per tree) are 32-bit
    if (static_cast<int64_t>(p->B) * (p->N + 2) > (1ll << 30)) return MPV_ERR_UNSUPPORTED;
    if (p->method < MPV_METHOD_SPECINFER || p->method > MPV_METHOD_SPECTR) return MPV_ERR_BAD_METHOD;
    if (p->logit_dtype != MPV_DTYPE_F32 && p->logit_dtype != MPV_DTYPE_BF16) return MPV_ERR_BAD_DTYPE;
    if (!(p->temperature > 0.0f) || !isfinite(p->temperature)) return MPV_ERR_BAD_TEMPERATURE;
    if (!p->parent) return MPV_ERR_NULL;
    TreeScan scan;
    const int rc = scan_tree(p->parent, p->N, p->max_depth, &scan);
    if (rc != MPV_OK) return rc;
    TreeDesc& t = plan->tree;
    memset(plan, 0, sizeof(*plan));
    t.N = p->N;
    t.parent[0] = -1;
    t.split_node = -1;
    int off = 0;
    for (int n = 0; n < p->N; ++n) {
        if (n) t.parent[n] = static_cast<int8_t>(p->parent[n]);
        t.depth[n] = static_cast<int8_t>(scan.depth[n]);
        t.nchild[n] = static_cast<int8_t>(scan.nch[n]);
        t.child_off[n] = static_cast<int8_t>(off);
        off += scan.nch[n];
    }
    int fill[MPV_MAX_NODES] = {0};
    for (int n = 1; n < p->N; ++n) {
        const int par = t.parent[n];
        t.child_list[t.child_off[par] + fill[par]++] = n;
    }
    {   // depth-first post-order without recursion
        int next_child[MPV_MAX_NODES] = {0};
        int n = 0, out = 0;
        for (;;) {
            if (next_child[n] < t.nchild[n]) {
                n = t.child_list[t.child_off[n] + next_child[n]++];
                continue;
            }
            t.postorder[out++] = n;
            if (n == 0) break;
            n = t.parent[n];
        }
    }
    for (int r = 0; r < p->N; ++r) t.rank[t.postorder[r]] = r;
    for (int r = 0; r < p->N; ++r) {                  // children come before their parent
        const int n = t.postorder[r];
        t.sub_lo[n] = t.nchild[n] ? t.sub_lo[t.child_list[t.child_off[n]]] : r;
    }
    {   // priority classes: 0 from the root down to the first node that branches, 1 below it
        int branch = 0;
        while (t.nchild[branch] == 1) branch = t.child_list[t.child_off[branch]];
        for (int n = 0; n < p->N; ++n) t.cls[n] = (t.depth[n] <= t.depth[branch]) ? 0 : 1;
    }
    plan->nclass = 1;
    count_tasks(scan, p->B, plan);
    plan->max_tree_depth = scan.max_depth;
    plan->n_internal = scan.internal;
    return MPV_OK;
}

static size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

static size_t carve(const mpv_problem* p, void* base, Workspace* ws) {
    const size_t bn = static_cast<size_t>(p->B) * p->N;
    size_t off = 0;
    char* b = static_cast<char*>(base);
    auto take = [&](size_t bytes) { void* q = b ? b + off : nullptr; off = align_up(off + bytes, 256); return q; };
    double* At = static_cast<double*>(take(bn * 8));
    double* Ad = static_cast<double*>(take(bn * 8));
    double* cf = static_cast<double*>(take(bn * 8));
    double* ax = static_cast<double*>(take(bn * 8));
    double* a0 = static_cast<double*>(take(bn * 8));
    double* at = static_cast<double*>(take(bn * 8));
    int32_t* qu = static_cast<int32_t*>(take(bn * 4));
    int32_t* qc = static_cast<int32_t*>(take(kCtlWords * 4));
    int32_t* mb = static_cast<int32_t*>(take(kMailboxWords * 4));
    unsigned long long* kn = static_cast<unsigned long long*>(take(static_cast<size_t>(p->B) * 8));
    unsigned long long* ac = static_cast<unsigned long long*>(take(static_cast<size_t>(p->B) * 8));
    int32_t* de = static_cast<int32_t*>(take(static_cast<size_t>(p->B) * 4));
    int32_t* cu = static_cast<int32_t*>(take(static_cast<size_t>(p->B) * 4));
    unsigned long long* ex = static_cast<unsigned long long*>(take(static_cast<size_t>(kMaxGrid) * 2 * kExchWords * 8));
    unsigned long long* tt = static_cast<unsigned long long*>(take(static_cast<size_t>(kMaxTeams) * 2 * 8));
    LaunchBlock* la = static_cast<LaunchBlock*>(take(sizeof(LaunchBlock)));
    if (ws) { ws->exch = ex; ws->team_task = tt; ws->launch = la; }
    if (ws) { ws->At = At; ws->Ad = Ad; ws->cfin = cf; ws->aux = ax; ws->a0 = a0; ws->atest = at; ws->queue = qu; ws->qctl = qc; ws->mailbox = mb; ws->known = kn; ws->acc = ac; ws->decided = de; ws->cur = cu; }
    return off < 256 ? 256 : off;
}

// Calls fn(b0, b1) for every run [b0, b1) of consecutive equal rows of rows[B][N], in order, until fn returns false.
template <typename F>
static void for_each_run(const int32_t* rows, int32_t B, int32_t N, F fn) {
    for (int32_t b0 = 0; b0 < B;) {
        int32_t b1 = b0 + 1;
        while (b1 < B && memcmp(rows + static_cast<size_t>(b0) * N, rows + static_cast<size_t>(b1) * N, sizeof(int32_t) * N) == 0)
            ++b1;
        if (!fn(b0, b1)) return;
        b0 = b1;
    }
}

static int compute_units() {
    static int cus = 0;
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) == hipSuccess &&
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0)
            cus = n;
        else
            cus = 256;
    }
    return cus;
}

// How a launch is shaped: G workgroups per team so that a member's part of a row fits on chip
// (kMaxTeam at most: beyond that the rest of a part is re-read in every sweep), as many teams
// as there are tasks at once (see launch_all), three workgroups per compute unit at most.
constexpr int kWantedPart = 1024;                     // vectors of a row per member where there are members to spare, see launch_shape
struct Shape { int team_size, teams, part_vecs, same_xcd; };

// Workgroups of a task kernel that one compute unit holds at a time, as the runtime computes it
// from the kernel's registers and LDS (3 by design); a team never has more members than can be
// resident together.
template <class K>
static int resident_per_cu(K kernel) {
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kTaskBlock, 0) != hipSuccess || n < 1) {
        (void)hipGetLastError();
        n = 1;
    }
    return n;
}

// tasks: how many there can be at once;  teams_wanted: parts are made shorter than that for as long as there are so many
// teams (0: not).
template <class E>
static Shape launch_shape(const mpv_problem* p, int tasks, int64_t independent, int64_t teams_wanted, int per_cu) {
    Shape s;
    const int nvec = (p->V + E::VEC - 1) / E::VEC;
    const int slots = per_cu * compute_units() < kMaxGrid ? per_cu * compute_units() : kMaxGrid;      // workgroups that can be resident
    // The fewest members whose kept parts (plus the one overflow slot a sweep hides) hold a row:
    // the most teams, which is what counts when there are more trees than teams.
    // With fewer a task's own time counts: more members, parts of about 2048 vectors (measured: shorter
    // parts no longer pay for the larger exchange), as long as there is a team for each.
    int g = 1;
    while (g < kMaxTeam && static_cast<long long>(g) * (kPartCapacity + kTaskBlock / 2) < nvec) ++g;
    const int fewest = g;
    while (g < kMaxTeam && slots / (g + 1) >= p->B && static_cast<long long>(g) * 2048 < nvec) ++g;
    while (teams_wanted > 0 && g < kMaxTeam && slots / (g + 1) >= teams_wanted && static_cast<long long>(g) * kWantedPart < nvec) ++g;
    auto teams_of = [&](int size) {
        const int most = max(1, min(slots / size, kMaxTeams));
        int teams = max(1, min(most, tasks));
        // workgroup i runs on chiplet i % 8: with a multiple of 8 teams every team can stay on one chiplet
        if (size > 1 && most >= 8) teams = min((teams + 7) / 8 * 8, most - most % 8);
        return teams;
    };
    // Tasks that do not depend on each other: the size whose rounds take the least time.  A task's own time is
    // a part that no team shortens (exchanges, scalar steps) and one that goes with a member's vectors; the two
    // are equal at about 1900 vectors (22 us a task with parts of 1 900, 30 with 3 165).  64 trees of 33 inner
    // nodes, V = 151936: 670 us with 72 teams of 10, 497 with 128 of 6 (392 by now); but 4 such trees of V = 262144 are three
    // rounds either way, 91 us with teams of 16, 97 with teams of 11.  (The constant is SpecInfer's in bf16 at V = 151936;
    // with the others the sizes it gives are faster too than those that the trees give: SpecTr 791 -> 609 us, NSS
    // 822 -> 628, Naive 783 -> 598; 24 trees of V = 100003 in float32, 12 inner nodes: 137 -> 98, 150 -> 109, 146 -> 106.)
    if (independent > 0) {
        double least = 0.0;
        for (int size = g; size >= fewest; --size) {
            const int64_t teams = teams_of(size);
            const double time = static_cast<double>((independent + teams - 1) / teams) * (1.0 + nvec / (1900.0 * size));
            if (size == g || time < least) { least = time; s.team_size = size; }
        }
        g = s.team_size;
    }
    const int teams = teams_of(g);
    s.same_xcd = (g > 1 && teams >= 8) ? 1 : 0;
    s.team_size = g;
    s.teams = teams;
    const int tiles = (nvec + kWave - 1) / kWave;                 // wave tiles of 64 vectors
    s.part_vecs = ((tiles + g - 1) / g) * kWave;
    return s;
}

template <class E>
static int launch_all(const mpv_problem* p, const Plan& plan, const Workspace& ws, const Args& a, hipStream_t s) {
    TreeDesc tree = plan.tree;
    (void)hipGetLastError();    // a stale error left by the caller's own HIP calls is not ours
    // Queue layout and initial tasks.  Computing only what is needed, both rules start from the
    // root: SpecInfer queues the accepted child, Traversal the children of positive weight.
    // Computing everything (debug outputs), SpecInfer's node tasks are independent and all
    // there from the start, nodes with many children (the long tasks) first.
    QueuePlan q;
    memset(&q, 0, sizeof(q));
    q.nclass = plan.nclass;
    for (int c = 0; c < q.nclass; ++c) q.off[c + 1] = q.off[c] + static_cast<int>(plan.class_tasks[c]);
    const bool all_up_front = (p->method != MPV_METHOD_TRAVERSAL && !a.lazy);
    int first_nodes = 0;
    for (int c = 0; c < q.nclass; ++c)
        for (int kk = MPV_MAX_CHILDREN; kk >= 1; --kk)
            for (int n = 0; n < p->N; ++n)
                if (tree.cls[n] == c && tree.nchild[n] == kk && (all_up_front || n == 0) && (a.walk != 1 || !a.lazy))      // NSS verification has no node tasks
                    q.init_node[first_nodes++] = static_cast<int8_t>(n);
    q.init_total = first_nodes * p->B;
    if (tree.nchild[0] == 0 || (a.walk == 1 && a.lazy)) {
        q.root_is_leaf = 1;
        q.init_total = p->B;
    }
    for (int c = 0; c <= q.nclass; ++c) tree.class_off[c] = q.off[c];
    const int tasks = q.off[q.nclass];
    static const int per_cu[3] = {min(min(resident_per_cu(node_task_kernel<E, MPV_METHOD_SPECINFER>), resident_per_cu(staged_part_kernel<E>)),
                                      min(resident_per_cu(walk_kernel<E>), resident_per_cu(short_part_kernel<E>))),
                                  resident_per_cu(node_task_kernel<E, MPV_METHOD_TRAVERSAL>),
                                  resident_per_cu(node_task_kernel<E, kKindAcceptance>)};
    // Tasks that do not depend on each other: every node's for the acceptance rates.  (A rate is 1 less a mass: with other
    // parts, so sums in another order, it moves by 7e-7 at most.)  Block efficiency keeps the size that the trees give,
    // although its tasks could be counted too (64 trees of 33 inner nodes, V = 151936, Traversal: 485 us, 399 with teams of
    // 6; SpecInfer 523 and 421): probabilities further down a tree are quotients of differences, p - c q over what is left of p, and sums in
    // another order then move single ones by 1e-5 (against 64 bits both are equally far off, up to 5e-5 over 71 such batches).
    const bool top_down = p->method != MPV_METHOD_TRAVERSAL;
    // Only what is needed: a top-down walk has one task at a time per tree, and teams without a task only take issue slots
    // and memory requests from the others (64 trees of V = 32000 in float32: 72.6 us with the 96 teams that tasks could be
    // queued for, 56.8 with 64; 200 trees of V = 4096: 110 and 72).  Traversal can follow the branches of a tree at the same
    // time, which pays for about two a tree, and up to 192 teams, beyond which they wait for the dispatcher (200 trees of
    // V = 1500, 3 branches: 138 us with 200 teams, 149 with 256, 213 with 416, 273 with 512; 2 trees want the 16 more).
    const int branches = min(2 * p->B + 16, max(p->B, 192));       // (B * (N + 2) is at most 2^30)
    const int at_once = !a.lazy ? tasks : min(tasks, top_down ? p->B : branches);
    // Shorter parts pay as long as every tree (Traversal: four branches of it) still has a team: one tree of V = 32000, top
    // down, 62 us with parts of 2000 vectors, 57 with 1333, 54 with 1000; 200 trees of V = 16000, Traversal, on fewer teams for it: 182 and 154.
    const int64_t teams_wanted = !a.lazy ? 0 : top_down ? p->B : 4ll * p->B;
    const int64_t independent = a.estimate == 2 ? static_cast<int64_t>(p->B) * plan.n_internal : 0;
    const Shape shape = launch_shape<E>(p, at_once, independent, teams_wanted, per_cu[a.estimate == 2 ? 2 : (p->method == MPV_METHOD_TRAVERSAL ? 1 : 0)]);
    q.teams = shape.teams;
    q.team_size = shape.team_size;
    q.part_vecs = shape.part_vecs;
    q.same_xcd = plan.teams_apart ? 0 : shape.same_xcd;
    // Walks draw their tokens themselves where the last slot of a part is kept, or is the one that a sweep reads again; longer
    // parts are drawn from by sample_task, like the calls with debug outputs of the draw (64 trees of V = 128256, SpecInfer: 88 us by it, 82
    // by draw_walk).
    const bool draws = top_down && a.lazy && !a.estimate && !a.dbg_accept && !a.dbg_resid && q.part_vecs <= kPartCapacity + kTaskBlock;
    // Up to four slots; six for SpecTr, which sweeps a part about seven times for one load.  With more the chip is full of teams
    // and loads, and what is asked for in vain holds the others up (64 trees of V = 128256, parts of 1 344 vectors: SpecInfer 73.2 us
    // by the other kernel, 74.9 by this, SpecTr 186 and 182; 64 of V = 32000, parts of 512: 65.2 and 62.9).
    const bool short_part = top_down && a.estimate != 2 && q.part_vecs <= (a.walk == 3 ? kRegVecs : 4) * kTaskBlock;
    q.box_step = 16;                                   // a cache line each, while there is room for it
    while (q.teams * q.box_step > kMailboxWords) q.box_step /= 2;
    // (The few teams that launch_shape adds to fill whole chiplets are not meant: with them in the comparison the branching
    // node was split at 200 and 208 trees, but not in between, 247 trees of V = 64000 took 238 us and 248 took 222.)
    const int teams_asked_for = min(q.teams, at_once);
    q.spare = teams_asked_for > q.init_total ? 1 : 0;
    const bool split = p->method == MPV_METHOD_TRAVERSAL && a.lazy && p->B >= teams_asked_for;
    if (a.per_tree) {
        // (the root of every tree is an inner node, N > 1: the first tasks are the same for all of them)
        const int per_chunk = kShapeChunkBytes / p->N;
        for (int b0 = 0; b0 < p->B; b0 += per_chunk) {
            const int trees = min(per_chunk, p->B - b0);
            ShapeChunk chunk;
            const int32_t* rows = plan.shapes + static_cast<size_t>(b0) * p->N;
            for (int i = 0; i < trees * p->N; ++i) chunk.parent[i] = static_cast<unsigned char>(rows[i]);
            launch(MPV_KERNEL_INIT, shape_kernel, dim3(trees), dim3(kWave), s, chunk, reinterpret_cast<unsigned long long*>(ws.aux), b0, p->N, split ? 1 : 0);
        }
    } else if (split) {
        int branch = 0;
        while (tree.nchild[branch] == 1) branch = tree.child_list[tree.child_off[branch]];
        if (tree.nchild[branch] >= 2) {
            const int first = tree.child_list[tree.child_off[branch]];
            if (tree.nchild[first] > 0) {
                const int hi = tree.rank[first], lo = tree.sub_lo[first];
                const unsigned long long upto = (hi >= 63) ? ~0ull : ((1ull << (hi + 1)) - 1ull);
                tree.split_node = branch;
                tree.split_mask = upto & ~((1ull << lo) - 1ull);
            }
        }
    }
    {
        const int threads = kInitBlock;
        const int blocks = (max(p->B, 64) + threads - 1) / threads;
        LaunchBlock block;
        block.l.q = q; block.l.ws = ws; block.l.a = a; block.tree = tree;
        launch(MPV_KERNEL_INIT, init_kernel, dim3(blocks, p->N), dim3(threads), s, block);
    }
    if (tasks > 0) {
        const dim3 grid(static_cast<unsigned>(q.teams * q.team_size)), block(kTaskBlock);
        if (a.estimate == 2) {
            launch(MPV_KERNEL_NODE_TASK, node_task_kernel<E, kKindAcceptance>, grid, block, s, const_cast<const LaunchBlock*>(ws.launch));
        } else if (p->method != MPV_METHOD_TRAVERSAL) {      // NSS, Naive and SpecTr are variants of the top-down kernels
            launch(MPV_KERNEL_NODE_TASK, draws ? (short_part ? short_part_kernel<E> : walk_kernel<E>)
                                               : (short_part ? staged_part_kernel<E> : node_task_kernel<E, MPV_METHOD_SPECINFER>),
                   grid, block, s, const_cast<const LaunchBlock*>(ws.launch));
        } else {
            launch(MPV_KERNEL_NODE_TASK, node_task_kernel<E, MPV_METHOD_TRAVERSAL>, grid, block, s, const_cast<const LaunchBlock*>(ws.launch));
        }
    }
    if (a.dbg_stats) {
        launch(MPV_KERNEL_DEBUG_STATS, debug_stats_kernel<E>, dim3(static_cast<unsigned>(p->B) * p->N), dim3(kTaskBlock), s, tree, a);
    }
    return hip_ok(hipGetLastError()) ? MPV_OK : MPV_ERR_HIP;
}

template <class E>
static void launch_nucleus(const typename E::T* in, typename E::T* out, int64_t rows, int32_t V, float k32, float top_p,
                           int keep_all, float* threshold_out, int32_t* kept_out, hipStream_t s) {
    const dim3 grid(static_cast<unsigned>(rows));
    if (V / E::VEC >= kNucleusLongRow)
        hipLaunchKernelGGL((nucleus_kernel<E, 1024>), grid, dim3(1024), 0, s, in, out, V, k32, top_p, keep_all, threshold_out, kept_out);
    else
        hipLaunchKernelGGL((nucleus_kernel<E, 256>), grid, dim3(256), 0, s, in, out, V, k32, top_p, keep_all, threshold_out, kept_out);
}

// ------------------------------------------------------------------ static scratch

// Scratch of mpv_verify_static: the workspace of one call, held by every device the library
// runs on until the process ends.  In host code the array's name is only a handle; its device
// address is looked up once per device (scratch_address) and only that pointer is ever used.
static __device__ __align__(256) unsigned char scratch[MPV_STATIC_WORKSPACE_BYTES];

constexpr int kMaxDevices = 64;
static std::atomic<void*> g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device (null + error code on failure).
static int scratch_address(void** out) {
    int dev = 0;
    if (!hip_ok(hipGetDevice(&dev))) return MPV_ERR_HIP;
    if (dev < 0 || dev >= kMaxDevices) return MPV_ERR_UNSUPPORTED;
    void* p = g_scratch_ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        if (!hip_ok(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch))) || !p) return MPV_ERR_HIP;
        g_scratch_ptr[dev].store(p, std::memory_order_release);     // every thread finds the same address
    }
    *out = p;
    return MPV_OK;
}

}  // namespace mpv

// ------------------------------------------------------------------ C ABI

extern "C" {

int mpv_version(void) { return MPV_ABI_VERSION; }

const char* mpv_strerror(int code) {
    switch (code) {
        case MPV_OK: return "success";
        case MPV_ERR_NULL: return "a required pointer is NULL";
        case MPV_ERR_BAD_SHAPE: return "invalid B, N, V or max_depth smaller than the tree depth";
        case MPV_ERR_BAD_TREE: return "invalid parent array (need parent[0] = -1 and 0 <= parent[n] < n)";
        case MPV_ERR_BAD_TEMPERATURE: return "temperature must be a finite number > 0";
        case MPV_ERR_BAD_METHOD: return "unknown method id";
        case MPV_ERR_BAD_DTYPE: return "unknown logit dtype";
        case MPV_ERR_WORKSPACE: return "workspace is NULL, not 256-byte aligned or too small";
        case MPV_ERR_UNSUPPORTED: return "problem exceeds MPV_MAX_NODES / MPV_MAX_CHILDREN / MPV_MAX_VOCAB, or a debug output this method does not provide was requested";
        case MPV_ERR_HIP: return "a HIP call failed (see mpv_last_hip_error)";
        case MPV_ERR_ALIGNMENT: return "logit base pointers must be 16-byte aligned";
        case MPV_ERR_BAD_TOP_P: return "top_p must lie in (0, 1]";
        default: return "unknown error code";
    }
}

int mpv_last_hip_error(void) { return mpv::g_last_hip_error; }

int mpv_workspace_bytes(const mpv_problem* problem, size_t* out) {
    if (!out) return MPV_ERR_NULL;
    mpv::Plan plan;
    const int rc = mpv::validate(problem, &plan);
    if (rc != MPV_OK) return rc;
    *out = mpv::carve(problem, nullptr, nullptr);
    return MPV_OK;
}

// part_of_batch: the buffers are those of a larger batch moved on by a whole number of trees (the two
// logit pointers by the same number of bytes, so the rows of a pair still share their offset modulo 16
// bytes, which is what the kernels rely on; the caller has checked the batch's own pointers);
// keep_counters: add to the counters instead of starting them at zero.
// context_node: see Args (device pointer, already moved on to the run's first tree).
// shapes: HOST [B,N], a parent array per tree, all of them checked (problem->parent is the first); null: one shape.
static int verify_with_workspace(const mpv_problem* problem, const mpv_buffers* buf, void* workspace,
                                 size_t workspace_bytes, void* hip_stream, bool part_of_batch = false,
                                 bool keep_counters = false, const int32_t* context_node = nullptr,
                                 const int32_t* shapes = nullptr, bool teams_apart = false);

// Only what the rule needs is computed: nobody has asked for per-node outputs.
static bool only_what_is_needed(const mpv_problem* p, const mpv_buffers* buf) {
    return (p->method != MPV_METHOD_SPECINFER && p->method != MPV_METHOD_TRAVERSAL) ||
           (!buf->edge_probs && !buf->accept_prob && !buf->stats);
}

int mpv_verify(const mpv_problem* problem, const mpv_buffers* buf, void* workspace,
               size_t workspace_bytes, void* hip_stream) {
    return verify_with_workspace(problem, buf, workspace, workspace_bytes, hip_stream);
}

// For tests, not in the header: mpv_verify with the members of a team on different chiplets (consecutive workgroups), where
// they exchange words at device scope.  No other call can choose this layout, and nothing but the layout differs.
int mpv_test_verify_teams_apart(const mpv_problem* problem, const mpv_buffers* buf, void* workspace,
                                size_t workspace_bytes, void* hip_stream) {
    return verify_with_workspace(problem, buf, workspace, workspace_bytes, hip_stream, false, false, nullptr, nullptr, true);
}

int mpv_verify_static(const mpv_problem* problem, const mpv_buffers* buf, void* hip_stream) {
    mpv::Plan plan;
    const int rc = mpv::validate(problem, &plan);
    if (rc != MPV_OK) return rc;
    if (mpv::carve(problem, nullptr, nullptr) > MPV_STATIC_WORKSPACE_BYTES) return MPV_ERR_WORKSPACE;
    void* ws = nullptr;
    const int rs = mpv::scratch_address(&ws);
    if (rs != MPV_OK) return rs;
    return verify_with_workspace(problem, buf, ws, MPV_STATIC_WORKSPACE_BYTES, hip_stream);
}

static int verify_with_workspace(const mpv_problem* problem, const mpv_buffers* buf, void* workspace,
                                 size_t workspace_bytes, void* hip_stream, bool part_of_batch, bool keep_counters,
                                 const int32_t* context_node, const int32_t* shapes, bool teams_apart) {
    mpv::Plan plan;
    const int rc = mpv::validate(problem, &plan);
    if (rc != MPV_OK) return rc;
    plan.teams_apart = teams_apart;
    if (shapes) {
        memset(plan.class_tasks, 0, sizeof(plan.class_tasks));
        mpv::TreeScan scan;
        mpv::for_each_run(shapes, problem->B, problem->N, [&](int32_t b0, int32_t b1) {
            (void)mpv::scan_tree(shapes + static_cast<size_t>(b0) * problem->N, problem->N, problem->max_depth, &scan);
            mpv::count_tasks(scan, b1 - b0, &plan);
            return true;
        });
        plan.shapes = shapes;
    }
    if (!buf) return MPV_ERR_NULL;
    if (problem->B == 0) return MPV_OK;
    if (!buf->target_logits || !buf->draft_logits || !buf->tokens || !buf->uniforms || !buf->accept_len ||
        !buf->path_nodes || !buf->path_tokens || !buf->bonus_token || !buf->counters)
        return MPV_ERR_NULL;
    if (!part_of_batch &&
        ((reinterpret_cast<uintptr_t>(buf->target_logits) & 15u) || (reinterpret_cast<uintptr_t>(buf->draft_logits) & 15u)))
        return MPV_ERR_ALIGNMENT;
    if (((reinterpret_cast<uintptr_t>(buf->target_logits) ^ reinterpret_cast<uintptr_t>(buf->draft_logits)) & 15u) != 0)
        return MPV_ERR_ALIGNMENT;
    const size_t need = mpv::carve(problem, nullptr, nullptr);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < need) return MPV_ERR_WORKSPACE;

    mpv::Workspace ws;
    mpv::carve(problem, workspace, &ws);
    mpv::Args a;
    const int walk = problem->method == MPV_METHOD_NSS ? 1 : problem->method == MPV_METHOD_NAIVE ? 2
                   : problem->method == MPV_METHOD_SPECTR ? 3 : 0;
    if (walk && !buf->draw_uniforms) return MPV_ERR_NULL;
    if (walk && (buf->stats || buf->edge_probs)) return MPV_ERR_UNSUPPORTED;
    a.zt = buf->target_logits; a.zd = buf->draft_logits; a.tokens = buf->tokens; a.uniforms = buf->uniforms;
    a.draw_uniforms = buf->draw_uniforms; a.walk = walk;
    a.accept_len = buf->accept_len; a.path_nodes = buf->path_nodes; a.path_tokens = buf->path_tokens;
    a.bonus = buf->bonus_token; a.counters = buf->counters;
    a.dbg_stats = buf->stats; a.dbg_edge = buf->edge_probs; a.dbg_accept = buf->accept_prob; a.dbg_resid = buf->final_residual;
    a.B = problem->B; a.N = problem->N; a.V = problem->V; a.max_depth = problem->max_depth;
    a.k32 = static_cast<float>(1.4426950408889634 / static_cast<double>(problem->temperature));
    a.lazy = only_what_is_needed(problem, buf) ? 1 : 0;
    a.per_tree = shapes ? 1 : 0;
    a.estimate = 0; a.reach_prob = nullptr; a.expected = nullptr;
    a.keep_counters = keep_counters ? 1 : 0;
    a.context_node = context_node;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (problem->logit_dtype == MPV_DTYPE_F32) return mpv::launch_all<mpv::ElemF32>(problem, plan, ws, a, s);
    return mpv::launch_all<mpv::ElemBF16>(problem, plan, ws, a, s);
}

int mpv_merge_duplicates(const int32_t* parent, const int32_t* tokens, int32_t B, int32_t N,
                         int32_t* merged_parent, int32_t* context_node) {
    if (!parent || !merged_parent || (B > 0 && !tokens)) return MPV_ERR_NULL;
    if (B < 0 || N < 1) return MPV_ERR_BAD_SHAPE;
    if (N > MPV_MAX_NODES) return MPV_ERR_UNSUPPORTED;
    if (parent[0] != -1) return MPV_ERR_BAD_TREE;
    for (int n = 1; n < N; ++n)
        if (parent[n] < 0 || parent[n] >= n) return MPV_ERR_BAD_TREE;
    for (int32_t b = 0; b < B; ++b) {
        const int32_t* tok = tokens + static_cast<size_t>(b) * N;
        int32_t* out = merged_parent + static_cast<size_t>(b) * N;
        // stands_for[n]: the node of slot n's context; entries[c]: the slots already placed under the
        // context node c that are nodes themselves (one per distinct token), in slot order
        int32_t stands_for[MPV_MAX_NODES];
        int8_t entries[MPV_MAX_NODES][MPV_MAX_NODES];
        int8_t count[MPV_MAX_NODES];
        memset(count, 0, sizeof(count));
        stands_for[0] = 0;
        out[0] = -1;
        for (int n = 1; n < N; ++n) {
            const int under = stands_for[parent[n]];
            out[n] = under;
            stands_for[n] = n;
            for (int j = 0; j < count[under]; ++j) {
                const int m = entries[under][j];
                if (tok[m] == tok[n]) { stands_for[n] = m; break; }
            }
            if (stands_for[n] == n) entries[under][count[under]++] = static_cast<int8_t>(n);
        }
        if (context_node) memcpy(context_node + static_cast<size_t>(b) * N, stands_for, sizeof(int32_t) * N);
    }
    return MPV_OK;
}

int mpv_verify_merged(const mpv_problem* problem, const int32_t* merged_parent, const int32_t* context_node,
                      const mpv_buffers* buf, void* workspace, size_t workspace_bytes, void* hip_stream) {
    if (!problem || !buf) return MPV_ERR_NULL;
    if (problem->B < 0 || problem->N < 1 || problem->V < 1) return MPV_ERR_BAD_SHAPE;
    if (problem->B == 0) return MPV_OK;
    if (!merged_parent) return MPV_ERR_NULL;
    if (problem->method == MPV_METHOD_SPECTR && !context_node) return MPV_ERR_NULL;
    if (problem->method != MPV_METHOD_SPECTR) context_node = nullptr;      // the other rules never accept a repeat
    const int32_t B = problem->B, N = problem->N;
    // first pass: every run of equal shapes is a valid problem, and the workspace holds the largest
    // (its size depends on the number of trees and of nodes only, and grows with both)
    mpv_problem run = *problem;
    int rc = MPV_OK;
    int64_t runs = 0;
    mpv::TreeScan scan;
    mpv::for_each_run(merged_parent, B, N, [&](int32_t b0, int32_t b1) {
        run.B = b1 - b0;
        run.parent = merged_parent + static_cast<size_t>(b0) * N;
        if (runs++ == 0) {                             // the sizes are the same for all: checked once
            mpv::Plan plan;
            rc = mpv::validate(&run, &plan);
        } else {
            rc = static_cast<int64_t>(run.B) * (N + 2) > (1ll << 30) ? MPV_ERR_UNSUPPORTED
                                                                      : mpv::scan_tree(run.parent, N, run.max_depth, &scan);
        }
        return rc == MPV_OK;
    });
    if (rc != MPV_OK) return rc;
    run.B = B;
    run.parent = merged_parent;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < mpv::carve(&run, nullptr, nullptr))
        return MPV_ERR_WORKSPACE;
    if ((reinterpret_cast<uintptr_t>(buf->target_logits) & 15u) || (reinterpret_cast<uintptr_t>(buf->draft_logits) & 15u))
        return MPV_ERR_ALIGNMENT;
    // One launch for the whole batch, every tree with its own tables.  Per-node outputs want every node's
    // task, which the top-down rules queue up front by node number: there (and beyond what one launch can
    // number) each run of equal shapes is a launch of its own.
    if (runs > 1 && only_what_is_needed(problem, buf) && static_cast<int64_t>(B) * (N + 2) <= (1ll << 30))
        return verify_with_workspace(&run, buf, workspace, workspace_bytes, hip_stream, false, false, context_node, merged_parent);
    const size_t elem = problem->logit_dtype == MPV_DTYPE_F32 ? 4 : 2;
    const size_t V = static_cast<size_t>(problem->V), D = static_cast<size_t>(problem->max_depth);
    auto moved = [](const void* p, size_t bytes) -> const void* { return p ? static_cast<const char*>(p) + bytes : nullptr; };
    auto moved_out = [](void* p, size_t bytes) -> void* { return p ? static_cast<char*>(p) + bytes : nullptr; };
    bool first = true;
    mpv::for_each_run(merged_parent, B, N, [&](int32_t b0, int32_t b1) {
        run.B = b1 - b0;
        run.parent = merged_parent + static_cast<size_t>(b0) * N;
        const size_t t = static_cast<size_t>(b0), tn = t * N;
        mpv_buffers part = *buf;
        part.target_logits = moved(buf->target_logits, tn * V * elem);
        part.draft_logits = moved(buf->draft_logits, tn * V * elem);
        part.tokens = static_cast<const int32_t*>(moved(buf->tokens, tn * 4));
        part.uniforms = static_cast<const float*>(moved(buf->uniforms, tn * 4));
        part.draw_uniforms = static_cast<const float*>(moved(buf->draw_uniforms, tn * 4));
        part.accept_len = static_cast<int32_t*>(moved_out(buf->accept_len, t * 4));
        part.path_nodes = static_cast<int32_t*>(moved_out(buf->path_nodes, t * D * 4));
        part.path_tokens = static_cast<int32_t*>(moved_out(buf->path_tokens, t * D * 4));
        part.bonus_token = static_cast<int32_t*>(moved_out(buf->bonus_token, t * 4));
        part.stats = static_cast<float*>(moved_out(buf->stats, tn * 4 * 4));
        part.edge_probs = static_cast<float*>(moved_out(buf->edge_probs, tn * 2 * 4));
        part.accept_prob = static_cast<float*>(moved_out(buf->accept_prob, tn * 4));
        part.final_residual = static_cast<float*>(moved_out(buf->final_residual, t * V * 4));
        rc = verify_with_workspace(&run, &part, workspace, workspace_bytes, hip_stream, true, !first,
                                   context_node ? context_node + tn : nullptr);
        first = false;
        return rc == MPV_OK;
    });
    return rc;
}

// part_of_batch, keep_counters: as for verify_with_workspace
static int block_efficiency_with_workspace(const mpv_problem* problem, const void* target_logits, const void* draft_logits,
                                           const int32_t* tokens, void* workspace, size_t workspace_bytes,
                                           float* reach_prob, float* expected, uint32_t* counters, void* hip_stream,
                                           bool part_of_batch, bool keep_counters, const int32_t* context_node = nullptr) {
    mpv::Plan plan;
    const int rc = mpv::validate(problem, &plan);
    if (rc != MPV_OK) return rc;
    if (problem->B == 0) return MPV_OK;
    if (!target_logits || !draft_logits || !tokens || !expected || !counters) return MPV_ERR_NULL;
    if (!part_of_batch && ((reinterpret_cast<uintptr_t>(target_logits) & 15u) || (reinterpret_cast<uintptr_t>(draft_logits) & 15u)))
        return MPV_ERR_ALIGNMENT;
    if (((reinterpret_cast<uintptr_t>(target_logits) ^ reinterpret_cast<uintptr_t>(draft_logits)) & 15u) != 0)
        return MPV_ERR_ALIGNMENT;
    const size_t need = mpv::carve(problem, nullptr, nullptr);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < need) return MPV_ERR_WORKSPACE;

    mpv::Workspace ws;
    mpv::carve(problem, workspace, &ws);
    mpv::Args a;
    a.zt = target_logits; a.zd = draft_logits; a.tokens = tokens;
    a.walk = problem->method == MPV_METHOD_NSS ? 1 : problem->method == MPV_METHOD_NAIVE ? 2
           : problem->method == MPV_METHOD_SPECTR ? 3 : 0;
    a.counters = counters;
    a.B = problem->B; a.N = problem->N; a.V = problem->V; a.max_depth = problem->max_depth;
    a.k32 = static_cast<float>(1.4426950408889634 / static_cast<double>(problem->temperature));
    a.lazy = 0;
    a.estimate = 1; a.reach_prob = reach_prob; a.expected = expected;
    a.keep_counters = keep_counters ? 1 : 0;
    a.context_node = context_node;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (problem->logit_dtype == MPV_DTYPE_F32) return mpv::launch_all<mpv::ElemF32>(problem, plan, ws, a, s);
    return mpv::launch_all<mpv::ElemBF16>(problem, plan, ws, a, s);
}

int mpv_block_efficiency(const mpv_problem* problem, const void* target_logits, const void* draft_logits,
                         const int32_t* tokens, void* workspace, size_t workspace_bytes,
                         float* reach_prob, float* expected, uint32_t* counters, void* hip_stream) {
    return block_efficiency_with_workspace(problem, target_logits, draft_logits, tokens, workspace, workspace_bytes,
                                           reach_prob, expected, counters, hip_stream, false, false);
}

int mpv_block_efficiency_merged(const mpv_problem* problem, const int32_t* merged_parent, const int32_t* context_node,
                                const void* target_logits, const void* draft_logits, const int32_t* tokens, void* workspace,
                                size_t workspace_bytes, float* reach_prob, float* expected, uint32_t* counters,
                                void* hip_stream) {
    if (!problem) return MPV_ERR_NULL;
    if (problem->B < 0 || problem->N < 1 || problem->V < 1) return MPV_ERR_BAD_SHAPE;
    if (problem->B == 0) return MPV_OK;
    if (!merged_parent) return MPV_ERR_NULL;
    if (problem->method == MPV_METHOD_SPECTR && !context_node) return MPV_ERR_NULL;
    if (problem->method != MPV_METHOD_SPECTR) context_node = nullptr;
    mpv_problem run = *problem;
    int rc = MPV_OK;
    mpv::for_each_run(merged_parent, problem->B, problem->N, [&](int32_t b0, int32_t b1) {
        run.B = b1 - b0;
        run.parent = merged_parent + static_cast<size_t>(b0) * problem->N;
        mpv::Plan plan;
        rc = mpv::validate(&run, &plan);
        return rc == MPV_OK;
    });
    if (rc != MPV_OK) return rc;
    run.B = problem->B;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < mpv::carve(&run, nullptr, nullptr))
        return MPV_ERR_WORKSPACE;
    if (!target_logits || !draft_logits || !tokens || !expected || !counters) return MPV_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(target_logits) & 15u) || (reinterpret_cast<uintptr_t>(draft_logits) & 15u))
        return MPV_ERR_ALIGNMENT;
    const size_t elem = problem->logit_dtype == MPV_DTYPE_F32 ? 4 : 2;
    const size_t N = static_cast<size_t>(problem->N), V = static_cast<size_t>(problem->V);
    bool first = true;
    mpv::for_each_run(merged_parent, problem->B, problem->N, [&](int32_t b0, int32_t b1) {
        run.B = b1 - b0;
        run.parent = merged_parent + static_cast<size_t>(b0) * N;
        const size_t t = static_cast<size_t>(b0), tn = t * N;
        rc = block_efficiency_with_workspace(&run, static_cast<const char*>(target_logits) + tn * V * elem,
                                             static_cast<const char*>(draft_logits) + tn * V * elem, tokens + tn,
                                             workspace, workspace_bytes, reach_prob ? reach_prob + tn : nullptr,
                                             expected + t, counters, hip_stream, true, !first,
                                             context_node ? context_node + tn : nullptr);
        first = false;
        return rc == MPV_OK;
    });
    return rc;
}


// part_of_batch, keep_counters: as for verify_with_workspace
static int acceptance_rates_with_workspace(const mpv_problem* problem, const void* target_logits, const void* draft_logits,
                                           void* workspace, size_t workspace_bytes, float* alpha, uint32_t* counters,
                                           void* hip_stream, bool part_of_batch, bool keep_counters) {
    mpv::Plan plan;
    const int rc = mpv::validate(problem, &plan);
    if (rc != MPV_OK) return rc;
    if (problem->method == MPV_METHOD_TRAVERSAL) return MPV_ERR_UNSUPPORTED;     // not an OTLP solver: App. C has no rate for it
    if (problem->B == 0) return MPV_OK;
    if (!target_logits || !draft_logits || !alpha || !counters) return MPV_ERR_NULL;
    if (!part_of_batch && ((reinterpret_cast<uintptr_t>(target_logits) & 15u) || (reinterpret_cast<uintptr_t>(draft_logits) & 15u)))
        return MPV_ERR_ALIGNMENT;
    if (((reinterpret_cast<uintptr_t>(target_logits) ^ reinterpret_cast<uintptr_t>(draft_logits)) & 15u) != 0)
        return MPV_ERR_ALIGNMENT;
    const size_t need = mpv::carve(problem, nullptr, nullptr);
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < need) return MPV_ERR_WORKSPACE;

    mpv::Workspace ws;
    mpv::carve(problem, workspace, &ws);
    mpv::Args a;
    a.zt = target_logits; a.zd = draft_logits;
    a.walk = problem->method == MPV_METHOD_NSS ? 1 : problem->method == MPV_METHOD_NAIVE ? 2
           : problem->method == MPV_METHOD_SPECTR ? 3 : 0;
    a.counters = counters;
    a.B = problem->B; a.N = problem->N; a.V = problem->V; a.max_depth = problem->max_depth;
    a.k32 = static_cast<float>(1.4426950408889634 / static_cast<double>(problem->temperature));
    a.lazy = 0;
    a.estimate = 2; a.alpha = alpha;
    a.keep_counters = keep_counters ? 1 : 0;
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    if (problem->logit_dtype == MPV_DTYPE_F32) return mpv::launch_all<mpv::ElemF32>(problem, plan, ws, a, s);
    return mpv::launch_all<mpv::ElemBF16>(problem, plan, ws, a, s);
}

int mpv_acceptance_rates(const mpv_problem* problem, const void* target_logits, const void* draft_logits,
                         void* workspace, size_t workspace_bytes, float* alpha, uint32_t* counters, void* hip_stream) {
    return acceptance_rates_with_workspace(problem, target_logits, draft_logits, workspace, workspace_bytes, alpha, counters,
                                           hip_stream, false, false);
}

int mpv_acceptance_rates_merged(const mpv_problem* problem, const int32_t* merged_parent, const void* target_logits,
                                const void* draft_logits, void* workspace, size_t workspace_bytes, float* alpha,
                                uint32_t* counters, void* hip_stream) {
    if (!problem) return MPV_ERR_NULL;
    if (problem->B < 0 || problem->N < 1 || problem->V < 1) return MPV_ERR_BAD_SHAPE;
    if (problem->method == MPV_METHOD_TRAVERSAL) return MPV_ERR_UNSUPPORTED;
    if (problem->B == 0) return MPV_OK;
    if (!merged_parent) return MPV_ERR_NULL;
    mpv_problem run = *problem;
    int rc = MPV_OK;
    mpv::for_each_run(merged_parent, problem->B, problem->N, [&](int32_t b0, int32_t b1) {
        run.B = b1 - b0;
        run.parent = merged_parent + static_cast<size_t>(b0) * problem->N;
        mpv::Plan plan;
        rc = mpv::validate(&run, &plan);
        return rc == MPV_OK;
    });
    if (rc != MPV_OK) return rc;
    run.B = problem->B;
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u) || workspace_bytes < mpv::carve(&run, nullptr, nullptr))
        return MPV_ERR_WORKSPACE;
    if (!target_logits || !draft_logits || !alpha || !counters) return MPV_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(target_logits) & 15u) || (reinterpret_cast<uintptr_t>(draft_logits) & 15u))
        return MPV_ERR_ALIGNMENT;
    const size_t elem = problem->logit_dtype == MPV_DTYPE_F32 ? 4 : 2;
    const size_t N = static_cast<size_t>(problem->N), V = static_cast<size_t>(problem->V);
    bool first = true;
    mpv::for_each_run(merged_parent, problem->B, problem->N, [&](int32_t b0, int32_t b1) {
        run.B = b1 - b0;
        run.parent = merged_parent + static_cast<size_t>(b0) * N;
        const size_t tn = static_cast<size_t>(b0) * N;
        rc = acceptance_rates_with_workspace(&run, static_cast<const char*>(target_logits) + tn * V * elem,
                                             static_cast<const char*>(draft_logits) + tn * V * elem, workspace,
                                             workspace_bytes, alpha + tn, counters, hip_stream, true, !first);
        first = false;
        return rc == MPV_OK;
    });
    return rc;
}

int mpv_timing_enable(int32_t max_launches) {
    mpv::LaunchTimer& t = mpv::g_timer;
    for (int i = 0; i < t.capacity; ++i) {
        (void)hipEventDestroy(t.start[i]);
        (void)hipEventDestroy(t.stop[i]);
    }
    delete[] t.start; delete[] t.stop; delete[] t.kernel;
    t = mpv::LaunchTimer();
    if (max_launches <= 0) return MPV_OK;
    t.start = new hipEvent_t[max_launches];
    t.stop = new hipEvent_t[max_launches];
    t.kernel = new int32_t[max_launches];
    for (int i = 0; i < max_launches; ++i) {
        if (!mpv::hip_ok(hipEventCreate(&t.start[i])) || !mpv::hip_ok(hipEventCreate(&t.stop[i]))) {
            t.capacity = i;
            mpv_timing_enable(0);
            return MPV_ERR_HIP;
        }
        t.capacity = i + 1;
    }
    t.enabled = true;
    return MPV_OK;
}

int mpv_timing_read(float* ms_out, int32_t* kernel_out, int32_t capacity, int32_t* count) {
    if (!count) return MPV_ERR_NULL;
    mpv::LaunchTimer& t = mpv::g_timer;
    const int n = t.used < capacity ? t.used : capacity;
    if (n > 0 && (!ms_out || !kernel_out)) return MPV_ERR_NULL;
    for (int i = 0; i < n; ++i) {
        float ms = 0.f;
        if (!mpv::hip_ok(hipEventElapsedTime(&ms, t.start[i], t.stop[i]))) return MPV_ERR_HIP;
        ms_out[i] = ms;
        kernel_out[i] = t.kernel[i];
    }
    *count = n;
    t.used = 0;
    return MPV_OK;
}

int mpv_row_stats(const void* logits, int32_t logit_dtype, int64_t rows, int32_t V, float temperature,
                  float* out, void* hip_stream) {
    if (!logits || !out) return MPV_ERR_NULL;
    if (rows < 0 || V < 1 || rows > 0x7fffffffLL) return MPV_ERR_BAD_SHAPE;
    if (V > MPV_MAX_VOCAB) return MPV_ERR_UNSUPPORTED;
    if (!(temperature > 0.0f) || !isfinite(temperature)) return MPV_ERR_BAD_TEMPERATURE;
    if (logit_dtype != MPV_DTYPE_F32 && logit_dtype != MPV_DTYPE_BF16) return MPV_ERR_BAD_DTYPE;
    if (rows == 0) return MPV_OK;
    const float k32 = static_cast<float>(1.4426950408889634 / static_cast<double>(temperature));
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    (void)hipGetLastError();
    if (logit_dtype == MPV_DTYPE_F32)
        hipLaunchKernelGGL((mpv::row_stats_kernel<mpv::ElemF32>), dim3(static_cast<unsigned>(rows)), dim3(mpv::kTaskBlock), 0, s,
                           static_cast<const float*>(logits), rows, V, k32, out);
    else
        hipLaunchKernelGGL((mpv::row_stats_kernel<mpv::ElemBF16>), dim3(static_cast<unsigned>(rows)), dim3(mpv::kTaskBlock), 0, s,
                           static_cast<const uint16_t*>(logits), rows, V, k32, out);
    return mpv::hip_ok(hipGetLastError()) ? MPV_OK : MPV_ERR_HIP;
}

int mpv_nucleus_mask(const void* logits, void* out, int32_t logit_dtype, int64_t rows, int32_t V,
                     float temperature, float top_p, float* threshold_out, int32_t* kept_out, void* hip_stream) {
    if (rows < 0 || V < 1) return MPV_ERR_BAD_SHAPE;
    if (V > MPV_MAX_VOCAB || rows > 0x7fffffffLL) return MPV_ERR_UNSUPPORTED;
    if (logit_dtype != MPV_DTYPE_F32 && logit_dtype != MPV_DTYPE_BF16) return MPV_ERR_BAD_DTYPE;
    if (!(temperature > 0.0f) || !isfinite(temperature)) return MPV_ERR_BAD_TEMPERATURE;
    if (!(top_p > 0.0f) || !(top_p <= 1.0f)) return MPV_ERR_BAD_TOP_P;
    if (rows == 0) return MPV_OK;
    if (!logits || !out) return MPV_ERR_NULL;
    if ((reinterpret_cast<uintptr_t>(logits) & 15u) || (reinterpret_cast<uintptr_t>(out) & 15u)) return MPV_ERR_ALIGNMENT;
    const float k32 = static_cast<float>(1.4426950408889634 / static_cast<double>(temperature));
    hipStream_t s = static_cast<hipStream_t>(hip_stream);
    (void)hipGetLastError();
    // top_p = 1 keeps every token: a threshold no mass can miss
    const float p = top_p < 1.0f ? top_p : 0.0f;
    if (logit_dtype == MPV_DTYPE_F32)
        mpv::launch_nucleus<mpv::ElemF32>(static_cast<const float*>(logits), static_cast<float*>(out), rows, V, k32, p,
                                          top_p < 1.0f ? 0 : 1, threshold_out, kept_out, s);
    else
        mpv::launch_nucleus<mpv::ElemBF16>(static_cast<const uint16_t*>(logits), static_cast<uint16_t*>(out), rows, V, k32, p,
                                           top_p < 1.0f ? 0 : 1, threshold_out, kept_out, s);
    return mpv::hip_ok(hipGetLastError()) ? MPV_OK : MPV_ERR_HIP;
}

int mpv_fill_uniforms(uint64_t seed, int64_t count, float* d_u, void* hip_stream) {
    if (count < 0) return MPV_ERR_BAD_SHAPE;
    if (count == 0) return MPV_OK;
    if (!d_u) return MPV_ERR_NULL;
    const int threads = 256;
    const int64_t blocks = (count + threads - 1) / threads;
    if (blocks > 0x7fffffffLL) return MPV_ERR_UNSUPPORTED;
    (void)hipGetLastError();
    hipLaunchKernelGGL(mpv::fill_uniforms_kernel, dim3(static_cast<unsigned>(blocks)), dim3(threads), 0,
                       static_cast<hipStream_t>(hip_stream), seed, count, d_u);
    return mpv::hip_ok(hipGetLastError()) ? MPV_OK : MPV_ERR_HIP;
}

}  // extern "C"
