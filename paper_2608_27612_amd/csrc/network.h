// Arguments of the network kernels (network.hip), shared with their host driver (networks.cpp).
//
// Numbering. Before pruning, genome g has raw nodes 0 .. n_sub - 1 (its substrate sources, in
// substrate order) and n_sub + i for the i-th set bit of its hidden-cell bitmap (ascending grid
// position); raw node j of genome g is entry raw_node[g] + j of the per-node arrays. Its raw edges
// (one per expressed connection of every phase, genome by genome, each genome's phases in order,
// each phase's pairs in order, each pair's connections in cell order) are entries
// raw_edge[g] .. raw_edge[g + 1] - 1 of eu/ev/ew, holding global raw node numbers raw_node[g] + j
// (kNoNode: the grid end is not a hidden node, the edge is dropped). After pruning, the kept nodes
// of genome g are renumbered in raw order (substrate nodes first, all kept) as entries
// node_offset[g] + k of the network arrays, and the kept edges are grouped by destination (CSR,
// in_offset), each group in raw order.
#pragma once
#include <stdint.h>

namespace emr {

constexpr uint32_t kNoNode = 0xFFFFFFFFu;
constexpr int kNetThreads = 256;

// Error bits of the network kernels.
constexpr uint32_t kNetErrIndex = 1u;   // an index outside its table (a host bug; never expected)

struct NetRankArgs {
  const uint32_t* known;  // [n_genomes * words] hidden-cell bitmaps
  uint32_t* rank;         // [n_genomes * words] set bits of the genome's earlier words
  uint32_t* hidden;       // [n_genomes] set bits per genome
  int64_t words;
  uint32_t n_genomes;
};

// One pair of a phase, for the edges of its connections: entry o of the raw edges is connection
// o - delta, between raw node `node` (its source's, global; kNoNode: an internal error) and the
// connection's grid cell in genome g.
struct NetPair {
  int64_t delta;
  int64_t lo, hi;  // the genome's raw edges
  uint32_t g_dir;  // genome << 1 | direction (0: node -> cell, 1: cell -> node)
  uint32_t node;
  uint32_t base, n;  // the genome's raw nodes
};

constexpr int kNetMaxPhases = 65;  // the substrate's and one per hidden-to-hidden iteration

// Raw edges genome by genome: one workgroup turns the phases' connection counts per genome into
// raw_edge and each phase's seg, and the hidden counts into raw_node.
struct NetLayoutArgs {
  const uint32_t* hidden;               // [n_genomes]
  // phase k: its connections' offsets per pair and genome g's pairs src_offsets[g] ..
  // src_offsets[g + 1] - 1 (NULL: g * n_sub ..)
  const int64_t* const* conn_offset;    // [n_phases]
  const int64_t* const* src_offsets;    // [n_phases]
  int64_t* seg;                         // [n_phases * n_genomes] raw edge index of g's first edge
  int64_t* raw_edge;                    // [n_genomes + 1]
  int64_t* raw_node;                    // [n_genomes + 1]
  int64_t n_raw, e_raw;                 // what the host expects the totals to be
  uint32_t n_phases;
  uint32_t n_sub;
  uint32_t n_genomes;
  uint32_t* err;
};

struct NetEdgeArgs {
  // one phase's expressed connections (CSR over its pairs)
  const int64_t* conn_offset;  // [n_pairs + 1]
  const uint32_t* conn_cell;
  const float* conn_w;
  int64_t n_pairs;
  int64_t total;               // conn_offset[n_pairs]
  // the phase's pairs: shared substrate sources (src_offsets == NULL: pair = g * n_sub + j) or
  // per-genome hidden sources (pair = source index, genome g owns src_offsets[g] .. [g + 1] - 1,
  // source r sits at heap cell src_cell[r])
  const int64_t* src_offsets;  // [n_genomes + 1] or NULL
  const uint32_t* src_cell;    // [n_sources] or NULL
  const uint8_t* sub_dir;      // [n_sub] 0: input (outgoing queries), 1: output (incoming)
  uint32_t n_sub;
  uint32_t n_genomes;
  const uint32_t* known;
  const uint32_t* rank;
  int64_t words;
  const int64_t* seg;          // [n_genomes] raw edge index of genome g's first edge of this phase
  const int64_t* raw_edge;     // [n_genomes + 1]
  const int64_t* raw_node;     // [n_genomes + 1]
  NetPair* pairs;              // [n_pairs] (k_net_pairs writes, k_net_edges reads)
  uint32_t* eu;                // [raw edges] global raw node numbers (raw_node[g] + local)
  uint32_t* ev;
  float* ew;
  int64_t e_raw;
  uint32_t* err;
};

// Pruning. Flags per raw node (global numbering): byte 0 reachable from an input, byte 1 reaches an
// output.
struct NetFlagArgs {
  const uint8_t* sub_dir;
  const int64_t* raw_node;  // [n_genomes + 1]
  uint16_t* flags;          // [raw nodes]
  uint32_t* kept_nodes;     // [n_genomes] kept nodes, substrate nodes among them (k_net_kept)
  int64_t* node_offset;     // [n_genomes + 1] (k_net_number)
  uint32_t n_sub;
  uint32_t n_genomes;
  int64_t* total;           // node_offset[n_genomes] once more, beside the pass words
};

// Copies of the first 16-byte units of buffers to others, in one launch.
constexpr int kNetFits = 5;
struct NetFitArgs {
  const void* src[kNetFits];
  void* dst[kNetFits];
  int64_t units[kNetFits];
  uint32_t count;
};

constexpr int kNetPasses = 6;  // reach passes enqueued before the host looks at them

struct NetReachArgs {
  const uint32_t* eu;       // [raw edges] global raw node numbers, kNoNode: dropped
  const uint32_t* ev;
  uint16_t* flags;
  uint32_t* changed;        // [kNetPasses] set to 1 by a pass that changed a flag
  uint32_t pass;            // of the batch: returns at once when pass - 1 changed nothing
  int64_t edges;            // raw edges
  int64_t nodes;            // raw nodes
};

struct NetNodeArgs {
  const uint32_t* known;
  const uint32_t* rank;
  int64_t words;
  const int64_t* raw_node;
  const uint16_t* flags;
  const int32_t* in_slot;      // [n_sub] input number of a substrate node, or -1
  const int64_t* node_offset;  // [n_genomes + 1] kept nodes
  uint32_t* gid;               // [raw nodes] kept node number (global), or kNoNode
  uint32_t* node_cell;         // [nodes] heap cell, kNoNode for substrate nodes
  int32_t* node_in;            // [nodes] input number of a substrate input node, else -1
  uint32_t* err;
  uint32_t n_sub;
  uint32_t n_genomes;
};

// The kept edges grouped by destination, each group in raw order: a stable sort of the raw edges
// by their destination's kept number (dropped edges get the key `sentinel`, above every kept
// number, and sort last) that carries each edge's source and weight along.
struct NetKeyArgs {
  const uint32_t* eu;
  const uint32_t* ev;
  const float* ew;
  const uint16_t* flags;
  const uint32_t* gid;
  uint32_t* key;            // [raw edges]
  uint64_t* val;            // [raw edges] source's kept number | weight bits << 32
  int64_t edges;            // raw edges
  int64_t nodes;            // raw nodes
  uint32_t sentinel;        // kept nodes in all
  uint32_t* err;
};

struct NetSplitArgs {
  const uint32_t* key;        // sorted
  const uint64_t* val;        // sorted
  const int64_t* node_offset; // [n_genomes + 1]
  int64_t* in_offset;         // [nodes + 1]
  int64_t* summary;           // [2 (n_genomes + 1) + 1] for the host: node_offset, the genomes'
                              // first kept edges, *err
  uint32_t* in_src;           // [edges] global node number of the source
  float* in_w;                // [edges]
  int64_t raw_edges;
  int64_t raw_nodes;
  uint32_t sentinel;
  uint32_t n_genomes;
  uint32_t* err;
};

// Synchronous activation. A genome whose node states fit the LDS can run all its steps in one
// workgroup per block of 4 Q patterns (k_net_run); the others, and those for which the host estimates
// that to take longer, run one launch per step over state buffers [pblocks][nodes] of float4 (4
// patterns per block), swapped after each step.
constexpr int kNetRunThreads = 1024;          // 16 waves: two workgroups fill a CU
constexpr uint32_t kNetRunMaxQ = 4;           // float4 pattern groups of a workgroup, at most
constexpr uint32_t kNetRunLds = 160u * 1024u;
// LDS of a genome of n nodes: two state buffers of n * q float4 and n + 1 edge offsets.
inline constexpr uint32_t net_run_lds(uint32_t n, uint32_t q) { return n * (32u * q + 4u) + 4u; }
constexpr int kNetRanges = 8;                 // classes of genomes in a launch, at most
constexpr uint32_t kNetStageFloats = 256;     // patterns small enough for the kernarg

// Patterns passed by value to the device buffer the kernels read.
struct NetStageArgs {
  float* dst;
  uint32_t n;
  float v[kNetStageFloats];
};

struct NetRunArgs {
  const uint32_t* order;       // genomes
  const int64_t* node_offset;  // [n_genomes + 1]
  const int32_t* node_in;
  const int64_t* in_offset;
  const uint32_t* in_src;
  const float* in_w;
  const float* patterns;       // [n_patterns * n_inputs]
  const float* targets;        // (fitness: one output, at most 4 patterns)
  const int32_t* out_node;     // [n_outputs] substrate index of output o
  float* outputs;              // [n_genomes * n_patterns * n_outputs] or NULL
  float* fitness;              // [n_genomes] or NULL
  int64_t nodes, edges;
  uint32_t n_genomes;
  uint32_t n_inputs, n_outputs, n_patterns;
  uint32_t steps;
  uint32_t lds_bytes;          // the launch's dynamic LDS
  // class r: genomes order[first[r]] .. (count[r] of them), blocks[r] blocks of 4 q[r] patterns
  uint32_t first[kNetRanges], count[kNetRanges], blocks[kNetRanges], q[kNetRanges];
};

// The genomes of a stepwise launch: up to kNetRanges runs of `order`, or (order NULL, one run from 0)
// all of them.
struct NetList {
  const uint32_t* order;
  uint32_t first[kNetRanges];  // run r: order[first[r]] ..
  uint32_t count[kNetRanges];
  uint32_t total;              // sum of the counts
  uint32_t max_nodes;          // nodes of its largest genome
  uint32_t n_genomes;
};

struct NetStateArgs {
  NetList list;
  const int64_t* node_offset;
  const int32_t* node_in;   // [nodes]
  const float* patterns;    // [n_patterns * n_inputs], or NULL: v
  float* state;             // [pblocks * nodes * 4]
  int64_t nodes;
  uint32_t n_inputs;
  uint32_t n_patterns;
  uint32_t pblocks;
  float v[kNetStageFloats];
};

struct NetStepArgs {
  NetList list;
  const int64_t* node_offset;
  const int32_t* node_in;
  const int64_t* in_offset;
  const uint32_t* in_src;
  const float* in_w;
  const float* cur;
  float* nxt;
  int64_t nodes;
  uint32_t pblocks;
};

struct NetOutArgs {
  NetList list;
  const int64_t* node_offset;  // [n_genomes + 1]
  const int32_t* out_node;     // [n_outputs] substrate index of output o
  const float* state;          // the final state
  float target[4];             // (fitness: one output, 4 patterns)
  float* outputs;              // [n_genomes * n_patterns * n_outputs] or NULL
  float* fitness;              // [n_genomes] or NULL
  int64_t nodes;
  uint32_t n_outputs;
  uint32_t n_patterns;
};

}  // namespace emr
