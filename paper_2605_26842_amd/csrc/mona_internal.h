// Internal descriptors shared between the host planner and the HIP kernels of libmona.
// Nothing here is part of the public ABI (see include/mona.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdint.h>

namespace mona {

typedef __bf16 bf16_t;

// Static per-matrix description, uploaded once when the state is built.
struct MatStatic {
  void* g_prev;        // G_{k-1}, state dtype (NULL in the one-buffer form and when the caller keeps it)
  void* acc;           // A_k (or, in the one-buffer form, C_{k+1}), state dtype
  float* mom;          // M_k, fp32
  void* x;             // where the Newton-Schulz input (M_k, unscaled) is written: bf16 or fp32
  int32_t m, n;        // shape
  int32_t ldx;         // leading dimension of x (>= n)
  int32_t w_dtype, g_dtype;
  int32_t first_block; // first block of the elementwise grid that belongs to this matrix
  int32_t num_blocks;  // number of such blocks
  int32_t x_f32;       // 1: x (and the whole Newton-Schulz workspace of this matrix) is fp32, else bf16
};

// Per-step pointers (the caller may pass fresh buffers every step).
struct MatDynamic {
  void* w;
  const void* g;
  void* slot;          // caller-kept G_{k-1} (streaming variant), else NULL
};

// Result of the per-matrix Frobenius norm (Sec. 3.2, X_0 = M / ||M||_F).
struct MatScale {
  float inv;        // 1 / (||M||_F + eps) for the working copy as it stands (see xexp), 0 when the
                    // denominator is 0 or not finite
  float inv2;       // inv * inv
  float norm;       // ||M||_F
  uint32_t status;  // MONA_STATUS_* bits
  int32_t xexp;     // the working copy holds M 2^xexp (0 unless the norm left the safe window)
  // of the launch that begins a small step, 0 outside of it (begin_norm_finalize_kernel): workgroups that have finished their part of the
  // matrix and those of them that stay; what the last of them found; pieces of a repair that were drawn and those who have left
  uint32_t arrived, verdict, shares;
};

// One entry per block of the elementwise grid.
struct BlockWork {
  int32_t mat;    // matrix index
  int32_t chunk;  // chunk index inside that matrix
};

constexpr int kEwThreads = 256;
constexpr int kEwChunk = 4096;  // elements per block of the elementwise kernel

// ---- Newton-Schulz product kernels -------------------------------------------------
// How the update of large tiles may take the parameters of a group, 8 values of a row at a time: all of them bf16 and rows a multiple of 8, all
// bf16, or any.
enum UpdateRows : int32_t { ROWS_WHOLE = 0, ROWS_BF16 = 1, ROWS_ANY = 2 };

// out = post * (beta * E + alpha * (P Q^T)) + diag * I,   P: M x K,  Q: N x K  (logical shapes)
// An operand flagged "transposed" is stored K-major (K x M or K x N, rows of length ld).
enum GemmEpilogue : int32_t {
  EPI_STORE = 0,   // store `out`
  EPI_UPDATE = 1,  // `out` is O_k: apply W <- (1 - eta lambda) W - eta gamma O, optionally store O
};

enum PostScale : int32_t { POST_NONE = 0, POST_INV = 1, POST_INV2 = 2 };

struct GemmArgs {
  const void* P; const void* Q; const void* E; void* C;
  int64_t strideP, strideQ, strideE, strideC;  // elements between consecutive matrices of the group
  int32_t ldp, ldq, lde, ldc;
  int32_t K;                // padded, a multiple of 128
  int32_t k_real;           // without padding
  int32_t tile_m, tile_n;   // BM, BN of the kernel that will run
  int32_t trans_p, trans_q; // 1: the operand is stored K-major
  int32_t tiles_m, tiles_n; // tiles that hold rows or columns of the result; tiles of padding alone are left out
  int32_t tiles_per_mat;    // tiles_m * tiles_n, or the triangle count when symmetric
  int32_t count;            // matrices in the group
  int32_t symmetric;        // 1: only tiles with tj >= ti are computed, the result is mirrored
  float alpha, beta;
  float diag;               // added to the main diagonal of the result (symmetric products only)
  int32_t diag_n;           // rows of the result without padding: small tiles add diag to these only
  int32_t post;             // PostScale, indexed through `members`
  int32_t epilogue;         // GemmEpilogue
  int32_t store_out;        // EPI_UPDATE: also store O
  int32_t w_rows;           // EPI_UPDATE: UpdateRows
  const int32_t* members;   // group member -> matrix index
  const MatScale* scales;   // per matrix
  const MatStatic* stat;    // per matrix (EPI_UPDATE: real m, n, w dtype)
  const MatDynamic* dyn;    // per matrix (EPI_UPDATE: w pointer)
  float w_keep;             // 1 - eta * lambda
  float o_scale;            // eta * gamma
};

// ---- products, compactly ------------------------------------------------------------------
// What all products of a shape group share, and what those of a step share; with an op code they say all that GemmArgs
// says (expand_op, on the host for a launch, on the device for the kernel that runs a whole chain of products).
struct GroupDesc {
  char* x;                  // ping-pong buffer 0 of X; buffer 1 is x_step bytes on
  char* pp;                 // p x p matrix 0; the others every pp_step bytes
  int64_t x_step, pp_step;
  char* fresh;              // products with a buffer each: S_0, B_0, S_1, .. of kFreshSteps iterations every pp_step bytes, then X_1, ..
                            // every x_step bytes
  const int32_t* members;   // group member -> matrix index
  int32_t count, m, n;      // matrices, their shape
  int32_t rows_pad, cols_pad;
  int32_t tall, f32;
  int32_t w_rows;           // UpdateRows
  float o_scale;            // eta * gamma
};
struct StepDesc {
  const MatScale* scales;
  const MatStatic* stat;
  const MatDynamic* dyn;
  float ns_a, ns_b, ns_c;
  float w_keep;             // 1 - eta * lambda
};

enum OpKind : uint32_t { OP_GRAM = 0, OP_POLY = 1, OP_APPLY = 2, OP_SYMPROD = 3 };
// Fields of an op code (bit offsets).  P, Q, C: numbers of p x p matrices; SRC: the ping-pong buffer an X operand is in.
enum OpField : uint32_t {
  OPF_KIND = 0, OPF_P = 2, OPF_Q = 5, OPF_C = 8, OPF_SRC = 11,
  OPF_E = 12,       // apply: adds a X
  OPF_DIAG = 13,    // poly: adds a I
  OPF_FIRST = 14,   // the first product that reads the unscaled working copy: carries the scale
  OPF_LAST = 15,    // apply: carries the parameter update
  OPF_STORE = 16,   // (with LAST) also stores O
  OPF_TP = 17, OPF_TQ = 18,   // the operand is read K-major
  OPF_TILE = 19,    // 0: 32 x 32, 1: 64 x 64, 2: 128 x 128, 3: 256 x 256
  OPF_FRESH = 21,   // t + 1 in iteration t of a literal schedule whose products have a buffer each (0: none such)
};
constexpr int kFreshSteps = 5;   // iterations that the workspace of small steps has such buffers for
__host__ __device__ inline uint32_t op_field(uint32_t code, uint32_t at, uint32_t mask = 1u) { return (code >> at) & mask; }

__host__ __device__ inline void expand_op(const StepDesc& st, const GroupDesc& g, uint32_t code, GemmArgs& a) {
  const uint32_t kind = op_field(code, OPF_KIND, 3u), src = op_field(code, OPF_SRC);
  const int32_t p_pad = g.tall ? g.cols_pad : g.rows_pad, p_real = g.m < g.n ? g.m : g.n;
  const int64_t x_stride = (int64_t)g.rows_pad * g.cols_pad, s_stride = (int64_t)p_pad * p_pad;
  const int32_t fresh = (int32_t)op_field(code, OPF_FRESH, 7u);
  char* const pps = fresh ? g.fresh + 2 * (fresh - 1) * g.pp_step : g.pp;
  auto fresh_x = [&](int32_t t) { return g.fresh + 2 * kFreshSteps * g.pp_step + (t - 1) * g.x_step; };   // X_t, t > 0
  char* const xs = fresh > 1 ? fresh_x(fresh - 1) : g.x + (src && !fresh ? g.x_step : 0);
  auto pp = [&](uint32_t at) { return pps + (int64_t)op_field(code, at, 7u) * g.pp_step; };
  const bool apply = kind == OP_APPLY, last = op_field(code, OPF_LAST), first = op_field(code, OPF_FIRST);
  a.count = g.count;
  a.members = g.members; a.scales = st.scales; a.stat = st.stat; a.dyn = st.dyn;
  a.symmetric = apply ? 0 : 1;
  a.trans_p = (int32_t)op_field(code, OPF_TP); a.trans_q = (int32_t)op_field(code, OPF_TQ);
  a.alpha = 1.0f; a.beta = 0.0f; a.diag = 0.0f; a.diag_n = p_real;
  a.post = POST_NONE; a.epilogue = EPI_STORE; a.store_out = 0; a.w_rows = g.w_rows;
  a.w_keep = st.w_keep; a.o_scale = g.o_scale;
  // operands: the p x p matrices numbered by the code, an X operand in place of one or both
  a.P = pp(OPF_P); a.Q = pp(OPF_Q); a.C = pp(OPF_C); a.E = nullptr;
  a.strideP = a.strideQ = a.strideE = a.strideC = s_stride;
  a.ldp = a.ldq = a.lde = a.ldc = p_pad;
  a.K = p_pad; a.k_real = p_real;
  if (kind == OP_GRAM) {                        // S = X X^T (tall: X^T X)
    a.P = a.Q = xs; a.strideP = a.strideQ = x_stride; a.ldp = a.ldq = g.cols_pad;
    a.K = g.tall ? g.rows_pad : g.cols_pad;
    a.k_real = g.tall ? g.m : g.n;
    if (first) a.post = POST_INV2;
  } else if (kind == OP_POLY) {                 // b S + c S S (+ a I)
    a.E = a.P;
    a.alpha = st.ns_c; a.beta = st.ns_b;
    if (op_field(code, OPF_DIAG)) a.diag = st.ns_a;
  } else if (apply) {                           // a X + B X (tall: a X + X B), or B X alone
    if (g.tall) { a.P = xs; a.strideP = x_stride; a.ldp = g.cols_pad; }
    else        { a.Q = xs; a.strideQ = x_stride; a.ldq = g.cols_pad; }
    a.C = fresh && !last ? fresh_x(fresh) : g.x + (src && !fresh ? 0 : g.x_step);
    a.strideE = a.strideC = x_stride;
    a.lde = a.ldc = g.cols_pad;
    if (op_field(code, OPF_E)) { a.E = xs; a.beta = st.ns_a; }
    if (first) a.post = POST_INV;
    if (last) { a.epilogue = EPI_UPDATE; a.store_out = (int32_t)op_field(code, OPF_STORE); }
  }
  // Tiles that hold nothing but padding are left out where the padding is wider than a tile: all of it is zero, in every
  // buffer of a group that runs small tiles (the large tiles of a group cover its padding in every product).
  const int32_t shift = 5 + (int32_t)op_field(code, OPF_TILE, 3u), tile = 1 << shift;
  const int32_t rm = apply ? g.m : p_real, rn = apply ? g.n : p_real;
  a.tile_m = a.tile_n = tile;
  a.tiles_m = (rm + tile - 1) >> shift;
  a.tiles_n = (rn + tile - 1) >> shift;
  a.tiles_per_mat = a.symmetric ? a.tiles_n * (a.tiles_n + 1) / 2 : a.tiles_m * a.tiles_n;
}

// One launch of the small-tile kernels: the products that several shape groups run at the same position of their
// chains (passed by value: nothing is copied from the host).
constexpr int kMaxMerged = 8;
struct GemmBatch {
  int32_t n;                        // products in the batch
  int32_t slot_end[kMaxMerged];     // workgroups per die up to and including product g (filled at launch)
  GemmArgs a[kMaxMerged];
};

// All products of a step of up to kMaxMerged shape groups as one launch (ns_chain_kernel), passed by value.
constexpr int kMaxChainOps = 180, kMaxChainTasks = 11264;   // (tasks: of all chains of a step)
struct ChainOp {
  int32_t end;             // tasks (tiles) up to and including this product
  int32_t before;          // first task of the same group's product before
  int32_t before_per_mat;  // tiles a matrix has there (0: none)
  uint32_t code;           // op code; the group in the bits from OPF_GROUP on
};
constexpr uint32_t OPF_GROUP = 24;
constexpr uint32_t kStatusIncomplete = 8u;           // MONA_STATUS_INCOMPLETE
constexpr int kRollPolls = 64;                       // about 50 us
constexpr int kPatience = 1 << 20;                   // polls of one wait in a chain: about a second
// Shared by the workgroups of a chain launch; zero when it starts.
struct ChainRoll {
  uint32_t reported;       // workgroups that have reported, and whether the roll is closed
  uint32_t pad[31];
  uint32_t workgroups;     // those that had reported, once it is closed
  uint32_t drawn;          // tasks drawn from then on, where it was closed without some
  uint32_t spoiled;        // (first roll, before the chain) a workgroup of the pass has found a chunk that is out of range by itself
  uint32_t pad2[29];
};
struct ChainArgs {
  StepDesc step;
  ChainRoll* roll;
  uint32_t* flags;         // one for each task; zero when the launch starts
  int32_t ops, tasks;
  int32_t roll_polls;      // polls of the roll before it is closed without some
  int32_t patience;        // polls of one wait
  int32_t fresh;           // every product has a buffer of its own, filled beforehand (FillArgs): no flags are needed
  GroupDesc group[kMaxMerged];
  ChainOp op[kMaxChainOps + 3];   // (looked through four at a time; those behind the last one end nowhere)
};
static_assert(sizeof(ChainArgs) <= 4000, "an argument block holds 4 KB");
// What every step clears before its products: the rolls and the flags of its chain launches, one after the other.
constexpr int kMaxChains = 4;
constexpr size_t kChainBytes = kMaxChains * sizeof(ChainRoll) + kMaxChainTasks * sizeof(uint32_t);

// What the buffers of fresh chains are filled with before the products: no result holds it (a store turns it into another NaN), so
// a reader sees of each value whether it has been written.  The tiles of a chain read and write whole multiples of 32 or 64; of these
// the ones behind the next multiple of 32 are filled with the zeros of padding.
constexpr uint32_t kUnwritten = 0xffffffffu;
constexpr int kFillPieces = 1024;
struct FillItem {
  char* at;                // buffers of equal shape
  uint32_t end;            // workgroups (of kFillPieces pieces of 16 bytes each) up to and including this item
  uint32_t pieces;         // of this item
  uint32_t rows, pitch;    // of a buffer: rows to fill, bytes from one to the next
  uint32_t cover_rows, cover;   // rows, pieces of a row that results will stand in
  uint32_t width;          // pieces of a row to fill
  uint32_t stride;         // bytes from one buffer to the next
};
struct FillArgs {
  int32_t n, groups;       // items, workgroups
  FillItem item[2 * kMaxMerged * kMaxChains];
};
static_assert(2 * kMaxMerged * kMaxChains <= 64, "a lane for each item");

// One launch of the kernel that takes a whole matrix through all its iterations in one workgroup.
struct MatrixBatch {
  StepDesc step;
  int32_t n, steps, store_o;
  int32_t end[kMaxMerged];          // matrices up to and including group i
  GroupDesc group[kMaxMerged];
};

constexpr int kXcds = 8;   // MI355X: 8 accelerator dies, workgroups are dealt to them round-robin
// workgroups per die of a launch of small tiles
inline long long slots_per_die(const GemmArgs& a) { return ((long long)a.tiles_per_mat * a.count + kXcds - 1) / kXcds; }

// records the text mona_last_error() returns (thread-local) and hands `code` back
int api_fail(int code, const char* fmt, va_list ap);

// The pointers of a short list, passed by value: 96 entries are 2.3 KB of the 4 KB an argument block may hold.
constexpr int kInlineMats = 96;
struct DynTable {
  MatDynamic v[kInlineMats];
};

// the same for the launch that begins a small step; n = 0: the table in memory holds them
constexpr int kBeginMats = 32;
constexpr int kBeginBlocks = 8192;   // blocks of one matrix that MatScale counts in 16 bits (a chain has no room for so many)
struct BeginTable {
  int32_t n;
  MatDynamic v[kBeginMats];
};
static_assert(sizeof(FillArgs) + sizeof(BeginTable) + 128 <= 4000, "an argument block holds 4 KB");

constexpr int kMaxDevices = 64;      // device ordinals that static arrays are looked up for
// a part of the pool of chain buffers on `device`, the current one (chain_pool.hip; nullptr: no room), and back again
char* take_from_pool(int device, size_t bytes);
void give_back(int device, const char* at, size_t bytes);

// kernels (defined in the .hip files)
// dyn[0 .. n) = t.v[0 .. n), n <= kInlineMats
hipError_t launch_write_dyn(const DynTable& t, int n, MatDynamic* dyn, hipStream_t s);
hipError_t launch_state_update(const MatStatic* stat, const MatDynamic* dyn, const BlockWork* work,
                               double* partials, int num_blocks, int g_bf16, int state_bf16, int one_buffer,
                               float mu, float beta_a, float alpha, int use_prev, int keep, hipStream_t s);
// what the caches are to keep of a pass over all matrices that writes so many bytes of working copies
int choose_keep(double copy_bytes);
// norms, scales and the repair of flagged working copies
// `list` (DEVICE, may be NULL = matrices 0 .. count - 1): the matrix indices to finalise; max_blocks: the most
// elementwise blocks any of them has; zero: memory to clear on the way (a multiple of 16 bytes); fill: buffers of fresh
// chains to fill, or NULL
hipError_t launch_norm_finalize(const MatStatic* stat, const double* partials, MatScale* scales,
                                const int32_t* list, int count, int max_blocks, float eps, void* zero, size_t zero_bytes,
                                const FillArgs* fill, hipStream_t s);
// the elementwise pass of matrices of any gradient dtype with what launch_write_dyn and launch_norm_finalize do, as one launch; the
// matrices are few and small (`partials` in the order of `work`, all of a matrix's blocks in it)
hipError_t launch_begin(const MatStatic* stat, const BlockWork* work, MatScale* scales, double* partials, MatDynamic* dyn, int num_blocks,
                        int state_bf16, int one_buffer, float mu, float beta_a, float alpha, int use_prev, float eps, void* zero,
                        size_t zero_bytes, const FillArgs& fill, const BeginTable& table, hipStream_t s);
// a one-matrix state prepared by one kernel from its arguments (no host copy): tables, scale, cleared workspace
hipError_t launch_single_prepare(const MatStatic& ms, const MatDynamic& md, void* o_ptr, MatStatic* stat,
                                 MatDynamic* dyn, void** o_ptrs, BlockWork* work, int num_blocks, int32_t* members,
                                 int32_t* order, MatScale* scale, void* zero, size_t zero_bytes, hipStream_t s);
hipError_t launch_plain_update(const MatStatic* stat, const MatDynamic* dyn, const MatScale* scales,
                               const BlockWork* work, int num_blocks, void* const* o_ptrs, float lr, float wd,
                               float gamma_coeff, int store_o, hipStream_t s);
// cu_cap > 0: the persistent large-tile kernel uses at most that many CUs (the rest are busy elsewhere)
hipError_t launch_ns_gemm(const GemmArgs& a, int cu_cap, hipStream_t s);   // 256 x 256 tiles, bf16
// 64 x 64 or 128 x 128 tiles; wide: eight wavefronts a tile and one workgroup per CU instead of four and two
hipError_t launch_ns_small(GemmBatch& b, bool f32, bool wide, hipStream_t s);
// fp32 products as bf16 ones, 64 x 64 or 128 x 128 tiles
hipError_t launch_ns_split(GemmBatch& b, hipStream_t s);
// all iterations of groups of bf16 matrices with a padded short side of 128 or 256, one workgroup per matrix
hipError_t launch_ns_matrix(const MatrixBatch& b, hipStream_t s);
// a whole chain of products on small tiles; `wgs` workgroups
hipError_t launch_ns_chain(const ChainArgs& c, int wgs, hipStream_t s);
int device_cu_count();
bool device_is_gfx950();   // the current device
hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t s);

}  // namespace mona
