// Internal definitions shared by the library's translation units.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <atomic>
#include <string>
#include <vector>

#include "../../include/rbffd.h"

#define RBFFD_MAX_STENCIL 128     // max(n, n_hv) supported
#define RBFFD_MAX_MONO 64         // monomials per local system
#define RBFFD_TILE 64             // nodes per packed tile (one wavefront)
#define RBFFD_WGT 256             // nodes per LDS-staged workgroup tile (4 wavefronts)
#define RBFFD_WGT_BATCH 128       // K-field batch: nodes per staged tile (two workgroups share a CU)
#define RBFFD_WGT_3D 512          // 3D: nodes per staged workgroup tile (8 wavefronts)
#define RBFFD_WGT_3D_F32 1024     // 3D with FP32 fields (16 wavefronts)
#define RBFFD_LDS_BUDGET 65536    // bytes of LDS one staged workgroup may use
#define RBFFD_LDS_BUDGET_3D 131072 // 3D: both operands together up to this size (one
                                   // workgroup per CU; the tuner also tries one operand
                                   // at a time, two per CU)
#define RBFFD_SMALL 65536         // node counts up to which single-field plans do not
#define RBFFD_SMALL_3D_F32 24576  // start on the staged kernels (plan.hip): FP32, BF16
#define RBFFD_SMALL_BLOCK 40000   // of these, one tile per workgroup
#define RBFFD_SMALL_2D 80000      // FP64, with at most this many weights
#define RBFFD_SMALL_3D 50000
#define RBFFD_SMALL_WEIGHTS 7000000
#define RBFFD_SMALL_2D_ANY 42000  // FP64, with any stencils
#define RBFFD_SMALL_3D_ANY 28000
// Operators (weights, positions) up to this size stay in the 256 MB memory-side
// cache between half steps, below 32 MB in the L2s, when loaded ordinarily; larger
// ones stream through it.  us per step, non-temporal / ordinary loads: 2D FP32 68k
// nodes (n 12, 19 MB) 17.1 / 11.0, 490k (n 25, 188 MB) 65.0 / 60.0, 1M (384 MB) 132 /
// 149; 2D FP64 250k (176 MB) 60.8 / 56.5, 490k (345 MB) 119 / 133; 3D FP32 125k (117
// MB) 53.6 / 46.7, 262k (245 MB) 79.6 / 74.7.  The exception: 2D operators of at most
// RBFFD_BAND_NODE bytes per node between these two sizes, too large for the L2s and
// with little to sum per byte: 160k nodes (n 25 FP32, 61 MB) 22.5 / 23.6, 123k (n 12
// FP64, 63 MB) 23.7 / 24.9, at 46 MB 20.2 / 19.8 and at 96 MB 33.1 / 32.6.
// 2D FP32, W22 and BF16 sets below RBFFD_CACHED_F32 nodes keep the streaming loads,
// though ordinary ones are faster there (90k nodes 18 to 29 us against 12.7 to 25):
// between about 40k and 110k nodes the tuner chooses between staged and small-set
// kernels (12 to 27 us), which sum in another order, and with faster staged ones
// tuned plans would move to them, their FP64 energies by 1e-8.
#define RBFFD_CACHED_BYTES ((int64_t)256 << 20)
#define RBFFD_BAND_LO ((int64_t)44 << 20)
#define RBFFD_BAND_HI ((int64_t)76 << 20)
#define RBFFD_BAND_NODE 512
#define RBFFD_CACHED_F32 120000
// Whole steps (step.hip): most tiles; how many runs of a plan have flags of their own
// (two in flight on the same flags wait for tiles whose flags the other overwrote: two
// streams on one 1M-node plan, us per step of both, 405 on shared flags, 191 on their
// own, 255 in halves); how long a workgroup waits for its neighbours' H before it
// computes it itself (ticks of 10 ns; the waits seen are below 10 us); and how many
// places ahead in the order of dispatch a tile may look: a third to a half of the
// workgroups a chip holds
#define RBFFD_STEP_TILES 16384
#define RBFFD_STEP_RUNS 64
#define RBFFD_STEP_PATIENCE 5000
#define RBFFD_STEP_AHEAD 256
#define RBFFD_KSLICE 16           // widest field slice of the staged K-field batch
#define RBFFD_LDS_BUDGET_BATCH 122880
#define RBFFD_LDS_CU 163840       // LDS of one CU (gfx950)

// ---------------------------------------------------------------------------
// Device-side layout of one operator block (the weights applied in one half
// step).  Packed arrays are "tile-sliced ELL": node i = 64 t + l lives in tile
// t, lane l; slot chunk q (4 consecutive non-self slots) of tile t occupies a
// contiguous run of 64 x 4 values, so one wavefront streams 1 KB (FP32) per
// load instruction.  Difference form: the slot whose value is used as
// reference (the node itself for collocated stencils) is not stored; since
// every weight vector sums to zero (constants are reproduced), sum_s w_s f_s
// = sum_{s != ref} w_s (f_s - f_ref).
// ---------------------------------------------------------------------------
struct OpBlock {
    int64_t Nt = 0;          // target (centre) nodes
    int64_t Ns = 0;          // source nodes
    int32_t n = 0, nh = 0;   // curl / HV stencil sizes
    int32_t ns = 0;          // union width (collocated) else 0
    bool cross = false;      // curl stencil drawn from the other set (two-set)
    int64_t tiles = 0;
    int32_t C4 = 0, V4 = 0, S4 = 0;  // slot chunks: curl, hv, union index
    // device pointers (inside the arena)
    int32_t* st_union = nullptr;   // [Nt][ns]          (collocated)
    int32_t* st_curl = nullptr;    // [Nt][n]           (two-set)
    int32_t* st_hv = nullptr;      // [Nt][nh]          (two-set)
    double* wc = nullptr;          // [Nt][dim][n]
    double* wh = nullptr;          // [Nt][nh]
    void* pidx = nullptr;          // collocated: [tiles][S4][64][4] i32 ; two-set: curl chunks
    void* pidx_h = nullptr;        // two-set: [tiles][V4][64][4] i32 hv chunks
    int32_t* pref = nullptr;       // two-set: [Nt] reference (slot 0) of the curl stencil
    void* pwc = nullptr;           // [tiles][C4][dim][64][4] weights
    void* pwh = nullptr;           // [tiles][V4][64][4] weights
    // node-major copies for the K-field batch (collocated only)
    int32_t* bidx = nullptr;       // [Nt][S4*4]
    float* bwc = nullptr;          // [Nt][dim][C4*4]
    float* bwh = nullptr;          // [Nt][V4*4]
    float* bw0 = nullptr;          // [Nt][4]: centre weights (curl x, curl y, hyperviscosity, 0)
    // LDS staging (collocated): per 256-node workgroup tile, the sorted unique
    // source nodes of all its stencils ("halo list") and, per node and slot,
    // the 16-bit position of the slot's node in that list
    uint16_t* lidx = nullptr;      // [tiles][Q8][64][8]
    uint16_t* lself = nullptr;     // [tiles * 64] each node's own position (K-field batch)
    int32_t* hpool = nullptr;      // concatenated halo lists
    int32_t* hoff = nullptr;       // [nwg + 1] start of each workgroup's list
    // whole steps (2D, single field): what each workgroup does, in order of dispatch.
    // Tiles whose halo reaches far in that order come twice: their H update first of
    // all, their E update last.  [2 nwg] (tile, kOnlyH or kOnlyE or 0, start and
    // length of the halo list), then the count of those tiles and the count of H
    // tiles that waiting workgroups computed by themselves so far
    int4* ord = nullptr;
    int32_t split = 0;             // that count on the host
    // whole steps: [RBFFD_STEP_RUNS][nwg] the run and step each tile's H is at; runs
    // of the plan take the rows in turn
    uint64_t* flags = nullptr;
    int32_t Q8 = 0;
    int64_t nwg = 0;
    int32_t wgt = RBFFD_WGT;       // nodes per staged workgroup tile (halo lists)
    int32_t hmax = 0;              // longest halo list (0 = staging unavailable)
    int32_t stage = 0;             // single field: 1 = both operands staged together,
                                   // 2 = one operand at a time (3D), 0 = none
    // transposed operator for the adjoint (collocated 2D)
    int64_t* t_off = nullptr;      // [tiles + 1] start of each tile's entries
    int32_t* t_width = nullptr;    // [tiles]
    int32_t* t_src = nullptr;      // [entries]  source row i
    int32_t* t_slot = nullptr;     // [entries]  slot s of row i (-1 = padding)
    void* t_w = nullptr;           // [entries][4] (wx, wy, wh, 0) in weight precision
    int64_t t_cap = 0;             // entry capacity
};

constexpr int32_t kOnlyH = 1, kOnlyE = 2;   // OpBlock::ord

struct NodeSet {
    int64_t N = 0;
    std::vector<double> xyz_host;
    std::vector<uint8_t> flags_host;
    double* xyz_in = nullptr;     // [N][dim] original order
    uint8_t* flags_in = nullptr;  // [N]
    int32_t* perm = nullptr;      // internal -> original
    int32_t* inv = nullptr;       // original -> internal
    double* xyz = nullptr;        // [N][dim] internal order
    uint8_t* emask = nullptr;     // [N] bit c = E component c free (E set only);
                                  // bit 3 = curved wall with a normal in nrm
    std::vector<double> nrm_host; // [N][dim] unit wall normals, original order
    double* nrm = nullptr;        // [N][dim] internal order (see has_wall_normals)
    double h = 0;
};

struct Variant {
    int block = 256;      // threads per workgroup (multiple of 64)
    int xcd = 1;          // XCD-aware block remap
    int persist = 8;      // K-field batch: resident workgroups per CU
    int lds = 1;          // 0 global gathers, 1 LDS-staged, 2 see rbffd_get_variant, 3 small sets
};

struct rbffd_plan {
    rbffd_params p{};
    int dim = 2;
    int n = 0, nh = 0, ns = 0;
    int M = 0, Mh = 0;
    int FE = 1, FH = 2;          // stored values per node
    int fe_comp = 1, fh_comp = 2;// physical components
    int K = 1;
    double dt = 0, gamma = 0, c0 = 1, eta0 = 1;
    double hv_fac = 0;           // gamma / c = (-1)^(alpha-1) h^(2 alpha)
    float* gk = nullptr;         // K-field batch: per-field gamma [K] (arena)
    NodeSet E, H;                // H unused unless two-set
    OpBlock opH, opE;            // operators of the H update and the E update
    bool collocated = true;
    // arena / workspace bookkeeping
    int64_t arena_bytes = 0, ws_bytes = 0, adj_ws_bytes = 0;
    int64_t t_entries = 0;       // entries of the transposed operator
    char* arena = nullptr;
    bool ready = false;
    Variant var;
    int32_t patience = RBFFD_STEP_PATIENCE;   // whole steps
    // private stream used only to capture HIP graphs (the caller's stream may
    // be the legacy null stream, which cannot be captured); default priority
    mutable hipStream_t cap_stream = nullptr;
    mutable std::atomic<uint32_t> whole_runs{0};   // runs that took whole steps so far (OpBlock::flags)
    std::string err;
    // Morton quantisation box (square): lo and common side
    double mlo[3] = {0, 0, 0};
    double mside = 1;
    int ex_m[RBFFD_MAX_MONO][3];   // monomial exponents (curl)
    int ex_h[RBFFD_MAX_MONO][3];   // monomial exponents (hv)
};

// Plans whose PEC walls may be curved keep per-node wall normals: where E is
// a vector (TEz, 3D) and the walls are PEC.
inline bool has_wall_normals(const rbffd_plan* p) {
    return p->p.bc == RBFFD_BC_PEC && (p->p.pol == RBFFD_POL_TE || p->dim == 3);
}

// plans with a kernel that takes a whole step (step.hip): it keeps the order of its
// tiles in OpBlock::ord
inline bool can_step_whole(const rbffd_plan* p) {
    return p->K == 1 && p->dim == 2 && p->collocated && p->p.pol != RBFFD_POL_TE && p->p.fdtype == RBFFD_F32 &&
           p->p.wdtype == RBFFD_F32;
}

// ---- run workspace: FP64 reduction partials ---------------------------------
constexpr int RED_BLOCKS = 1024;
struct RunWS {
    double* part;       // [RED_BLOCKS * 12]
};
inline RunWS run_ws(void* ws) {   // fits the smallest workspace (1 MB)
    RunWS w;
    w.part = (double*)ws;
    return w;
}

// one single-field step from (E, H) into (Eout, Hout) with the soft sources of
// that step (wave: their waveform row), as a run computes it (step.hip)
int plain_step_into(const rbffd_plan* p, const void* E, const void* H, void* Eout, void* Hout, const void* eps_r, int n_src,
                    const int32_t* src_node, const void* src_amp, const void* wave, hipStream_t st);

// K-field batch: per-field gamma from per-field constants c (device [K]), or
// every field the plan's gamma when c is null (batched.hip)
int fill_field_gamma(const rbffd_plan* p, const double* c_dev, hipStream_t st);

// ---- helpers --------------------------------------------------------------
int set_err(const rbffd_plan* p, int code, const std::string& msg);
#define HIPCHK(plan, call)                                                       \
    do {                                                                         \
        hipError_t e_ = (call);                                                  \
        if (e_ != hipSuccess)                                                    \
            return set_err(plan, RBFFD_EHIP, std::string(#call) + ": " +         \
                                                 hipGetErrorString(e_));         \
    } while (0)

static inline int64_t align_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }
static inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

int64_t n_monomials(int d, int m);
void fill_exponents(int d, int m, int ex[RBFFD_MAX_MONO][3]);
int field_elem_bytes(int fdtype);
int weight_elem_bytes(int wdtype);

// layout: assigns offsets (when base != nullptr also the pointers); returns
// arena bytes; ws receives the workspace requirement
int64_t layout_arena(rbffd_plan* p, char* base, int64_t* ws, int64_t* adj_ws);

// set-up entry points (setup.hip)
int setup_nodes_and_stencils(rbffd_plan* p, void* ws, hipStream_t s);
int setup_weights(rbffd_plan* p, void* ws, hipStream_t s);
int pack_all(rbffd_plan* p, void* ws, hipStream_t s);
int build_transpose(rbffd_plan* p, void* ws, hipStream_t s);
int refill_transpose(rbffd_plan* p, hipStream_t s);
int build_halos(rbffd_plan* p, void* ws, hipStream_t s);
int64_t setup_ws_bytes(const rbffd_plan* p);
int capture_stream(const rbffd_plan* p, hipStream_t* out);

// ---- HIP-graph step loop -----------------------------------------------------
// Stretches of plain steps (no sample, checkpoint, source or receiver in them)
// are replayed from a HIP graph of RBFFD_GRAPH_STEPS captured steps where
// launching them one by one is bound by the host: node sets of at most
// RBFFD_GRAPH_TILES tiles, whose half steps take less than the 4 us of a launch,
// and at least RBFFD_GRAPH_MIN_STEPS steps, which hide the capture (0.8 ms).
// us per step of the 51^2 cavity, launched / replayed, runs one after another:
// 100 steps 7.5 / 12.8, 200 steps 7.7 / 6.9, 1000 steps 8.0 / 6.6; on 40k nodes
// (two 8 us kernels) 15.8 / 16.0 at 1000 steps.  rec(c, stream) records one full
// step reading buffer set c; the buffers alternate within a graph and, its
// steps being even, every replay leaves them as it found them.  *done receives
// the number of steps replayed (even); the caller runs the rest.
#define RBFFD_GRAPH_STEPS 64
#define RBFFD_GRAPH_MIN_STEPS 192
#define RBFFD_GRAPH_TILES 256
template <typename Rec>
int replay_steps(const rbffd_plan* p, int T, int cur, hipStream_t st, Rec rec, int* done) {
    *done = 0;
    const int reps = T / RBFFD_GRAPH_STEPS;
    if (reps < 1) return RBFFD_OK;
    hipStream_t cs;
    int rc = capture_stream(p, &cs);
    if (rc) return rc;
    hipGraph_t g;
    hipGraphExec_t ge;
    HIPCHK(p, hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal));
    for (int k = 0; k < RBFFD_GRAPH_STEPS; ++k) rec((cur + k) & 1, cs);
    HIPCHK(p, hipStreamEndCapture(cs, &g));
    HIPCHK(p, hipGraphInstantiate(&ge, g, nullptr, nullptr, 0));
    for (int r = 0; r < reps; ++r) HIPCHK(p, hipGraphLaunch(ge, st));
    HIPCHK(p, hipGraphExecDestroy(ge));
    HIPCHK(p, hipGraphDestroy(g));
    *done = reps * RBFFD_GRAPH_STEPS;
    return RBFFD_OK;
}

// XCD-aware mapping of a linear workgroup id: consecutive logical ids land on
// the same XCD (round-robin dispatch sends block b to XCD b % 8), so
// spatially adjacent tiles share one L2.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
    const int x = b & 7, q = nb >> 3, r = nb & 7;
    return x * q + (x < r ? x : r) + (b >> 3);
}
// The same tiles, each XCD's in reverse: the E update of a staged step starts with
// what the H update read last and still finds it in cache (90k FP32 nodes, n 12,
// 13.3 -> 12.7 us per step; larger sets gain nothing and lose nothing).
__device__ __forceinline__ int tile_back(int xcd) {
    const int b = blockIdx.x, nb = gridDim.x, x = b & 7, q = nb >> 3, r = nb & 7;
    const int back = ((q + (x < r ? 1 : 0) - 1 - (b >> 3)) << 3) | x;
    return xcd ? xcd_remap(back, nb) : back;
}
