// Prefill / training GEMM of the sparse ternary linear layer on CDNA4 int8 matrix cores (2:4).
//   acc[t, o] = sum_k W_eff[o, k] * xq[t, k],   Y = acc * gamma / s_x[t] (+ bias)
// Section 2.2 (forward-pass equation).  Two paths:
//   sparse  v_smfmac_i32_32x32x64_i8: the packed weights ARE the compressed A operand (code word ->
//           16 int8 values, index word -> the instruction's index register), tokens are B;
//   dense   v_mfma_i32_32x32x32_i8 on W_eff expanded to int8 with explicit zeros: the in-run
//           comparison a dense ternary layer would run.
#include <algorithm>
#include <type_traits>
#include <vector>

#include "sbn_internal.hpp"
#include "sbn_mfma.hpp"

namespace sbn {

namespace {

constexpr int BO = 256;        // output rows (of W) per block
constexpr int BT = 128;        // tokens per block
constexpr int KSTEP = 128;     // input features per main-loop iteration = one packed chunk

struct GemmArgs {
    const int8_t *xq;
    const float *sx;
    const uint8_t *packed;   // sparse path
    const int8_t *w_dense;   // dense path
    const float *gamma;
    const float *bias;
    float *Y;
    int32_t *acc_out;
    int tokens, d_in, d_out;
    int tiles_o, tiles_t;
};

// A launch of the sparse kernel covers up to GEMM_GROUP_MAX problems with a work list, or up to GEMM_GROUP_WIDE
// problems of few tokens each (decode batches), whose work is dealt by row tile (see gemm_smfmac_kernel).
constexpr int GEMM_GROUP_MAX = 8, GEMM_GROUP_WIDE = 32;
template <int NP>
struct GemmGroupT {
    GemmArgs g[NP];
    int count;
};
using GemmGroup = GemmGroupT<GEMM_GROUP_MAX>;
using GemmGroupWide = GemmGroupT<GEMM_GROUP_WIDE>;

// Work list of a launch of the sparse kernel, made on the host: block b runs the pieces piece[b * per_block + i],
// i < per_block, up to the first empty one (width 0).  A piece = (problem, row tile of 512, first token unit of 32 tokens,
// width in units 1 .. 4).  per_block == 0: no list, the kernel splits the units by formula.
// per_block < 0: no list either, the problems have few tokens and the pieces are (problem, row tile, four token units),
// -per_block of them in all, dealt to the blocks in contiguous runs.
constexpr int PIECE_TABLE_MAX = 768;
template <int NE>
struct PieceTableT {
    int per_block;
    uint32_t piece[NE];   // bits [2:0] width, [15:3] first unit, [24:16] row tile, [27:25] problem
};
using PieceTable = PieceTableT<PIECE_TABLE_MAX>;
using PieceTableNone = PieceTableT<1>;
static_assert(sizeof(GemmGroup) + sizeof(PieceTable) <= 4000, "both travel as kernel arguments");
static_assert(sizeof(GemmGroupWide) + sizeof(PieceTableNone) <= 4000, "both travel as kernel arguments");

// Tile order of the dense comparison kernel.
// Blocks are dealt round-robin to the 8 XCDs, each with its own 4 MB L2.  XCD x takes the token
// tiles [x, x+1) * tiles_t/8 and walks them in groups of four: inside a group the token tile is the
// fastest index, then the row tile.  The 64 blocks an XCD runs at a time then share four token tiles
// (1.3 MB, resident for the whole group) while the packed weights stream through its L2 once per
// group, instead of every row tile being re-fetched for every token tile (measured: L2 miss traffic
// 15x the unique input bytes with the row tile fastest).
__device__ __forceinline__ void tile_of_block(const GemmArgs &g, int id, int &to, int &tt)
{
    const int tpx = g.tiles_t >> 3;   // token tiles per XCD
    if ((g.tiles_t & 7) == 0 && (tpx % 4 == 0 || tpx < 4)) {
        const int tg = tpx < 4 ? tpx : 4;
        const int x = id & 7, j = id >> 3;
        const int group = j / (g.tiles_o * tg), rem = j % (g.tiles_o * tg);
        to = rem / tg;
        tt = x * tpx + group * tg + rem % tg;
    } else {
        to = id % g.tiles_o;
        tt = id / g.tiles_o;
    }
}

__device__ __forceinline__ void store_tile(const GemmArgs &g, const v16i &acc, int o_base, int t, float scale)
{
    // lane holds token t and rows o_base + 8*(i/4) + i%4  (o_base already includes 4*(lane/32))
    if (t >= g.tokens) return;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int o = o_base + 8 * q;
        if (o + 3 < g.d_out && (g.d_out & 3) == 0) {
            float4 y;
            y.x = (float)acc[4 * q + 0] * scale;
            y.y = (float)acc[4 * q + 1] * scale;
            y.z = (float)acc[4 * q + 2] * scale;
            y.w = (float)acc[4 * q + 3] * scale;
            if (g.bias) {
                const float4 b = *reinterpret_cast<const float4 *>(g.bias + o);
                y.x += b.x; y.y += b.y; y.z += b.z; y.w += b.w;
            }
            *reinterpret_cast<float4 *>(g.Y + (int64_t)t * g.d_out + o) = y;
            if (g.acc_out)
                *reinterpret_cast<int4 *>(g.acc_out + (int64_t)t * g.d_out + o) =
                    make_int4(acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]);
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (o + i < g.d_out) {
                    float y = (float)acc[4 * q + i] * scale;
                    if (g.bias) y += g.bias[o + i];
                    g.Y[(int64_t)t * g.d_out + o + i] = y;
                    if (g.acc_out) g.acc_out[(int64_t)t * g.d_out + o + i] = acc[4 * q + i];
                }
            }
        }
    }
}

// Epilogue of the dense comparison kernel.  A wavefront owns RA row tiles x TB token tiles of 32x32; a lane
// holds one token and rows 8q + 4c + i of each row tile, so a direct store would put only 32
// contiguous bytes per token into each instruction (measured: 1.5x the algorithmic write traffic).
// The accumulators are rescaled, transposed through the now idle LDS ring (32 tokens x 32*RA rows of
// fp32 per wavefront and pass) and leave as whole rows of 128*RA bytes.  Ragged row edges and the
// int32 accumulator output take the plain per-lane stores.
//   orow = first output row of the wavefront, tok0 = its first token
template <int RA, int TB>
__device__ __forceinline__ void block_epilogue(const GemmArgs &g, v16i (&acc)[RA][TB], const float (&sxv)[TB + 1],
                                               int8_t *lds, int o0, int orow, int tok0, int wave, int lane)
{
    const int r = lane & 31, c = lane >> 5;
    const bool fast_store = (g.d_out & 3) == 0 && o0 + BO <= g.d_out && !g.acc_out;
    if (fast_store) {
        constexpr int EROW = 128 * RA + 16;     // bytes per staged token row (padded)
        constexpr int LPR = 8 * RA;             // lanes (float4) per token row
        constexpr int RPI = 64 / LPR;           // token rows per store instruction
        int8_t *const est = lds + wave * (32 * EROW);
        __syncthreads();   // every wavefront has left the main loop: the ring can be overwritten
        v4f bias4 = {0.f, 0.f, 0.f, 0.f};
        if (g.bias) bias4 = *reinterpret_cast<const v4f *>(g.bias + orow + 4 * (lane % LPR));
        const int tokens = g.tokens;
        const int64_t d_out = g.d_out;
        const bool all_tokens = tok0 + 32 * TB <= tokens;
        float *const ybase = g.Y + (int64_t)(tok0 + lane / LPR) * d_out + orow + 4 * (lane % LPR);
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const float scale = __fdiv_rn(sxv[TB], sxv[b]);
#pragma unroll
            for (int a = 0; a < RA; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float4 y;
                    y.x = (float)acc[a][b][4 * q + 0] * scale;
                    y.y = (float)acc[a][b][4 * q + 1] * scale;
                    y.z = (float)acc[a][b][4 * q + 2] * scale;
                    y.w = (float)acc[a][b][4 * q + 3] * scale;
                    *reinterpret_cast<float4 *>(est + r * EROW + (32 * a + 8 * q + 4 * c) * 4) = y;
                }
            // the wavefront reads back what it wrote itself (its LDS operations complete in order):
            // all reads of the pass first, then the stores, so that the LDS latency is paid once
            v4f yv[32 / RPI];
#pragma unroll
            for (int j = 0; j < 32 / RPI; ++j)
                yv[j] = *reinterpret_cast<const v4f *>(est + (RPI * j + lane / LPR) * EROW + (lane % LPR) * 16);
#pragma unroll
            for (int j = 0; j < 32 / RPI; ++j) {
                yv[j] += bias4;
                // streaming store: Y is not read again here and must not push the operands out of L2
                if (all_tokens || tok0 + 32 * b + RPI * j + lane / LPR < tokens)
                    __builtin_nontemporal_store(yv[j], reinterpret_cast<v4f *>(ybase + (int64_t)(32 * b + RPI * j) * d_out));
            }
        }
        return;
    }
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        const int t = tok0 + 32 * b + r;
#pragma unroll
        for (int a = 0; a < RA; ++a) store_tile(g, acc[a][b], orow + 32 * a + 4 * c, t, __fdiv_rn(sxv[TB], sxv[b]));
    }
}

// gamma and s_x[t] of the TB tokens a lane holds (token tile b: tok0 + 32 b + lane % 32), fetched
// before the first DMA so that they are long there when the epilogue divides them (a chain of
// dependent global loads at the start of the epilogue otherwise); absent tokens read the last token
template <int TB>
__device__ __forceinline__ void load_scales(const GemmArgs &g, int tok0, int lane, float (&sxv)[TB + 1])
{
    sxv[TB] = *g.gamma;
#pragma unroll
    for (int b = 0; b < TB; ++b) {
        const int t = tok0 + 32 * b + (lane & 31);
        sxv[b] = g.sx[t < g.tokens ? t : g.tokens - 1];
    }
}

// ---- sparse path --------------------------------------------------------------------------------
// One persistent block of eight wavefronts per multiprocessor; block tile 512 rows x 128 tokens.  Wavefront w owns the
// rows 64 w .. 64 w + 63 (two row tiles of 32) and all tokens of the piece (TB = 1 .. 4 token tiles of 32), so one code
// expansion (a shift and a mask for each of four registers) feeds TB matrix instructions: measured on this part, up to
// four vector instructions per matrix instruction hide under it, more cost their full time.  The two wavefronts of a SIMD cover
// each other's waits.  Per 128-k step the wavefronts read 144 KB of operand fragments from LDS and the DMA deposits
// 32 KB; measured with a microbenchmark, reads (475 bytes/ns) and deposits (105 bytes/ns from L2) overlap, so it is
// the deposit path that is scarce: a step's 32 KB are 0.3 us of it against 0.5 us of matrix work.  Against two
// independent blocks of 256 x 128 the shared token tile saves a third of those bytes (256 instead of 384 bytes per
// matrix instruction).
// Both operands reach LDS through LDS-DMA loads (lane l of a wavefront deposits its 16 bytes at base + 16*l), so no
// staging registers are needed and every load instruction reads whole cache lines:
//   tokens   128 tokens x 128 int8 per stage, ring of NST stages; one instruction fills 8 token rows of 128 bytes; the
//            16-byte column a lane fetches is XOR-swizzled with (row >> 1) & 7 so that 16-byte reads of 16
//            consecutive rows fall in distinct banks;
//   weights  512 rows x 64 bytes (two 32-byte chunks = two iterations) per pair slot, ring of NWP slots; one instruction
//            fills 16 rows; 16-byte granules swizzled with (row >> 2) & 3.
// A lane (row r = lane % 32, half c = lane / 32) reads index words 2c, 2c+1 and code words 2c, 2c+1 of its row's chunk
// (two 8-byte LDS reads per row tile); sub-step u = 0, 1 uses word 2c + u, i.e. the lane supplies weights
// [64c + 32u, +32) of the chunk.
// Pieces follow one another without draining the pipeline: the requests run on from a piece into the block's next one
// under the last products, and the epilogue transposes through a staging area of its own, so the ring is never idle.
// What bounds it: no one thing.  The board's power holds the clock at 1.6 GHz, where 2:4 products of random operands from
// registers run at 6.5 POP/s dense-equivalent with codes +-1 and 6.9 with +-64, but a matrix instruction executes in 46 % of the SIMD
// cycles of 32768 tokens, 2560 -> 6912 (14 pieces per multiprocessor), and in 29 % at 4096 tokens (one or two): a step takes 1500
// cycles for 1024 of matrix work, and the results stand beside it, all multiprocessors storing at about the same time: 365 us, 306
// without an output store; 4096 tokens 54 and 43, 2560 -> 2560 22.2 and 19.4 (a build for timing alone).  Before codes of +-64, the
// tiles of the epilogue and the running requests 416, 56.6 and 22.5.
namespace sp {

constexpr int ROWS = 512;                      // rows of W per block tile
constexpr int NW = 8;                          // wavefronts
constexpr int RA = 2;                          // row tiles per wavefront
constexpr int NST = 3;                         // token stages (16 KB each)
constexpr int NWP = 2;                         // weight pair slots (32 KB each)
constexpr int TSTAGE = 128 * KSTEP;
constexpr int WPAIR = ROWS * 64;
constexpr int RING_BYTES = NST * TSTAGE + NWP * WPAIR;
// epilogue staging, one area per wavefront: a tile of 32 tokens x 32 rows of fp32, its 16-byte granules swizzled with (token >> 1) & 7
constexpr int STG_WAVE = 32 * 128;
// per-token scales of a piece (128 floats), fetched by DMA with its first stages; two areas, used alternately, because
// the scales of the next piece arrive while the epilogue of the current one still reads its own
constexpr int SCALES_OFF = RING_BYTES + NW * STG_WAVE;
constexpr int LDS_BYTES = SCALES_OFF + 2 * 512;
static_assert(LDS_BYTES <= 160 * 1024, "ring, staging and scales share the multiprocessor's LDS");
constexpr int NDW = 32 / NW;                   // weight DMA instructions per wavefront and pair (16 rows each)
constexpr int token_dma(int TB) { return (4 * TB + NW - 1) / NW; }   // token DMA instructions per wavefront and stage (8 rows each)
constexpr int cmin(int a, int b) { return a < b ? a : b; }

// Bookkeeping of the DMA ring at compile time.  Iteration j (negative j = the prologue) issues, in this order,
// weight pair (j - 1) / 2 + NWP if j is odd (NDW instructions), then token stage j + NST (NDT instructions); items with
// a negative number do not exist.  Returns how many DMA instructions of a wavefront are issued after the given item
// in iterations jlo .. jhi: the count a wait for that item may leave outstanding (the loads of a wavefront complete
// in issue order).
constexpr int issued_after(int NDT, int jlo, int jhi, bool want_pair, int id)
{
    int n = -1;
    for (int j = jlo; j <= jhi; ++j) {
        if (j & 1) {
            const int pid = (j - 1) / 2 + NWP;
            if (pid >= 0) {
                if (n >= 0) n += NDW;
                else if (want_pair && pid == id) n = 0;
            }
        }
        const int sid = j + NST;
        if (sid >= 0) {
            if (n >= 0) n += NDT;
            else if (!want_pair && sid == id) n = 0;
        }
    }
    return n;
}
constexpr int LEAD = NST > 2 * NWP - 1 ? NST : 2 * NWP - 1;          // prologue iterations -LEAD .. -1

// A piece of the work list: (problem, row tile, first token, width in token tiles); width 0 = none.
struct Piece {
    int prob, to, t0, tb;
    int parity;   // which of the two scale areas the piece uses
};

// The stream of requests of a block, ahead of its products by NST token stages and NWP weight pairs and continuing from one
// piece into the next.  Everything in it is uniform: the operands of the piece it is in as buffers (rows past the matrix or the
// piece, and chunks past the last row, read as zeros and fetch nothing), and how far it has come.  Token instruction i of
// wavefront w fills tile rows (NW i + w) 8 .. + 7, weight instruction i fills block rows (NDW w + i) 16 .. + 15: a row of a slot is
// always filled by the same wavefront, whatever the width of the piece, so requests for it land in the order they were made.
struct Stream {
    v4i tokens, weights;
    uint32_t token_at, weight_at;   // bytes into a row
    int ts, ps;                     // ring slots of the next piece's first stage and pair
    bool landed;                    // everything asked for so far
};

// The sizes of both buffers, at most 128 tokens or 512 rows of weights, have 32 bits.
constexpr int64_t ROW_END = (int64_t)1 << 25;   // of d_in: 128 times as many bytes do not fit them
__device__ __forceinline__ v4i token_buffer(const GemmArgs &g, const Piece &p)
{
    const int left = g.tokens - p.t0, rows = left < 32 * p.tb ? left : 32 * p.tb;
    return buffer_of(g.xq + (int64_t)p.t0 * g.d_in, (uint32_t)rows * (uint32_t)g.d_in);
}

__device__ __forceinline__ v4i weight_buffer(const GemmArgs &g, const Piece &p)
{
    const int left = g.d_out - p.to * ROWS, rows = left < ROWS ? left : ROWS, pitch = g.d_in / KSTEP * 32;
    return buffer_of(g.packed + (int64_t)p.to * ROWS * pitch, (uint32_t)rows * (uint32_t)pitch);
}

__device__ __forceinline__ v4i no_buffer() { return v4i{0, 0, 0, 0x00027000}; }

// lane offsets; the further instructions of a wavefront are 64 token rows or 16 weight rows on
__device__ __forceinline__ uint32_t token_offset(int d_in, int wave, int lane)
{
    const int row = 8 * wave + (lane >> 3);
    return (uint32_t)row * (uint32_t)d_in + 16u * ((lane & 7) ^ ((row >> 1) & 7));
}

__device__ __forceinline__ uint32_t weight_offset(int d_in, int wave, int lane)
{
    const int row = 16 * NDW * wave + (lane >> 2);
    return (uint32_t)row * (uint32_t)(d_in / KSTEP * 32) + 16u * ((lane & 3) ^ ((row >> 2) & 3));
}

// s_x of a piece's tokens, by the first wavefront
__device__ __forceinline__ void request_scales(const GemmArgs &g, const Piece &p, uint32_t lds0, int wave, int lane)
{
    if (wave != 0) return;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = p.t0 + 64 * i + lane;
        lds_dma4(g.sx, 4u * (uint32_t)(t < g.tokens ? t : g.tokens - 1), lds0 + SCALES_OFF + 512 * p.parity + 256 * i);
    }
}

// Starts the stream at a piece: its first stages and pairs go to the slots (ts, ps) and on.
__device__ __forceinline__ void start_stream(Stream &st, const GemmArgs &g, const Piece &p, uint32_t lds0, int wave, int lane)
{
    const uint32_t K = (uint32_t)g.d_in, pitch = K / KSTEP * 32;
    st.tokens = token_buffer(g, p);
    st.weights = weight_buffer(g, p);
    const bool wide = token_dma(p.tb) > 1;
    const uint32_t xoff = token_offset(g.d_in, wave, lane), woff = weight_offset(g.d_in, wave, lane);
    auto pair = [&](const int s) {
        const uint32_t slot = (uint32_t)(st.ps + s) % NWP;
        const v4i buffer = 64u * s < pitch ? st.weights : no_buffer();
#pragma unroll
        for (int i = 0; i < NDW; ++i)
            lds_dma16_buffer(buffer, woff, 64u * s + 16u * i * pitch, lds0 + NST * TSTAGE + slot * WPAIR + (NDW * wave + i) * 1024);
    };
    auto stage = [&](const int s) {
        const uint32_t slot = (uint32_t)(st.ts + s) % NST;
        const v4i buffer = (uint32_t)KSTEP * s < K ? st.tokens : no_buffer();
        lds_dma16_buffer(buffer, xoff, (uint32_t)KSTEP * s, lds0 + slot * TSTAGE + wave * 1024);
        if (wide) lds_dma16_buffer(buffer, xoff, (uint32_t)KSTEP * s + 64u * K, lds0 + slot * TSTAGE + (NW + wave) * 1024);
    };
    // the order in which the iterations in front of the first would have asked
#pragma unroll
    for (int j = -LEAD; j < 0; ++j) {
        if ((j & 1) && (j - 1) / 2 + NWP >= 0) pair((j - 1) / 2 + NWP);
        if (j + NST >= 0) stage(j + NST);
    }
    st.token_at = NST * KSTEP;
    st.weight_at = NWP * 64;
}

// the stream of a block at its first piece
template <class Group>
__device__ __forceinline__ Stream first_stream(const Group &grp, const Piece &p, int8_t *lds, int wave, int lane)
{
    const uint32_t lds0 = lds_address(lds);
    Stream st;
    st.ts = st.ps = 0;
    request_scales(grp.g[p.prob], p, lds0, wave, lane);
    start_stream(st, grp.g[p.prob], p, lds0, wave, lane);
    st.landed = false;
    return st;
}

// Main loop and epilogue of one piece whose first stages have landed or are in flight: rows [512 to, +512) of W against tokens
// [t0, t0 + 32 TB), the whole input dimension.  LIVE = false: a wavefront whose rows lie past the matrix (ragged last
// row tile) only moves data and keeps the barriers.  UNIT = false: the codes are +-64 (expand_codes_x64), the accumulators 64 times
// the sums.
template <int TB, bool LIVE, bool DENSE, bool UNIT, class Group>
__device__ __forceinline__ void piece_body(const Group &grp, const Piece &p, const Piece &next, Stream &st, int8_t *lds, const int wave,
                                           int lane)
{
    // everything derived from the lane number is computed anew for every piece: hoisted out of the loop over pieces,
    // the lane addresses of all instantiations would be live at once and spill
    asm volatile("" : "+v"(lane));
    constexpr int NDT = token_dma(TB);
    constexpr int WAIT_TOP = cmin(issued_after(NDT, -LEAD, -1, false, 0), issued_after(NDT, -LEAD, -1, true, 0));
    // in the middle of iteration kc: token stage kc + 1 and, for odd kc, weight pair (kc + 1) / 2 must have landed
    constexpr int WAIT_EVEN = issued_after(NDT, -LEAD, 99, false, 101);
    // (in front of which an odd iteration has already asked for its weight pair)
    constexpr int WAIT_ODD = cmin(issued_after(NDT, -LEAD, 100, false, 102), issued_after(NDT, -LEAD, 100, true, 51)) + NDW;
    static_assert(WAIT_TOP >= 0 && WAIT_EVEN >= 0 && WAIT_ODD >= 0 && WAIT_TOP < 64 && WAIT_EVEN < 64 && WAIT_ODD < 64,
                  "ring bookkeeping");
    const GemmArgs &g = grp.g[p.prob];
    const int to = p.to, t0 = p.t0;
    const uint32_t lds0 = lds_address(lds), wlds0 = lds0 + NST * TSTAGE;
    const int r = lane & 31, c = lane >> 5;
    const int nchunks = g.d_in / KSTEP;
    const int o0 = to * ROWS;

    // ---- requests: at the end of the piece the stream goes on with the next one, where that has rows of the same length and needs
    // no more instructions per stage (whether it does is not asked between the matrix instructions: that branch cost 90 cycles per
    // chunk, 12.8 us against 11.7 at 777 tokens, 2560 -> 2560); otherwise it is started anew behind the main loop, and until
    // then asks for nothing
    const uint32_t K = (uint32_t)g.d_in, pitch = K / KSTEP * 32;
    const uint32_t xoff = token_offset(g.d_in, wave, lane), woff = weight_offset(g.d_in, wave, lane);
    const bool goes_on = next.tb > 0 && token_dma(next.tb) <= NDT && grp.g[next.prob].d_in == g.d_in && nchunks >= NST && nchunks > 2 * (NWP - 1);
    const v4i next_tokens = goes_on ? token_buffer(grp.g[next.prob], next) : no_buffer();
    const v4i next_weights = goes_on ? weight_buffer(grp.g[next.prob], next) : no_buffer();
    auto request_tokens = [&](const int slot, const int i) {   // instruction i of NDT
        if (i == 0) {   // selections: a branch would part the instructions around it
            const bool turn = st.token_at >= K;
            st.tokens = turn ? next_tokens : st.tokens;
            st.token_at = turn ? 0 : st.token_at;
        }
        lds_dma16_buffer(st.tokens, xoff, st.token_at + 64u * i * K, lds0 + slot * TSTAGE + (NW * i + wave) * 1024);
        if (i == NDT - 1) st.token_at += KSTEP;
    };
    auto request_weights = [&](const int slot, const int i) {   // instruction i of NDW
        if (i == 0) {
            const bool turn = st.weight_at >= pitch;
            st.weights = turn ? next_weights : st.weights;
            st.weight_at = turn ? 0 : st.weight_at;
        }
        lds_dma16_buffer(st.weights, woff, st.weight_at + 16u * i * pitch, lds0 + NST * TSTAGE + slot * WPAIR + (NDW * wave + i) * 1024);
        if (i == NDW - 1) st.weight_at += 64;
    };

    // ---- LDS read addresses (swizzles as in the DMA patterns above)
    uint32_t b_lo[2], b_hi[2];   // [sub-step]; the token tile is an immediate offset, the ring slot a scalar
    {
        const int sw = (r >> 1) & 7;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            b_lo[u] = lds0 + r * KSTEP + 16 * ((2 * u + c) ^ sw);
            b_hi[u] = lds0 + r * KSTEP + 16 * ((4 + 2 * u + c) ^ sw);
        }
    }
    // [chunk of the pair][row tile], slot 0.  2:4: index words 2c, 2c+1 and code words 2c, 2c+1 of the chunk (8 bytes
    // each); dense codes: words 4c .. 4c+3 of the chunk's eight code words (a_idx alone, 16 bytes)
    uint32_t a_idx[2][RA], a_code[2][RA];
#pragma unroll
    for (int a = 0; a < RA; ++a) {
        const int row = wave * (32 * RA) + 32 * a + r, sw = (row >> 2) & 3;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if constexpr (DENSE) {
                a_idx[h][a] = wlds0 + row * 64 + 16 * ((2 * h + c) ^ sw);
                a_code[h][a] = 0;
            } else {
                a_idx[h][a] = wlds0 + row * 64 + 8 * c + 16 * ((2 * h) ^ sw);
                a_code[h][a] = wlds0 + row * 64 + 8 * c + 16 * ((2 * h + 1) ^ sw);
            }
        }
    }
    typedef __attribute__((address_space(3))) const v4i *lds_v4i;
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) const v2u *lds_u2;
    const uint32_t ones = UNIT ? vgpr_ones() : 0;

    v16i acc[RA][TB];
#pragma unroll
    for (int a = 0; a < RA; ++a)
#pragma unroll
        for (int b = 0; b < TB; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0;

    // 2:4: (icur, ccur) = the lane's two index and two code words of the current chunk; dense codes: its four code words
    v2u icur[RA], ccur[RA], inext[RA], cnext[RA];
    v8i bq[2][TB];
    auto read_weights = [&](const int slot, const int h, const int a, v2u (&iv)[RA], v2u (&cv)[RA]) {
        if constexpr (DENSE) {
            const v4u w = *(__attribute__((address_space(3))) const v4u *)(uintptr_t)(a_idx[h][a] + slot * WPAIR);
            iv[a] = v2u{w.x, w.y};
            cv[a] = v2u{w.z, w.w};
        } else {
            iv[a] = *(lds_u2)(uintptr_t)(a_idx[h][a] + slot * WPAIR);
            cv[a] = *(lds_u2)(uintptr_t)(a_code[h][a] + slot * WPAIR);
        }
    };
    auto token_read = [&](const int slot, const int u, const int b, v8i &bf) {   // the tile is an index, hence an immediate offset
        bf.lo = ((lds_v4i)(uintptr_t)(b_lo[u] + slot * TSTAGE))[32 * b * KSTEP / 16];
        bf.hi = ((lds_v4i)(uintptr_t)(b_hi[u] + slot * TSTAGE))[32 * b * KSTEP / 16];
    };
    // One sub-step: RA x TB matrix instructions; side(s) is issued after instruction s (s = 0 .. RA * TB - 1).  A
    // wavefront issues at most one instruction every few cycles, so what is placed between matrix instructions is free
    // while the matrix pipe is busy, and a block of other instructions after them leaves the pipe idle: the source order
    // is the intended issue order and a scheduling barrier after every matrix instruction keeps it.
    // Dense codes: every group of four weights is the sum of a 2:4 group holding its positions 0, 1 and one holding its
    // positions 2, 3, so the same B fragment feeds two sparse instructions with constant index words.
    constexpr int NSLOT = (DENSE ? 2 : 1) * RA * TB;
    auto substep = [&](const int u, const v8i (&bf)[TB], auto &&side) {
#pragma unroll
        for (int a = 0; a < RA; ++a) {
            if constexpr (LIVE && DENSE) {
                v4i a01, a23;   // sub-step u covers the lane's code words 2u, 2u + 1
                if constexpr (UNIT) expand_dense_codes(u ? ccur[a].x : icur[a].x, u ? ccur[a].y : icur[a].y, a01, a23);
                else expand_dense_codes_x64(u ? ccur[a].x : icur[a].x, u ? ccur[a].y : icur[a].y, a01, a23);
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    acc[a][b] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(a01, bf[b], acc[a][b], 0x44444444, 0, 0);
                    side(2 * a * TB + b);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    acc[a][b] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(a23, bf[b], acc[a][b], (int)0xeeeeeeeeu, 0, 0);
                    side((2 * a + 1) * TB + b);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else if constexpr (LIVE) {
                const int iv = (int)(u ? icur[a].y : icur[a].x);
                v4i av;
                if constexpr (UNIT) av = expand_codes(u ? ccur[a].y : ccur[a].x, ones);
                else av = expand_codes_x64(u ? ccur[a].y : ccur[a].x);
#pragma unroll
                for (int b = 0; b < TB; ++b) {
                    acc[a][b] = __builtin_amdgcn_smfmac_i32_32x32x64_i8(av, bf[b], acc[a][b], iv, 0, 0);
                    side(a * TB + b);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int s = 0; s < NSLOT / RA; ++s) side(a * (NSLOT / RA) + s);
            }
        }
    };

    // gamma, from constant memory: behind the requests, which may write any memory as far as the compiler knows, it would be a vector load in
    // front of the epilogue, waited for there together with everything that has been asked for of the next piece
    float gamma = *reinterpret_cast<const __attribute__((address_space(4))) float *>(reinterpret_cast<uintptr_t>(g.gamma));
    int ts = st.ts, ps = st.ps;
    if (!st.landed) SBN_WAIT_VMCNT(WAIT_TOP);   // pair 0 and stage 0; what was asked for after them may fly
    __syncthreads();
    asm volatile("" : "+s"(gamma));   // here it is
    if (next.tb > 0) request_scales(grp.g[next.prob], next, lds0, wave, lane);   // its area was read by the epilogue before this piece
    if constexpr (LIVE) {
#pragma unroll
        for (int a = 0; a < RA; ++a) read_weights(ps, 0, a, icur, ccur);
#pragma unroll
        for (int b = 0; b < TB; ++b) token_read(ts, 0, b, bq[0][b]);
    }
    // One iteration; ts, ps are the slots of its token stage and weight pair, h = kc & 1 is a literal.
    //   sub-step 0   compute (kc, first half); the token fragments of the second half are read under it.  Odd kc, and the last: the
    //                words of this pair are in the wavefront's registers (the instructions of the second row tile have waited
    //                for the last of them) and its rows of the slot are read by no other, so they take the pair NWP further on
    //   middle       wait for token stage kc + 1 (odd kc: and weight pair (kc + 1) / 2), barrier: every wavefront
    //                now holds all of stage kc in registers, so its slot takes the stage NST further on
    //   sub-step 1   compute (kc, second half); under it go the weight words of chunk kc + 1, the token fragments of (kc + 1,
    //                first half) and the requests for tokens, one per matrix instruction: what the next iteration begins with
    //                is asked for first
    // The wait counts hold the outstanding requests of this wavefront only.  Everything that was asked for in front of a piece behind
    // another has landed when it begins, so its first two iterations wait for nothing: there the stores of the epilogue before may
    // still be in flight, and would be waited for.  Later they make a wait longer, never shorter.
    const int settled = st.landed ? 2 : 0;
    st.landed = true;
    auto iteration = [&](const int kc, const int h, auto last) {
        constexpr bool LAST = last();
        substep(0, bq[0], [&](const int s) {
            if constexpr (LIVE) { if (s < TB) token_read(ts, 1, s, bq[1][s]); }
            if (h == 1 || LAST) {
                constexpr int FIRST = NSLOT / RA;
#pragma unroll
                for (int k = 0; k < NDW; ++k)
                    if (FIRST + k * (NSLOT - FIRST) / NDW == s) request_weights(ps, k);
            }
        });
        if (!LAST && kc >= settled) { if (h == 0) SBN_WAIT_VMCNT(WAIT_EVEN); else SBN_WAIT_VMCNT(WAIT_ODD); }
        __syncthreads();
        const int nts = ts + 1 == NST ? 0 : ts + 1;                            // slot of token stage kc + 1
        const int nps = h == 1 || LAST ? (ps + 1 == NWP ? 0 : ps + 1) : ps;    // slot of the pair of chunk kc + 1
        substep(1, bq[1], [&](const int s) {
            constexpr int READS = LAST ? 0 : RA + TB, NOPS = READS + NDT;
#pragma unroll
            for (int k = 0; k < NOPS; ++k) {
                if ((k < NSLOT ? k : NSLOT - 1) != s) continue;
                if (k >= READS) request_tokens(ts, k - READS);
                else if constexpr (LIVE) {
                    if (k < RA) read_weights(nps, h ^ 1, k, inext, cnext);
                    else token_read(nts, 0, k - RA, bq[0][k - RA]);
                }
            }
        });
        if constexpr (LIVE && !LAST) {
#pragma unroll
            for (int a = 0; a < RA; ++a) { icur[a] = inext[a]; ccur[a] = cnext[a]; }
        }
        ts = nts;
        ps = nps;
    };
    constexpr std::false_type more{};
    constexpr std::true_type last{};
    int kc = 0;
    for (; kc + 2 < nchunks; kc += 2) {
        iteration(kc, 0, more);
        iteration(kc + 1, 1, more);
    }
    if (kc + 1 < nchunks) iteration(kc, 0, more);
    iteration(nchunks - 1, 0, last);
    st.ts = ts;
    st.ps = ps;
    if (next.tb > 0 && !goes_on) start_stream(st, grp.g[next.prob], next, lds0, wave, lane);

    // ---- epilogue: rescale, transpose through the wavefront's staging area (4 KB of fp32 at a time) and
    // write runs of 128 or 256 bytes (per-lane stores of 32 contiguous bytes measured 1.5x the write traffic).
    // A vector load of the epilogue makes the compiler wait for everything outstanding, the requests for the next piece included,
    // so there is none but the bias where there is one: gamma has been fetched with the piece, its s_x came into LDS.
    if constexpr (LIVE) {
        float sxv[TB];
#pragma unroll
        for (int b = 0; b < TB; ++b) sxv[b] = *reinterpret_cast<const float *>(lds + SCALES_OFF + 512 * p.parity + 4 * (32 * b + r));
        const int orow = o0 + wave * (32 * RA);
        float scale[TB];
        bool exact = true;   // whether a 64th of the scales is
#pragma unroll
        for (int b = 0; b < TB; ++b) {
            const float v = __fdiv_rn(gamma, sxv[b]);
            exact = exact && fabsf(v) >= 0x1p-100f;
            scale[b] = UNIT ? v : v * (1.0f / (1 << CODE_SHIFT));
        }
        // (a piece's outputs are addressed with 31 bits behind its first)
        const bool fast_store = (g.d_out & 3) == 0 && !g.acc_out && g.d_out <= (1 << 22) && (UNIT || __all(exact));
        if (fast_store) {
            int8_t *const est = lds + RING_BYTES + wave * STG_WAVE;
            const bool has_bias = g.bias != nullptr;
            // tokens past the matrix lie past the end of the buffer, where stores are dropped, and so do, by an offset of their own,
            // rows of W past it (a ragged last wavefront; 2181 tokens 512 -> 480 stored lane by lane 6.6 us, this way 6.25)
            const int64_t first = (int64_t)t0 * g.d_out + orow;
            const uint32_t pitch = 4u * (uint32_t)g.d_out;
            const auto out = __builtin_amdgcn_make_buffer_rsrc(g.Y + first, (short)0, (int)((uint32_t)(g.tokens - t0 < 32 * TB ? g.tokens - t0 : 32 * TB) * pitch - 4u * (uint32_t)orow), 0x00027000);
            auto offset = [&](const uint32_t at, const int row) { return orow + row < g.d_out ? at + 4u * (uint32_t)row : 0x80000000u; };
            auto bias_of = [&](const int row) { return has_bias && orow + row < g.d_out ? *reinterpret_cast<const v4f *>(g.bias + orow + row) : v4f{0.f, 0.f, 0.f, 0.f}; };
            v4f yv[4];
            auto rescaled = [&](const int a, const int b, const int q) {
                return v4f{(float)acc[a][b][4 * q + 0] * scale[b], (float)acc[a][b][4 * q + 1] * scale[b],
                           (float)acc[a][b][4 * q + 2] * scale[b], (float)acc[a][b][4 * q + 3] * scale[b]};
            };
            // A wavefront's LDS operations complete in order, so a tile is written behind the reads of the one before without a wait.
            // Tile by tile: with a tile's stores behind the conversions of the next one (and their order kept by scheduling barriers)
            // the results took 0.1 to 0.3 us longer per launch (2048 tokens 512 -> 2048 7.8 us / 7.6, 1714 tokens 384 -> 1800 8.2 /
            // 7.9), 32768 tokens 2560 -> 6912 362 / 357.
            static_assert(RA == 2, "two tiles of 32 rows x 32 tokens, or of 64 x 16, for 32 tokens");
            auto sweep = [&](auto stage, auto leave) {
                SBN_WAIT_VMCNT(0);   // what was asked for of the next piece (the youngest half a step ago), in front of the first store
#pragma unroll
                for (int n = 0; n < RA * TB; ++n) {
                    stage(n);
                    leave(n);
                }
            };
            // Output rows of whole 64 bytes: tiles of 32 x 32, 128 bytes of a token at a time, written past the caches.  Where a run of
            // 128 bytes shares its 64-byte sectors with its neighbours, because rows have another length or the first does not begin
            // on 64 bytes, runs of 256 bytes (64 rows x 16 tokens) share half as many, and the L2 puts their halves together.  4096
            // tokens, 2560 -> 6920: 80 us in tiles past the caches, 64 in tiles, 66 in runs past the caches, 59.5 in runs (6924: 92 /
            // 66 / 69 / 61; 6912: 51 past the caches, 59 through them; 6912 behind 16 bytes, quantizer included: 108 in tiles past the
            // caches, 66 in runs).  Runs through the caches also where the rows of inputs are so short that the stores are all there is
            // to wait for and the caches hold them: tiles / runs at 8192 tokens 128 -> 6912 (226 MB) 49.8 / 39.7, 4096 tokens 256 ->
            // 4096 (67 MB) 16.9 / 16.1, 2851 tokens 256 -> 7632 24.8 / 20.6; but 16384 tokens 256 -> 4096 (268 MB) 54.1 / 55.2.
            const int64_t outputs = (int64_t)g.tokens * g.d_out;
            const bool short_rows = g.d_in <= 256 && outputs > (48 << 18) && outputs < (256 << 18);
            if ((g.d_out & 15) == 0 && (reinterpret_cast<uintptr_t>(g.Y) & 63) == 0 && !short_rows) {
                v4f bias4[RA];
                uint32_t voff[RA];
#pragma unroll
                for (int a = 0; a < RA; ++a) {
                    bias4[a] = bias_of(32 * a + 4 * (lane & 7));
                    voff[a] = offset((uint32_t)(lane >> 3) * pitch, 32 * a + 4 * (lane & 7));
                }
                sweep([&](const int n) {
                    const int a = n % RA, b = n / RA;
#pragma unroll
                    for (int q = 0; q < 4; ++q) *reinterpret_cast<v4f *>(est + r * 128 + 16 * ((2 * q + c) ^ ((r >> 1) & 7))) = rescaled(a, b, q);
                    asm volatile("" ::: "memory");   // the reads are of what other lanes have written
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int t = 8 * i + (lane >> 3);
                        yv[i] = *reinterpret_cast<const v4f *>(est + t * 128 + 16 * ((lane & 7) ^ ((t >> 1) & 7)));
                    }
                    asm volatile("" ::: "memory");   // the next tile's writes stay behind them
                }, [&](const int n) {
                    const int a = n % RA, b = n / RA;
                    if (has_bias) {
                        asm volatile("");   // a branch, not additions and selections
#pragma unroll
                        for (int i = 0; i < 4; ++i) yv[i] += bias4[a];
                    }
#pragma unroll
                    for (int i = 0; i < 4; ++i)
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, yv[i]), out, voff[a] + (uint32_t)(32 * b + 8 * i) * pitch, 0, 2);   // 2: streaming
                });
            } else {
                const v4f bias4 = bias_of(4 * (lane & 15));
                const uint32_t voff = offset((uint32_t)(lane >> 4) * pitch, 4 * (lane & 15));
                // Past the caches where the outputs would push out operands that are worth more, beyond 512 MB of them, of long rows
                // (through the caches / past them at 32768 tokens 2560 -> 6920 (907 MB) 460 / 421 us, 6912 -> 6920 919 / 803, 65536 tokens
                // 2560 -> 2568 (673 MB) 360 / 338; but 32768 tokens 2560 -> 2568 (337 MB) 174 / 176, 16384 tokens 2560 -> 6920 (454 MB)
                // 221 / 227, 32768 tokens 1024 -> 6920 315 / 333, 512 -> 6920 287 / 327, 512 -> 2568 86 / 124), and where there are so
                // few that the end of the launch waits for the caches to give them back, if no run ends within 32 bytes (2048 tokens 512
                // -> 2056 (17 MB) 9.9 / 9.0, 2000 tokens 2560 -> 2568 17.5 / 16.2, 3898 tokens 256 -> 888 7.75 / 7.5; but 4096 tokens
                // 512 -> 1496 (25 MB) 10.2 / 11.3, 4096 tokens 1024 -> 1000 (16 MB) 10.2 / 10.3).
                const bool halves = (g.d_out & 7) == 0 && (reinterpret_cast<uintptr_t>(g.Y) & 63) == 0;
                const bool streaming = (halves && outputs < (20 << 18)) || (g.d_in >= 2048 && outputs > (512 << 18));
                sweep([&](const int n) {
                    if ((r >> 4) == (n & 1)) {
#pragma unroll
                        for (int a = 0; a < RA; ++a)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
                                *reinterpret_cast<v4f *>(est + (r & 15) * 256 + 16 * ((8 * a + 2 * q + c) ^ (r & 15))) = rescaled(a, n / 2, q);
                    }
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const int t = 4 * i + (lane >> 4);
                        yv[i] = *reinterpret_cast<const v4f *>(est + t * 256 + 16 * ((lane & 15) ^ t));
                    }
                    asm volatile("" ::: "memory");
                }, [&](const int n) {
                    if (has_bias) {
                        asm volatile("");
#pragma unroll
                        for (int i = 0; i < 4; ++i) yv[i] += bias4;
                    }
                    if (streaming) {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, yv[i]), out, voff + (uint32_t)(16 * n + 4 * i) * pitch, 0, 2);
                    } else {
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, yv[i]), out, voff + (uint32_t)(16 * n + 4 * i) * pitch, 0, 0);
                    }
                });
            }
        } else {
            // Anything else: 32 tokens x 32 rows at a time into the staging area and out again a word per lane, two tokens side by side
            // (each lane its own values, a row of Y apart: 4096 tokens 2560 -> 6913 110 us, 57 this way, 8000 tokens 512 -> 6911 176 /
            // 58, 600 tokens 512 -> 1030 with accumulators 17.3 / 9.0).
            SBN_WAIT_VMCNT(0);
            int8_t *const est = lds + RING_BYTES + wave * STG_WAVE;
            const int8_t *const back = est + c * 128 + 4 * (r & 3);   // of token c; 2 i + c lies 256 i on, its granules swizzled with i & 7
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const float v = __fdiv_rn(gamma, sxv[b]);
                const int t = t0 + 32 * b + c, left = (g.tokens - t + 1) >> 1;
#pragma unroll
                for (int a = 0; a < RA; ++a) {
                    const int o = orow + 32 * a + r, steps = o < g.d_out ? (left < 16 ? left : 16) : 0;
                    const float bias = g.bias && o < g.d_out ? g.bias[o] : 0.0f;
                    const int64_t at = (int64_t)t * g.d_out + o;
                    auto sum = [&](const int i) { return UNIT ? acc[a][b][i] : acc[a][b][i] >> CODE_SHIFT; };
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<v4f *>(est + r * 128 + 16 * ((2 * q + c) ^ ((r >> 1) & 7))) =
                            v4f{(float)sum(4 * q) * v, (float)sum(4 * q + 1) * v, (float)sum(4 * q + 2) * v, (float)sum(4 * q + 3) * v};
                    asm volatile("" ::: "memory");   // the reads are of what other lanes have written
                    float *y = g.Y + at;
#pragma unroll 2
                    for (int i = 0; i < steps; ++i, y += 2 * (int64_t)g.d_out) {
                        const float value = *reinterpret_cast<const float *>(back + 256 * i + 16 * ((r >> 2) ^ (i & 7)));
                        *y = g.bias ? value + bias : value;
                    }
                    asm volatile("" ::: "memory");   // the next writes stay behind them
                    if (g.acc_out) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            *reinterpret_cast<v4i *>(est + r * 128 + 16 * ((2 * q + c) ^ ((r >> 1) & 7))) = v4i{sum(4 * q), sum(4 * q + 1), sum(4 * q + 2), sum(4 * q + 3)};
                        asm volatile("" ::: "memory");
                        int32_t *out = g.acc_out + at;
#pragma unroll 2
                        for (int i = 0; i < steps; ++i, out += 2 * (int64_t)g.d_out)
                            *out = *reinterpret_cast<const int32_t *>(back + 256 * i + 16 * ((r >> 2) ^ (i & 7)));
                        asm volatile("" ::: "memory");
                    }
                }
            }
        }
    } else {
        SBN_WAIT_VMCNT(0);
    }
}

template <int TB, bool DENSE, bool UNIT, class Group>
__device__ __forceinline__ void piece_live(const Group &grp, const Piece &p, const Piece &next, Stream &st, int8_t *lds, int wave, int lane)
{
    const bool live = p.to * ROWS + wave * (32 * RA) < grp.g[p.prob].d_out;   // a ragged last row tile leaves whole wavefronts idle
    if (live) piece_body<TB, true, DENSE, UNIT>(grp, p, next, st, lds, wave, lane);
    else piece_body<TB, false, DENSE, UNIT>(grp, p, next, st, lds, wave, lane);
}

template <bool DENSE, bool UNIT, class Group>
__device__ __forceinline__ void piece_run(const Group &grp, const Piece &p, const Piece &next, Stream &st, int8_t *lds, int wave, int lane)
{
    if (p.tb == 4) piece_live<4, DENSE, UNIT>(grp, p, next, st, lds, wave, lane);
    else if (p.tb == 3) piece_live<3, DENSE, UNIT>(grp, p, next, st, lds, wave, lane);
    else if (p.tb == 2) piece_live<2, DENSE, UNIT>(grp, p, next, st, lds, wave, lane);
    else piece_live<1, DENSE, UNIT>(grp, p, next, st, lds, wave, lane);
}

}  // namespace sp

// The work of a launch is counted in units of 512 rows x 32 tokens.  Blocks go round-robin to the 8 XCDs (each with
// its own 4 MB L2); XCD x owns the token units [x, x + 1) * ceil(units / 8) of every problem, cut into groups of 16
// units (512 tokens: their int8 activations stay in its L2 while the packed weights stream through once per group).
// A strip = (problem, group, row tile).  Launches small enough for a work list (made on the host, see
// make_piece_table) run the pieces listed for each block; larger ones give every block of an XCD a consecutive run of
// the XCD's units in the order strip, unit (the same number of units each, +-1), cut into pieces of at most four units
// that do not cross a strip.
// DENSE = the weights are dense 2-bit codes (the stored form of N = M, or any pattern converted to it) instead of 2:4.
// UNIT = the rows are longer than CODE_SHIFT_MAX_K: codes +-1, whose sums fit an int32 up to 2^24 values (2:4: 2^25).
template <bool DENSE, bool UNIT, class Group, class Table>
__global__ void __launch_bounds__(64 * sp::NW) gemm_smfmac_kernel(Group grp, Table tab)
{
    __shared__ __attribute__((aligned(1024))) int8_t lds[sp::LDS_BYTES];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const sp::Piece none{0, 0, 0, 0, 0};
    if constexpr (sizeof(Table) == sizeof(PieceTableNone)) {
        // Decode batches (every problem at most 16 token units): a piece = (problem, row tile, a share of the token
        // units of at most tab.piece[0] = 4, 2 or 1: the widest that still gives every multiprocessor a piece), in that
        // order, -per_block pieces in all.  XCD x runs the x-th of eight contiguous runs of them, as long as its share
        // of the blocks, and deals it to its blocks in contiguous runs, so the pieces of a row tile that has more than
        // one run side by side or one behind the other on one XCD, and its L2 fetches the tile's weights once.  With
        // run b for block b they sit on as many XCDs, each of which fetches them.  Both orders in turn: 2560 -> 6912 13.95 us
        // against 12.60 at 256 tokens and 14.56 against 13.60 at 512; twice that in one launch at 512 tokens 31.0 against
        // 23.1; eight layers of 2560 -> 2560 at 256 tokens 26.9 against 24.1 (dense codes, twice 6912 at 512: 33.3 against
        // 28.8).  A tile of one piece gains nothing and loses nothing (100 tokens: 12.2).  (From a graph, with the results
        // tile by tile, these take 11.5, 12.8, 22.2, 21.6, 29.1 and 11.1 by now.)  Dealing token units to XCDs, as below,
        // would leave most XCDs without work here.
        const int P = -tab.per_block, nbk = (int)gridDim.x, wmax = (int)tab.piece[0];
        const int x = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3, b8 = nbk >> 3, more8 = nbk & 7;
        const int before = x * b8 + (x < more8 ? x : more8), mine = b8 + (x < more8 ? 1 : 0);   // blocks of lower XCDs, of this one
        const int whole = P / nbk, part = P % nbk;
        const int run = whole * before + part * before / nbk;
        const int len = whole * (before + mine) + part * (before + mine) / nbk - run;
        const int q = len / mine, rem = len % mine;
        int f = run + j * q + (j < rem ? j : rem);
        const int end = f + q + (j < rem ? 1 : 0);
        int prob = 0, base = 0, parity = 0;
        auto piece_at = [&](int &f) {
            if (f >= end) return none;
            int units, groups;
            for (;;) {
                units = (grp.g[prob].tokens + 31) >> 5;
                groups = (units + wmax - 1) / wmax;
                const int cnt = ((grp.g[prob].d_out + sp::ROWS - 1) / sp::ROWS) * groups;
                if (f < base + cnt) break;
                base += cnt;
                ++prob;
            }
            const int local = f - base, to = local / groups, g = local % groups;
            const int wide = units / groups, more = units % groups;   // the first `more` shares hold one unit more
            ++f;
            parity ^= 1;
            return sp::Piece{prob, to, (g * wide + (g < more ? g : more)) * 32, wide + (g < more ? 1 : 0), parity};
        };
        sp::Piece cur = piece_at(f);
        if (cur.tb == 0) return;
        sp::Stream st = sp::first_stream(grp, cur, lds, wave, lane);
        while (cur.tb > 0) {
            const sp::Piece next = piece_at(f);
            sp::piece_run<DENSE, UNIT>(grp, cur, next, st, lds, wave, lane);
            cur = next;
        }
    } else {
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3, nb = gridDim.x >> 3;
    constexpr int GROUP_UNITS = 16;
    // units of problem p that XCD x owns: [x * upx, min((x + 1) * upx, units)), upx = ceil(units / 8)
    auto own_units = [&](int p, int &first) {
        const int units = (grp.g[p].tokens + 31) >> 5, upx = (units + 7) >> 3;
        first = x * upx;
        const int n = units - first;
        return n < 0 ? 0 : n < upx ? n : upx;
    };
    const bool listed = tab.per_block > 0;
    int total = 0;
    for (int p = 0; p < grp.count && !listed; ++p) {
        int first;
        total += (int)((grp.g[p].d_out + sp::ROWS - 1) / sp::ROWS) * own_units(p, first);
    }
    const int q = total / nb, rem = total % nb;
    int f = j * q + (j < rem ? j : rem);
    const int end = f + q + (j < rem ? 1 : 0);
    // Where the next piece starts: token unit u of a strip of gsz units from unit0 on, row tile `to` of tiles_o, group `group` of
    // problem `prob`, of which the XCD owns n units from `first` on.  Found once and then moved on without a division.
    int prob = 0, group = 0, to = 0, u = 0, first = 0, n = 0, gsz = 0, tiles_o = 0, parity = 0;
    auto enter_group = [&]() {   // the first group with units from (prob, group) on
        for (; prob < grp.count; ++prob, group = 0) {
            n = own_units(prob, first);
            gsz = n - group * GROUP_UNITS;
            gsz = gsz > GROUP_UNITS ? GROUP_UNITS : gsz;
            tiles_o = (grp.g[prob].d_out + sp::ROWS - 1) / sp::ROWS;
            if (gsz > 0) return;
        }
    };
    if (!listed && f < end) {
        int skip = f;   // units in front of the block's first
        for (enter_group(); skip >= tiles_o * gsz; ++group, enter_group()) skip -= tiles_o * gsz;
        to = skip / gsz;
        u = skip % gsz;
    }
    // the next piece of the block's list, whose pieces are listed without gaps (the first empty entry ends it), or the next by formula
    int entry = 0;
    auto piece_at = [&](int &f) {
        if (listed) {
            if (entry >= tab.per_block) return none;
            const uint32_t pc = tab.piece[blockIdx.x * tab.per_block + entry++];
            return sp::Piece{(int)(pc >> 25), (int)((pc >> 16) & 0x1ff), (int)((pc >> 3) & 0x1fff) * 32, (int)(pc & 7), entry & 1};
        }
        if (f >= end) return none;
        int w = gsz - u;
        w = w > 4 ? 4 : w;
        w = w > end - f ? end - f : w;
        f += w;
        parity ^= 1;
        const sp::Piece piece{prob, to, (first + group * GROUP_UNITS + u) * 32, w, parity};
        u += w;
        if (u == gsz) {
            u = 0;
            if (++to == tiles_o) {
                to = 0;
                ++group;
                enter_group();
            }
        }
        return piece;
    };
    sp::Piece cur = piece_at(f);
    if (cur.tb == 0) return;
    sp::Stream st = sp::first_stream(grp, cur, lds, wave, lane);
    while (cur.tb > 0) {
        const sp::Piece next = piece_at(f);
        sp::piece_run<DENSE, UNIT>(grp, cur, next, st, lds, wave, lane);
        cur = next;
    }
    }
}

// ---- dense comparison path ---------------------------------------------------------------------
// packed -> int8 W_eff with explicit zeros, one thread per group of four weights
__global__ void __launch_bounds__(256) expand_dense_kernel(const uint8_t *__restrict__ packed, int8_t *__restrict__ w,
                                                          int64_t ngroups)
{
    const int64_t gidx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (gidx >= ngroups) return;
    const int64_t chunk = gidx >> 5;
    const int gi = (int)(gidx & 31), word = gi >> 3, t = gi & 7;
    const uint32_t *cw = reinterpret_cast<const uint32_t *>(packed + chunk * 32);
    const uint32_t nib = (cw[word] >> (4 * t)) & 0xfu;
    const uint32_t codes = cw[4 + word];
    uint32_t out = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int v = 2 * t + h;
        const uint32_t code = (codes >> (8 * (v & 3) + 2 * (v >> 2))) & 3u;
        const uint32_t byte = code == 1u ? 0x01u : code == 3u ? 0xffu : 0u;
        const uint32_t pos = h ? (nib >> 2) : (nib & 3u);
        out |= byte << (8 * pos);
    }
    reinterpret_cast<uint32_t *>(w)[gidx] = out;
}

// Same block and wave shapes as the sparse kernel and the same LDS-DMA machinery, so that the two
// paths differ only in what the matrix instruction is fed: dense int8 rows with explicit zeros
// (no index register, no code expansion) into v_mfma_i32_32x32x32_i8, twice as many of them.
// Stage = 64 k of the 256 weight rows and 128 token rows (64-byte rows, 24 KB), ring of 3 stages;
// one DMA instruction fills 16 rows, 16-byte granules swizzled with (row >> 2) & 3.
constexpr int STAGES = 3;
constexpr int DK = 64;
constexpr int DSTAGE = (BO + BT) * DK;   // 24 KB

__global__ void __launch_bounds__(256, 2) gemm_dense_kernel(GemmArgs g)
{
    __shared__ __attribute__((aligned(1024))) int8_t lds[STAGES * DSTAGE];
    const uint32_t lds0 = lds_address(lds);
    int to, tt;
    tile_of_block(g, blockIdx.x, to, tt);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wo = wave & 1, wt = wave >> 1;
    const int r = lane & 31, c = lane >> 5;
    const int K = g.d_in, nk = K / DK;
    const int o0 = to * BO, t0 = tt * BT;

    const int8_t *const wbase = g.w_dense + (int64_t)o0 * K;
    const int8_t *const xbase = g.xq + (int64_t)t0 * K;
    uint32_t woff[4], xoff[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = (4 * wave + i) * 16 + (lane >> 2);
        const int o = o0 + row < g.d_out ? row : g.d_out - 1 - o0;
        woff[i] = (uint32_t)o * (uint32_t)K + 16u * ((lane & 3) ^ ((row >> 2) & 3));
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = (2 * wave + i) * 16 + (lane >> 2);
        const int t = t0 + row < g.tokens ? row : g.tokens - 1 - t0;
        xoff[i] = (uint32_t)t * (uint32_t)K + 16u * ((lane & 3) ^ ((row >> 2) & 3));
    }
    // lane (r, c) supplies k = 32u + 16c + 0..15 of the stage = granule 2u + c, for both operands;
    // row tile and ring stage are immediate offsets of the lane addresses below
    typedef __attribute__((address_space(3))) const v4i *lds_v4i;
    uint32_t aaddr[2], baddr[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int sw = (r >> 2) & 3;   // (row >> 2) & 3 with row = 32 a + r + a multiple of 64
        aaddr[u] = lds0 + (wo * 128 + r) * DK + 16 * ((2 * u + c) ^ sw);
        baddr[u] = lds0 + BO * DK + (wt * 64 + r) * DK + 16 * ((2 * u + c) ^ sw);
    }

    v16i acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[a][b][i] = 0;

    float sxv[3];
    load_scales<2>(g, t0 + wt * 64, lane, sxv);
    // Same software pipeline as the sparse kernel: ring of 3 stages, one barrier per iteration
    // between its two sub-steps, the DMA of stage kt+3 and the LDS reads of the next sub-step issued
    // between the matrix instructions, unconditional clamped DMA, stage as a literal.
    auto dma_one = [&](int kt, int stage, const int i) {   // i = 0..5: four weight and two token instructions
        const uint32_t dst = lds0 + stage * DSTAGE;
        if (i < 4) lds_dma16(wbase + (int64_t)kt * DK, woff[i], dst + (4 * wave + i) * 1024);
        else lds_dma16(xbase + (int64_t)kt * DK, xoff[i - 4], dst + BO * DK + (2 * wave + i - 4) * 1024);
    };
    auto dma = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < 6; ++i) dma_one(kt, stage, i);
    };
    v4i af[2][4], bf[2][2];
    auto read_a = [&](const int stage, const int u, const int a) {
        af[u][a] = *(lds_v4i)(uintptr_t)(aaddr[u] + stage * DSTAGE + 32 * a * DK);
    };
    auto read_b = [&](const int stage, const int u, const int b) {
        bf[u][b] = *(lds_v4i)(uintptr_t)(baddr[u] + stage * DSTAGE + 32 * b * DK);
    };
    auto mma = [&](const int u, const int a, const int b) {
        acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(af[u][a], bf[u][b], acc[a][b], 0, 0, 0);
    };
    dma(0, 0);
    dma(nk > 1 ? 1 : 0, 1);
    dma(nk > 2 ? 2 : nk - 1, 2);
    SBN_WAIT_VMCNT(12);   // stage 0 is in
    __syncthreads();
#pragma unroll
    for (int a = 0; a < 4; ++a) read_a(0, 0, a);
#pragma unroll
    for (int b = 0; b < 2; ++b) read_b(0, 0, b);
    auto iteration = [&](const int kt, const int stage) {   // stage = kt % 3 as a literal
        // sub-step 0; the six reads of sub-step 1 go out under its first matrix instructions
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mma(0, i >> 1, i & 1);
            if (i < 4) read_a(stage, 1, i);
            else if (i < 6) read_b(stage, 1, i - 4);
            __builtin_amdgcn_sched_barrier(0);
        }
        SBN_WAIT_VMCNT(6);   // stage kt+1 is in; stage kt+2 may fly
        __syncthreads();
        const int kf = kt + 3 < nk ? kt + 3 : nk - 1;
        const int nstage = stage == 2 ? 0 : stage + 1;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            mma(1, i >> 1, i & 1);
            if (i < 6) dma_one(kf, stage, i);
            if (i >= 2 && i < 6) read_a(nstage, 0, i - 2);
            else if (i >= 6) read_b(nstage, 0, i - 6);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const int nsteady = nk - 1;
    int kt = 0;
    for (; kt + 3 <= nsteady; kt += 3) {
        iteration(kt, 0);
        iteration(kt + 1, 1);
        iteration(kt + 2, 2);
    }
    if (kt < nsteady) { iteration(kt, 0); ++kt; }
    if (kt < nsteady) { iteration(kt, 1); ++kt; }
    {
        const int stage = kt % STAGES;
#pragma unroll
        for (int a = 0; a < 4; ++a) af[1][a] = *(lds_v4i)(uintptr_t)(aaddr[1] + stage * DSTAGE + 32 * a * DK);
#pragma unroll
        for (int b = 0; b < 2; ++b) bf[1][b] = *(lds_v4i)(uintptr_t)(baddr[1] + stage * DSTAGE + 32 * b * DK);
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int i = 0; i < 8; ++i) mma(u, i >> 1, i & 1);
    }
    SBN_WAIT_VMCNT(0);   // surplus DMA of the last iterations must not land in the epilogue's staging area
    block_epilogue<4, 2>(g, acc, sxv, lds, o0, o0 + wo * 128, t0 + wt * 64, wave, lane);
}

GemmArgs make_args(const LinearItem &it, int block_tokens = BT)
{
    GemmArgs g;
    g.xq = it.xq; g.sx = it.sx; g.packed = static_cast<const uint8_t *>(it.packed); g.w_dense = nullptr;
    g.gamma = it.gamma; g.bias = it.bias; g.Y = it.Y; g.acc_out = it.acc_out;
    g.tokens = (int)it.tokens; g.d_in = (int)it.d_in; g.d_out = (int)it.d_out;
    g.tiles_o = (int)ceil_div(it.d_out, BO);
    g.tiles_t = (int)ceil_div(it.tokens, block_tokens);
    return g;
}

}  // namespace

// Deals the work of a launch to the blocks (host side).  Per XCD: the strips (problem, token group of 16 units, row
// tile of 512) are cut into exactly m * nb pieces of at most four units, as even as the strip lengths allow (no block
// is left with single-unit crumbs: a piece of one unit pays a whole expansion per matrix instruction).  The
// pieces stay in strip order and are dealt in m rounds of nb: the pieces that run at about the same time belong to a
// few neighbouring strips, whose weights and tokens fit the XCD's L2 together (dealt by width alone, across all strips,
// the same launch fetched 88 MB instead of 50 at 6912 x 2560 x 4096).  Inside a round the widest pieces go to the
// blocks with the least work so far, so every block ends up with the same number of units (+-1).  Odd XCDs run their
// rounds in reverse order, so that the chip's XCDs do not all reach their epilogues (bursts of Y stores) together.
// Returns blocks per XCD; leaves tab.per_block = 0 (formula split in the kernel) when the list would not fit.
static int make_piece_table(const GemmGroup &grp, PieceTable &tab)
{
    constexpr int GROUP_UNITS = 16;
    struct Strip { int prob, to, unit0, len, npieces; };
    static thread_local std::vector<Strip> strips;
    static thread_local std::vector<uint32_t> pieces;
    static thread_local std::vector<std::vector<uint32_t>> per_block;
    int nb = device_cus() / 8;
    nb = nb < 1 ? 1 : nb;
    int most = 0;   // units of the XCD with the most work
    for (int x = 0; x < 8; ++x) {
        int total = 0;
        for (int p = 0; p < grp.count; ++p) {
            const int units = (grp.g[p].tokens + 31) / 32, upx = (units + 7) / 8;
            const int n = units - x * upx;
            total += (int)ceil_div(grp.g[p].d_out, sp::ROWS) * (n < 0 ? 0 : n < upx ? n : upx);
        }
        most = total > most ? total : most;
    }
    nb = most < nb ? most : nb;
    nb = nb < 1 ? 1 : nb;
    const int m = (int)ceil_div(ceil_div(most, nb), 4);   // pieces per block: the busiest XCD's units per block, four at a time
    tab.per_block = 0;
    if (m * nb * 8 > PIECE_TABLE_MAX) return nb;
    for (int i = 0; i < m * nb * 8; ++i) tab.piece[i] = 0;
    per_block.resize(nb);
    for (int x = 0; x < 8; ++x) {
        strips.clear();
        int minpieces = 0;
        for (int p = 0; p < grp.count; ++p) {
            const int units = (grp.g[p].tokens + 31) / 32, upx = (units + 7) / 8;
            int n = units - x * upx;
            n = n < 0 ? 0 : n < upx ? n : upx;
            const int tiles_o = (int)ceil_div(grp.g[p].d_out, sp::ROWS);
            for (int g0 = 0; g0 < n; g0 += GROUP_UNITS)
                for (int to = 0; to < tiles_o; ++to) {
                    const int len = n - g0 < GROUP_UNITS ? n - g0 : GROUP_UNITS;
                    strips.push_back(Strip{p, to, x * upx + g0, len, (len + 3) / 4});
                    minpieces += (len + 3) / 4;
                }
        }
        if (strips.empty()) continue;
        // more pieces than the minimum: cut the strips with the widest pieces finer, one more piece at a time
        int extra = m * nb - minpieces;
        while (extra > 0) {
            int best = -1;
            for (size_t i = 0; i < strips.size(); ++i)
                if (strips[i].npieces < strips[i].len &&
                    (best < 0 || strips[i].len * strips[best].npieces > strips[best].len * strips[i].npieces))
                    best = (int)i;
            if (best < 0) break;
            ++strips[best].npieces;
            --extra;
        }
        pieces.clear();
        for (const Strip &st : strips) {
            int u = 0;
            for (int k = 0; k < st.npieces; ++k) {
                const int w = st.len / st.npieces + (k < st.len % st.npieces ? 1 : 0);
                pieces.push_back((uint32_t)w | ((uint32_t)(st.unit0 + u) << 3) | ((uint32_t)st.to << 16) | ((uint32_t)st.prob << 25));
                u += w;
            }
        }
        // Pieces stay in strip order: round i (the i-th piece of every block, roughly the same stretch of time) takes
        // the pieces [i * nb, (i + 1) * nb), i.e. a few neighbouring strips whose weights and tokens fit the XCD's L2
        // together.  Inside a round the widest pieces go to the blocks with the least work so far.
        for (int j = 0; j < nb; ++j) per_block[j].clear();
        static thread_local std::vector<int> load, by_load, by_width;
        load.assign(nb, 0);
        const int rounds = ((int)pieces.size() + nb - 1) / nb;
        if (rounds > m) return nb;   // cannot happen: the strips were cut into at most m * nb pieces
        for (int i = 0; i < rounds; ++i) {
            const int first = i * nb, n = (int)pieces.size() - first < nb ? (int)pieces.size() - first : nb;
            by_width.resize(n);
            for (int k = 0; k < n; ++k) by_width[k] = first + k;
            std::stable_sort(by_width.begin(), by_width.end(), [&](int a, int b) { return (pieces[a] & 7) > (pieces[b] & 7); });
            by_load.resize(nb);
            for (int j = 0; j < nb; ++j) by_load[j] = j;
            std::stable_sort(by_load.begin(), by_load.end(), [&](int a, int b) { return load[a] < load[b]; });
            for (int k = 0; k < n; ++k) {
                per_block[by_load[k]].push_back(pieces[by_width[k]]);
                load[by_load[k]] += (int)(pieces[by_width[k]] & 7);
            }
        }
        for (int j = 0; j < nb; ++j) {
            std::vector<uint32_t> &l = per_block[j];
            if (x & 1) std::reverse(l.begin(), l.end());   // odd XCDs run their rounds last to first
            for (size_t i = 0; i < l.size(); ++i) tab.piece[(size_t)(j * 8 + x) * m + i] = l[i];
        }
    }
    tab.per_block = m;
    return nb;
}

sbn_status launch_gemm_pieces(int count, const LinearItem *items, bool dense_codes, hipStream_t stream)
{
    for (int i = 0; i < count; ++i)
        if (items[i].d_in >= sp::ROW_END) return SBN_EUNSUPPORTED;
    // problems of at most 16 token units (512 tokens: decode batches) are dealt by row tile, up to GEMM_GROUP_WIDE per launch
    auto few_tokens = [&](int i) { return items[i].tokens <= 16 * 32 && items[i].d_in <= CODE_SHIFT_MAX_K; };
    auto long_rows = [&](int i) { return items[i].d_in > CODE_SHIFT_MAX_K; };   // a kernel of their own
    for (int first = 0; first < count;) {
        const bool few = few_tokens(first);
        const int most = few ? GEMM_GROUP_WIDE : GEMM_GROUP_MAX;
        int n = 1;
        while (first + n < count && n < most && few_tokens(first + n) == few && long_rows(first + n) == long_rows(first)) ++n;
        if (few) {
            GemmGroupWide grp;
            grp.count = n;
            for (int i = 0; i < n; ++i) grp.g[i] = make_args(items[first + i]);
            // pieces of four token units feed the matrix pipe best; a launch with fewer pieces than multiprocessors (one
            // layer of a decode step) is cut finer, down to single units, so that its latency is that of a small piece
            int wmax = 4, pieces = 0;
            for (;; wmax >>= 1) {
                pieces = 0;
                for (int i = 0; i < n; ++i)
                    pieces += (int)ceil_div(items[first + i].d_out, sp::ROWS) * (int)ceil_div(ceil_div(items[first + i].tokens, 32), wmax);
                if (wmax == 1 || pieces >= device_cus()) break;
            }
            PieceTableNone tab;
            tab.per_block = -pieces;
            tab.piece[0] = (uint32_t)wmax;
            const int blocks = pieces < device_cus() ? pieces : device_cus();
            if (dense_codes) hipLaunchKernelGGL((gemm_smfmac_kernel<true, false, GemmGroupWide, PieceTableNone>), dim3(blocks), dim3(64 * sp::NW), 0, stream, grp, tab);
            else hipLaunchKernelGGL((gemm_smfmac_kernel<false, false, GemmGroupWide, PieceTableNone>), dim3(blocks), dim3(64 * sp::NW), 0, stream, grp, tab);
        } else {
            GemmGroup grp;
            grp.count = n;
            for (int i = 0; i < n; ++i) grp.g[i] = make_args(items[first + i]);
            static thread_local PieceTable tab;
            const int per_xcd = make_piece_table(grp, tab);
            auto launch = [&](auto dense, auto unit) {
                hipLaunchKernelGGL((gemm_smfmac_kernel<dense(), unit(), GemmGroup, PieceTable>), dim3(8 * per_xcd), dim3(64 * sp::NW), 0, stream, grp, tab);
            };
            if (long_rows(first)) {
                if (dense_codes) launch(std::true_type(), std::true_type());
                else launch(std::false_type(), std::true_type());
            } else {
                if (dense_codes) launch(std::true_type(), std::false_type());
                else launch(std::false_type(), std::false_type());
            }
        }
        sbn_status st = check_launch("gemm_smfmac_kernel");
        if (st != SBN_OK) return st;
        first += n;
    }
    return SBN_OK;
}

// Estimated time in us of a call on the streaming kernel or the pieces, next to which gemm_tile_estimate_us stands; every
// problem counts with its own input dimension.  Measured behind the quantizer, weights from memory, quantizer not included:
//   streaming kernel (<= 64 tokens)  one strip of 128 rows per block: 4 us + 5 us (up to 32 tokens) or 8.5 us per 2560 weights
//       of the input dimension; strips of 256 rows: 12.5 or 17.5 us per round of the device
//       (16 x (2560 -> 6912) at 32 / 64 tokens: 26 / 34 us; one layer alone 10 / 14, 6912 -> 2560 18 / 27)
//   pieces of 512 rows x 32 .. 128 tokens  3.9 us, 10.5 us (dense codes 14.5) per 2560 weights of the deepest problem, 0.75 of
//       that for each further unit of 32 tokens a multiprocessor has, 0.11 us per MB of outputs
//       (2560 -> 2560 at 17 .. 1500 tokens 13.2 .. 15.0 us, 6912 -> 2560 39 .. 43, 2560 -> 6912 at 512 / 777 / 1500 / 3000
//       tokens, up to 1 / 2 / 3 / 6 units, 18 / 20 / 25 / 47).  Output rows of no whole 16 bytes are stored in single words,
//       another 3.2 us and 0.55 us per MB of them (512 -> 476 / 478 at 1000 tokens 6.5 / 10.2 us, 512 -> 6911 at 8000 179)
// The fit is of pieces before their requests ran on, decode batches were dealt by XCD and odd widths left through LDS.  By name, without
// the quantizer, 2560 -> 6912 takes 18.9 us at 1024 tokens and 365 at 32768 by now, where this says 23 and 547, and 512 -> 6911 at
// 8000 tokens 60, so that the choice leans to the small tiles: a little where d_out % 4 is 0, much where it is not.
static float gemm_large_estimate_us(int count, const LinearItem *items, bool dense)
{
    bool stream = true;
    int64_t strips = 0, tokens = 0, depth = 0;
    double units = 0, out_mb = 0, word_mb = 0;   // units weighted with their input dimension; outputs, those stored in words
    for (int i = 0; i < count; ++i) {
        const LinearItem &li = items[i];
        stream = stream && gemv_batch_takes(li);
        strips += ceil_div(li.d_out, 256);
        units += (double)(ceil_div(li.d_out, sp::ROWS) * ceil_div(li.tokens, 32)) * (double)li.d_in / 2560.0;
        out_mb += 4e-6 * (double)li.tokens * (double)li.d_out;
        if (li.d_out % 4 != 0) word_mb += 4e-6 * (double)li.tokens * (double)li.d_out;
        tokens = li.tokens > tokens ? li.tokens : tokens;
        depth = li.d_in > depth ? li.d_in : depth;
    }
    const float k = (float)depth / 2560.0f;
    const int cus = device_cus();
    if (stream) {
        if (strips < cus) return 4.0f + k * (tokens <= 32 ? 5.0f : 8.5f);
        return 4.0f + k * (tokens <= 32 ? 12.5f : 17.5f) * (float)strips / (float)cus;
    }
    const float more = (float)units / (float)cus - k;
    // (768 -> 6912 at 16384 tokens and 8192 -> 768 at 17 in one call: 278 us as small tiles, 158 this way, quantizers included)
    return 3.9f + (dense ? 14.5f : 10.5f) * (k + 0.75f * (more > 0.0f ? more : 0.0f)) + 0.11f * (float)out_mb +
           (word_mb > 0.0 ? 3.2f + 0.55f * (float)word_mb : 0.0f);
}

// Rows longer than the pieces can address; a block tile addresses 64 of them, a small tile 32.
static bool beyond_pieces(int count, const LinearItem *items)
{
    for (int i = 0; i < count; ++i)
        if (items[i].d_in >= sp::ROW_END && !gemv_batch_takes(items[i])) return true;
    return false;
}

// Small block tiles where they are faster: their time grows with rows x tokens from 4.5 us on, that of the large kernels
// starts two to five times higher and grows slower.  Over 279 calls of 17 to 16384 tokens, input dimensions 256 to 8192 and
// one to sixteen problems, all kernels measured, the choice costs 0.6 % against the faster kernel of each (at worst 1.40, 384 tokens
// 4096 -> 14336 with dense codes: 56 us against 40); 256 tokens, 2560 -> 6912: 13.5 us in tiles, 17.8 in pieces as they were
// then (11.5 by name by now); 512 tokens, 2560 -> 2560: 11.1 / 14.0 (11.3); 777 tokens: 14.9 / 13.8 (11.7).  Over 365 calls more of 200 to 8000 tokens with 475 to 6912 outputs, most
// of them no multiple of four: 0.2 %, at worst 1.09 (8000 tokens, 512 -> 1500: 23 / 25 us); 2181 tokens, 512 -> 475 7.6 in tiles,
// 11.4 in pieces (7.2), 512 -> 512 6.9 either way (6.3).
bool gemm_takes_tiles(int count, const LinearItem *items, bool dense_codes)
{
    return beyond_pieces(count, items) || gemm_tile_estimate_us(count, items, dense_codes) < gemm_large_estimate_us(count, items, dense_codes);
}

float gemm_estimate_us(int count, const LinearItem *items, bool dense_codes)
{
    return std::min(gemm_block_estimate_us(count, items, dense_codes),
                    std::min(gemm_tile_estimate_us(count, items, dense_codes), gemm_large_estimate_us(count, items, dense_codes)));
}

// Block tiles of middle size where they are faster by more than the estimates are off: over 220 calls of 96 to 2048 tokens through
// eleven layers, 2:4 and dense codes, all kernels measured, they are taken for 70 and are 1.14 times as fast there (at worst 0.93,
// 256 tokens 2560 -> 1000: 6.2 us against 5.7; at best 1.35, 640 tokens 6912 -> 2560: 17.6 against 23.7).  Of 420 others, whole calls of
// 17 to 2500 tokens, 69 take them, in 0.84 of the time of tiles and pieces; two are slower by more than 2 % (55 tokens, 4608 -> 3 x 2984
// 13.6 us against 12.3).
bool gemm_takes_blocks(int count, const LinearItem *items, bool dense_codes)
{
    return !beyond_pieces(count, items) && gemm_block_estimate_us(count, items, dense_codes) <
           0.95f * std::min(gemm_tile_estimate_us(count, items, dense_codes), gemm_large_estimate_us(count, items, dense_codes));
}

sbn_status launch_gemm_smfmac(int count, const LinearItem *items, bool dense_codes, hipStream_t stream)
{
    if (gemm_takes_blocks(count, items, dense_codes)) return launch_gemm_block(count, items, dense_codes, stream);
    if (gemm_takes_tiles(count, items, dense_codes)) return launch_gemm_tile(count, items, dense_codes, stream);
    for (int first = 0; first < count;) {
        const bool streams = gemv_batch_takes(items[first]);
        int n = 1;
        while (first + n < count && gemv_batch_takes(items[first + n]) == streams) ++n;
        sbn_status st = streams ? launch_gemv_batch(n, items + first, dense_codes, stream) : launch_gemm_pieces(n, items + first, dense_codes, stream);
        if (st != SBN_OK) return st;
        first += n;
    }
    return SBN_OK;
}

sbn_status launch_gemm_dense_expanded(const LinearItem &it, const int8_t *w_dense, hipStream_t stream)
{
    GemmArgs g = make_args(it);
    g.w_dense = w_dense;
    hipLaunchKernelGGL(gemm_dense_kernel, dim3(g.tiles_o * g.tiles_t), dim3(256), 0, stream, g);
    return check_launch("gemm_dense_kernel");
}

sbn_status launch_gemm_dense(const LinearItem &it, const Pattern &pat, int8_t *w_dense, hipStream_t stream)
{
    sbn_status st;
    if (pat.N == 2 && pat.M == 4 && it.d_in % CHUNK == 0) {
        const int64_t ngroups = it.d_out * it.d_in / 4;
        hipLaunchKernelGGL(expand_dense_kernel, dim3((unsigned)ceil_div(ngroups, 256)), dim3(256), 0, stream,
                           static_cast<const uint8_t *>(it.packed), w_dense, ngroups);
        st = check_launch("expand_dense_kernel");
    } else {
        // any other pattern (6:8, 2:8, 1:4, ...): the format-generic group decoder writes the same int8 W_eff
        st = launch_expand_groups(it.packed, it.d_out, it.d_in, pat, w_dense, stream);
    }
    if (st != SBN_OK) return st;
    return launch_gemm_dense_expanded(it, w_dense, stream);
}

}  // namespace sbn
