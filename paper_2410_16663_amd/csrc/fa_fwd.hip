// Exact attention forward for gfx950 (MI355X): kernels and the C ABI of include/fa.h.
//
// Dataflow (FastAttention appendix A, the FlashAttention2 forward): for each block of
// queries, walk the key/value blocks once; per block compute the logits on the matrix
// cores, exponentiate against a running reference, multiply by V on the matrix cores,
// and carry the reference / row sum.  Mask handling follows section 4.1: blocks that are
// entirely masked are skipped, blocks that are entirely visible take no mask, and only the
// others get a per-element predicate computed from indices -- no mask tensor exists.
//
// Where things are (the .inc files are fragments of this one translation unit, included below):
//  * fa_row_tile.inc -- one wave's rows and the work of one tile on them, for fa_fwd_kernel.
//  * fa_attention_kernel.inc -- fa_fwd_kernel, the attention kernel, one source for most variants (template
//    flags): WIDE (all NW waves walk the same tiles: 256 query rows with eight, 128 with four) or split (128 rows,
//    two groups of four waves on alternate tiles, merged through LDS); CAUSAL; PAIR (folded rows for short causal
//    problems); SPLITKV (one run of the key tiles per workgroup, unnormalised result to a workspace); GENMASK
//    (window / prefix / key-count masks from a descriptor).  Entry points fa_fwd, fa_fwd_splitkv, fa_fwd_masked.
//  * fa_attention_wide64_kernel.inc -- fa_fwd_wide64_kernel, long walks at D = 128: 64 query rows per wave.
//  * fa_attention_rows_kernel.inc -- fa_fwd_rows_kernel, D = 128 problems of short and middle length: persistent
//    workgroups of four waves that take 128-row blocks from a balanced list.
//  * fa_decode_kernels.inc -- fa_decode_kernel, the single-query decoding step with K/V streamed through
//    registers, and fa_combine_kernel, which merges the split-KV runs.
//  * fa_linear_kernel.inc -- the output projection that follows the attention block by block (section 4.2),
//    entry points fa_attn_linear_block / fa_attn_linear.
//  * fa_mask.inc -- descriptor masks: tile classification and walk, shared by the kernel and the host entry
//    points fa_mask_*.
//  * fa_types.inc, fa_device.inc -- vector types and parameter block; device helpers (LDS swizzles,
//    global-to-LDS load, cross-half exchange).
//  * this file -- the host side: argument checks, choice of decomposition, launch shapes, the C ABI.
//
// gfx950 mapping common to all variants of the attention kernel (this library's own design):
//  * one wavefront owns 32 query rows; a SIMD holds two wavefronts, of one workgroup of eight or of two
//    workgroups of four.  Each wavefront runs a tile as three clusters (logits, softmax, second
//    product), or with the softmax dealt out among the products (fa_row_tile.inc).  In clusters the overlap of the matrix
//    and vector units comes mostly from the two wavefronts of a SIMD being in different ones; those of a workgroup run
//    free between its one barrier per tile.
//  * logits are produced TRANSPOSED, S^T = K Q^T, with v_mfma_f32_16x16x32 (v_mfma_f32_32x32x16 where few workgroups are
//    bound by their chain of tiles): keys on the M side (A operand, read from LDS with ds_read_b128), queries on the N
//    side (B operand, held in registers for the whole kernel).  A lane then owns one query column or two, so row
//    max / row sum are in-lane reductions plus exchanges between four lanes or two (v_permlane32_swap,
//    v_permlane16_swap), and the exponentiated tile is already in the
//    B-operand register layout of the second product O^T = V^T P^T (no shuffle, no LDS
//    round trip -- the MFMA counterpart of the paper's appendix-B layout converter).
//  * V^T fragments come straight out of the row-major V tile with the transposing LDS
//    read ds_read_b64_tr_b16.
//  * K and V tiles (64 keys) go from global memory straight into LDS (global_load_lds),
//    double-buffered (three-deep for split-KV), bank-swizzled on the global side.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <sys/random.h>

#include <atomic>
#include <chrono>
#include <mutex>
#include <type_traits>
#include <utility>

#include "../../include/fa.h"

// Workspace of fa_fwd_splitkv_static: the split-KV partial results of callers that cannot pass a workspace of their
// own.  Every GPU the library's code object is loaded on holds its own copy at its own address, until the process
// ends.  In host code this name is only a handle for hipGetSymbolAddress, never a device address.
#define FA_STATIC_WORKSPACE_BYTES (64ll << 20)
static __device__ __align__(256) unsigned char scratch[FA_STATIC_WORKSPACE_BYTES];

namespace {

#include "fa_types.inc"
#include "fa_mask.inc"
#include "fa_device.inc"
#include "fa_row_tile.inc"
#include "fa_attention_kernel.inc"
#include "fa_attention_wide64_kernel.inc"
#include "fa_attention_rows_kernel.inc"
#include "fa_linear_kernel.inc"
#include "fa_decode_kernels.inc"

template <int DT, int D, bool CAUSAL, bool WIDE, int NW = 8, bool TWO_SUMS = DT == FA_DTYPE_BF16>
hipError_t launch(const FaParams &p, int nwork_padded, hipStream_t stream) {
    hipLaunchKernelGGL((fa_fwd_kernel<DT, D, CAUSAL, WIDE, false, false, false, NW, TWO_SUMS>), dim3(nwork_padded), dim3(NW * 64), 0,
                       stream, p);
    return hipGetLastError();
}

// descriptor masks, on workgroups of four waves (128 query rows) or eight (256)
template <int DT, int D>
hipError_t launch_masked(const FaParams &p, int rows, int nwork_padded, hipStream_t stream) {
    if (rows == 128) hipLaunchKernelGGL((fa_fwd_kernel<DT, D, false, true, false, true, false, 4>), dim3(nwork_padded), dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((fa_fwd_kernel<DT, D, false, true, false, true, false, 8>), dim3(nwork_padded), dim3(512), 0, stream, p);
    return hipGetLastError();
}

// fa_fwd_rows_kernel: p holds the whole problem (nqt 128-row blocks per head); the shape of the list is set here, and as
// many workgroups are launched as the chip holds at a time (two per compute unit), fewer if the list is shorter. The order
// of the list balances causal work: with all heads of an XCD mixed, heaviest row blocks first, the largest share is within
// 5% of the mean where a workgroup has many blocks, and one heaviest block where it has one or two (3 x 20 x 1531: 24 tiles,
// the mean 18.4; 40 and 36.8 on a compute unit's two workgroups) (1 x 40 x 4096: 199 us head by head, 171 mixed; 20 heads of
// 8192: 382, 329; 96 of 2048: 117, 112).  Two exceptions, for the sake of the L2, where the workgroups that run at a time
// should share K/V: up to four row blocks per head (512 heads of 512 rows: 62 head by head, 81 mixed), and more heads per
// XCD than 16 over at least four turns, which are mixed in groups of eight.
constexpr int ROWS_SLOTS = 64;                     // workgroups an XCD's 32 compute units hold at a time
long long rows_entries(long long heads, long long nqt) { return heads / 8 * nqt + (heads % 8 * nqt + 7) / 8; }   // of XCD 0
int rows_grid(long long heads, long long nqt) {
    const long long n = rows_entries(heads, nqt);
    return 8 * (int)(n < ROWS_SLOTS ? n : ROWS_SLOTS);
}
hipError_t launch_rows(FaParams p, int dtype, bool causal, hipStream_t stream) {
    const int heads = p.nwork / p.nqt;
    const long long entries = rows_entries(heads, p.nqt);
    p.head_run = heads / 8;
    p.head_rest = heads % 8;
    if (!causal || p.nqt < 5) {
        p.group = 1;
        p.grouped = p.head_run;
    } else {
        p.group = 8;
        p.grouped = p.head_run <= 16 || entries < 4 * ROWS_SLOTS ? 0 : p.head_run & ~7;
    }
    if (!causal) p.off = p.Nk - 1;                 // the diagonal past every key
    const dim3 grid(rows_grid(heads, p.nqt));
    if (dtype == FA_DTYPE_F16) hipLaunchKernelGGL((fa_fwd_rows_kernel<FA_DTYPE_F16>), grid, dim3(256), 0, stream, p);
    else hipLaunchKernelGGL((fa_fwd_rows_kernel<FA_DTYPE_BF16>), grid, dim3(256), 0, stream, p);
    return hipGetLastError();
}

template <int DT, int D, bool CAUSAL>
hipError_t launch_splitkv(const FaParams &p, int nwork_padded, long long rows, bool long_runs, hipStream_t stream) {
    // long runs of a compute-bound shape (several query blocks per head) at D = 128: the 64-row waves with the
    // pipelined loop; everything else the tile kernel's split-KV instantiation, which is tuned for streaming K/V
    if constexpr (D == 128) {
        if (long_runs)
            hipLaunchKernelGGL((fa_fwd_wide64_kernel<DT, CAUSAL, true>), dim3(nwork_padded, p.nsplit), dim3(256), 0, stream, p);
        else
            hipLaunchKernelGGL((fa_fwd_kernel<DT, D, CAUSAL, true, true>), dim3(nwork_padded, p.nsplit), dim3(512), 0, stream, p);
    } else {
        hipLaunchKernelGGL((fa_fwd_kernel<DT, D, CAUSAL, true, true>), dim3(nwork_padded, p.nsplit), dim3(512), 0, stream, p);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    constexpr int RPB = 256 / (D / 4);            // rows per combine block
    hipLaunchKernelGGL((fa_combine_kernel<DT, D>), dim3((unsigned)((rows + RPB - 1) / RPB)), dim3(256), 0, stream,
                       p.part_o, p.part_ml, p.o, p.lse, rows, p.nsplit, 0u, 0u);
    return hipGetLastError();
}

// single query; p.stream_wgs pieces, or p.nsplit runs of each head
template <int DT, int D>
hipError_t launch_decode(const FaParams &p, int heads, long long rows, hipStream_t stream) {
    const dim3 block(DECODE_WAVES * 64);
    if (p.stream_wgs > 0) hipLaunchKernelGGL((fa_decode_kernel<DT, D, false, true>), dim3(p.stream_wgs), block, 0, stream, p);
    else if (p.tag != 0) hipLaunchKernelGGL((fa_decode_kernel<DT, D, false, false, true>), dim3(heads, p.nsplit), block, 0, stream, p);
    else hipLaunchKernelGGL((fa_decode_kernel<DT, D>), dim3(heads, p.nsplit), block, 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.nsplit == 1 || p.tag != 0) return e;   // a single run stores o and lse itself, and so does the last of several
    constexpr int RPB = 256 / (D / 4);
    hipLaunchKernelGGL((fa_combine_kernel<DT, D>), dim3((unsigned)((rows + RPB - 1) / RPB)), dim3(256), 0, stream,
                       p.part_o, p.part_ml, p.o, p.lse, rows, p.nsplit, (unsigned)((p.Nk + BN - 1) / BN), (unsigned)p.stream_wgs);
    return hipGetLastError();
}

// single query under a mask descriptor: p.nsplit workgroups per (batch, head); a single one stores o and lse itself
template <int DT, int D>
hipError_t launch_decode_masked(const FaParams &p, int heads, hipStream_t stream) {
    const dim3 grid(heads, p.nsplit), block(DECODE_WAVES * 64);
    if (p.tag != 0) hipLaunchKernelGGL((fa_decode_kernel<DT, D, true, false, true>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((fa_decode_kernel<DT, D, true>), grid, block, 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.nsplit == 1 || p.tag != 0) return e;
    constexpr int RPB = 256 / (D / 4);
    hipLaunchKernelGGL((fa_combine_kernel<DT, D>), dim3((unsigned)((heads + RPB - 1) / RPB)), dim3(256), 0, stream,
                       p.part_o, p.part_ml, p.o, p.lse, (long long)heads, p.nsplit, 0u, 0u);
    return hipGetLastError();
}

thread_local int g_last_hip_error = 0;

// Where the count behind decode_tag starts: random, so that two processes' tags differ.  (Not std::random_device, which throws where
// it finds no source, through the C entry points; here the clock is left then.)
unsigned long long tag_seed() noexcept {
    unsigned long long x;
    if (getrandom(&x, sizeof x, GRND_NONBLOCK) != (ssize_t)sizeof x) x = 0;
    return x + (unsigned long long)std::chrono::system_clock::now().time_since_epoch().count();
}
// Whether fa_decode_kernel merges the runs of a head, `runs` of them at most, by itself: their tags fit into a row of o
bool merges_itself(int runs, int D) { return runs > 1 && runs <= D / 4; }
// FaParams::tag of a call that does: 64 bits that no other memory holds by chance.  Every call of the process gets a value of its
// own, so that what an earlier one left in o is not taken for a mark.  A captured call's value is an argument of its node, the same
// on every replay: a replay leaves none of its marks behind, because the kernel does not end before every head of several runs has
// its marks replaced by the result.
unsigned long long decode_tag() noexcept {
    static std::atomic<unsigned long long> calls{tag_seed()};
    unsigned long long x = calls.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);   // (SplitMix64: a bijection)
    x = (x ^ (x >> 30)) * 0xbf58476d1ce4e5b9ull;
    x = (x ^ (x >> 27)) * 0x94d049bb133111ebull;
    x ^= x >> 31;
    return x != 0 ? x : 1;
}

// fa_set_option's values (FA_AUTO: the library chooses).  Every entry point takes them once, when it is called, and hands that copy
// on: a call that launches several kernels, or chooses twice, chooses by the same values throughout.
std::atomic<int> g_options[5] = {{FA_AUTO}, {FA_AUTO}, {FA_AUTO}, {FA_AUTO}, {FA_AUTO}};
struct Options {
    int value[5];
    int operator[](int which) const { return value[which]; }
};
Options options_now() {
    Options opt;
    for (int i = 0; i < 5; ++i) opt.value[i] = g_options[i].load(std::memory_order_relaxed);
    return opt;
}

// Shape checks shared by fa_fwd and fa_fwd_plan; everything here runs before any HIP call.
int check_shape(int B, int H, int Nq, int Nk, int D, int dtype) {
    if (B <= 0 || H <= 0 || Nq <= 0 || Nk <= 0) return FA_ERR_SHAPE;
    if (D != 64 && D != 128) return FA_ERR_HEADDIM;
    if (dtype != FA_DTYPE_F16 && dtype != FA_DTYPE_BF16) return FA_ERR_DTYPE;
    if ((long long)B * H > 0x7fffffffLL) return FA_ERR_SHAPE;
    if ((long long)B * H * (((long long)Nq + 127) / 128) > 0x7ffffff0LL) return FA_ERR_SHAPE;   // grid size
    if ((long long)Nq + Nk > 0x7fffff00LL) return FA_ERR_SHAPE;                                   // int index arithmetic
    if ((long long)Nk * D * 2 > 0x7fffffffLL) return FA_ERR_SHAPE;                                // 32-bit offsets inside one head of K/V
    return FA_OK;
}

// One query row per head goes through the streaming kernel (FA_OPT_DECODE_KERNEL = 1 keeps the tile kernel:
// tests, tuning)
bool use_streaming_decode(const Options &opt, int Nq) { return Nq == 1 && opt[FA_OPT_DECODE_KERNEL] != 1; }

// Work decomposition for a problem: the mode, and the query rows of a workgroup (256, or 128 in FA_MODE_SPLIT and in
// FA_MODE_WIDE on workgroups of four waves).  W = B * H * ceil(Nq / 256), blocks = B * H * ceil(Nq / 128); the chip has 256
// compute units.  At D = 128 one eight-wave or two four-wave workgroups fill a compute unit, at D = 64 two or four. The
// lines come from sweeps of forced modes over 900 random shapes (us per launch, bf16 and fp16 mixed; "rows" is the
// persistent four-wave kernel of D = 128, "four" its plain counterpart of D = 64):
//  * at most one 128-row block per compute unit: FA_MODE_SPLIT puts eight waves on each and halves its chain of tiles,
//    unless the chain is short (split over four, bf16: D = 64 250 keys 1.03, 350 0.99, 500 0.96, 750 0.88; D = 128 250 1.08,
//    430 1.00, 520 0.97, 750 0.92, 1000 0.85; fp16, where both carry two sums: D = 64 350 1.02, 500 0.98, 750 0.91, D = 128
//    500 1.00, 750 0.89).
//  * whole rounds of causal work (one to four rounds of 256-row workgroups, the last one filled to 85%), D = 128:
//    FA_MODE_WIDE_FOLD, whose workgroups all carry the same triangular work and whose finished waves help the others, for a
//    single round (1 x 32 x 2048: 40.5, rows 44.5; several rounds: rows, 1 x 32 x 4096: 130 instead of 153).
//  * causal triangles at D = 64 (Nk little over Nq, Nq > 768) up to four rounds: FA_MODE_WIDE_FOLD as well (11 x 8365, 1.4
//    rounds: fold 149, split 175, four 181, wide 239; 94 x 2048, 2.9 rounds: 69, 79, 85, 91; beyond four rounds the forms
//    are within 5%, 204 x 2341 bf16: four 213, fold 227), but for a second or third round that would be nearly empty (16 x
//    5216, 1.31 rounds: split 84, fold 96; 16 x 5841, 1.44: 97, 109; 20 x 6533 fp16, 2.03: split 160, wide 165, fold 176),
//    for long walks in many rounds (32 x 6992 on 8441 fp16: wide 341, fold 366) and four blocks that are mostly padding (131
//    x 791 fp16: four 29, fold 37).
//  * long caches behind a block of rows at D = 64 (a causal Nk well over Nq, 1000 keys per query): FA_MODE_SPLIT up to 1.6
//    rounds (70 x 1024 on 2165: 52, four 62, wide 67; 81 x 1101 on 7241: 185, four 203, wide 206, fold 217), then the fold
//    to two (217 x 512 on 1969: 70, split 74, four 75); full attention likewise (169 x 321 on 3162: split 1.00, four 1.11,
//    wide 1.48 of the best; 50 x 1878: 1.00, 1.01, 1.14; 32 x 3209, 1.62 rounds: 1.05, 1.07, 1.00).
//  * long walks at D = 128 (4096 keys per query on average): FA_MODE_WIDE64, where its rounds of 256 are filled (1 x 20 x
//    8192, two and a half rounds: 437, rows 329), unless the last of a few blocks is mostly padding, which the fold spreads over
//    a head's workgroups (80 x 1302 on 16068 fp16: 1020, rows 1047, fold 939).
//  * the same kernel at D = 128 below 4096 keys (rows64; plans report FA_MODE_WIDE), where rounds are filled:
//    - full attention from 960 keys in one round, 1216 in several, 2048 where the last tile is ragged (rows, rows64: 1 x 32 x 2048
//      on 768 29.2, 29.3; on 1024 36.4, 35.0; on 1536 49.9, 46.4; on 2048 63.5, 58.1; on 2100 65.7, 66.3; 128 x 1024 on 1024 75.8,
//      77.9; on 1280 89.5, 87.0; on 2048 134, 125; on 2100 137.6, 137.4; wide is behind both, and is left with less than a round
//      on a ragged 1536 to 2047 keys);
//    - causal blocks of rows on long caches, 2400 keys on average, where no block's walk is over 4/3 of the average, before the
//      fold (fold, rows, rows64: 1 x 32 x 2048 on 3072 71.6, 72.1, 73.5; on 4096 107, 102, 97; on 6144 165, 154, 145; 64 x 2048
//      on 4096 215, 195, 190; 128 x 1024 on 2048 122, 111, 116; on 3072 185, 174, 162).  Triangles stay on rows, where they are
//      about level (3 x 32 x 4096 402, 400, the walks' first references closer to 64 bits), and so do uneven rounds (1 x 40 x
//      2048 on 6144: 225, 239; full on 2048: 98.7, 100).
//  * a second round of 512 256-row workgroups that would be nearly empty, full attention at D = 64 over 1535 keys: FA_MODE_SPLIT
//    (wide and split: 9 x 2 x 8712, 2.46 times 256 of them, 436, 391; 13 x 5 x 1896, 2.03, 96, 77; 1 x 20 x 7058, 2.19, 344, 311;
//    10 x 20 x 599 on 2673, 2.34, 112, 98), unless the last round of 256 128-row workgroups is as empty and the walk below 3000
//    keys (10 x 8 x 1587 on 1683, 1040 of them, 79, 81; 2 x 32 x 2119, 1088, 104, 106).
//  * causal triangles at D = 64 over 2200 keys on average in three to seven and a half rounds that are not the fold's: FA_MODE_SPLIT
//    (over 4096 keys against wide: 12 x 2 x 13340, 5.0 rounds, 696, 631; 2 x 12 x 9332, 3.5, 348, 314; 2 x 12 x 13540 fp16, 5.0, 685,
//    640; 4 x 12 x 9280, 6.9, 631, 600; below against four waves: 3 x 12 x 7581 fp16, 4.2, 387, 370; 3 x 20 x 5446, 5.2, 301, 286; 2 x
//    32 x 6731, 6.75, 486, 475; 6 x 20 x 4496, 8.4, level; 10 x 12 x 5019, 9.4, 520, 523).
//  * everything else on four waves, whose waves share a SIMD with other workgroups' (D = 128 causal: 16 x 32 x 2048 590,
//    wide 745; 3 x 20 x 1531 47, split 68, wide 70; full: 47 x 32 x 280 122, wide 205), but at D = 64 for full attention over
//    1536 keys and more (in bf16 and filled rounds 850), where the tiles loaded per 256 rows count (8 x 32 x 4096: wide 1141,
//    four 1184), and for causal walks over 4096 keys.  129 .. 144
//    rows at D = 64 stay one workgroup (464 x 144 on 161: wide 11.5, four 14.6; 1452 x 133 full: 32, 35; equal for square
//    causal ones).
//  * FA_MODE_SPLIT besides for causal Nq >= 2048 below 2.5 rounds at D = 128, its place in fa_fwd_plan's documented answer
//    (1 x 12 x 3000: 47, rows 57; but 2 x 20 x 2048: 66, rows 55), and over 4096 up to 2.25 rounds of 128-row blocks (1 x 8
//    x 8192: 137, rows 161; 8 x 8945, 2.19 rounds: 173, rows 192; 1 x 10 x 8192, 2.5: 220, rows 191).
// fa_set_option(FA_OPT_FWD_MODE, ...) overrides.
struct Decomposition {
    int mode, rows;
    bool two_sums = false;       // fp16 on 256 rows or in two groups: both row sums (the four-wave kernels on 128 rows always carry both)
    bool rows64 = false;         // FA_MODE_WIDE on waves of 64 rows: the kernel of FA_MODE_WIDE64
};
Decomposition choose_form(int forced, int B, int H, int Nq, int Nk, int D, int causal, int dtype) {
    const Decomposition split = {FA_MODE_SPLIT, 128}, wide = {FA_MODE_WIDE, 256}, four = {FA_MODE_WIDE, 128},
                        fold = {FA_MODE_WIDE_FOLD, 256}, wide64 = {FA_MODE_WIDE64, 256},
                        wide_rows64 = {FA_MODE_WIDE, 256, false, true};
    const long long heads = (long long)B * H, blocks = heads * (((long long)Nq + 127) / 128);
    const bool four_fits = blocks < (1ll << 28);                // list positions and their multiples by 8 stay inside int
    if (forced == FA_MODE_SPLIT) return split;
    if (forced == FA_MODE_WIDE) return wide;
    if (forced == FA_MODE_WIDE4) return four_fits ? four : wide;
    if (forced == FA_MODE_WIDE64) return D == 128 ? wide64 : wide;
    if (forced == FA_MODE_WIDE_FOLD) return causal ? fold : wide;
    const long long nqt = ((long long)Nq + 255) / 256, W = heads * nqt;
    const long long rounds = (W + 255) / 256;
    const bool full_rounds = rounds * 256 * 100 <= W * 115;     // the last round of 256-row workgroups at least 85% full
    const long long avg_keys = causal ? (long long)Nk - Nq / 2 : (long long)Nk;
    if (blocks <= 256) {
        const int short_walk = dtype == FA_DTYPE_F16 ? 500 : D == 64 ? 350 : 460;   // (fp16's two sums cost the split form more)
        return Nk <= short_walk ? four : split;
    }
    if (!four_fits) return D == 64 ? wide : avg_keys >= 4096 ? wide64 : wide_rows64;
    if (D == 64) {
        if (W >= 256 && Nq > 128 && Nq <= 144 && (!causal || Nk >= Nq + 16)) return wide;
        if (!causal && avg_keys >= 1000 && W > 256 && W <= 404) return split;
        const bool full_split = (blocks + 255) / 256 * 256 * 100 <= blocks * 116;   // rounds of 128-row workgroups, 86% of their places taken
        if (!causal && avg_keys > 1535 && W > 512 && W <= 640 && (full_split || avg_keys >= 3000)) return split;
        if (!causal) return avg_keys > 1535 || (dtype == FA_DTYPE_BF16 && avg_keys >= 850 && (W < 256 || full_rounds)) ? wide : four;
        if (nqt >= 4 && 10ll * Nq >= 7ll * Nk) {
            if ((W > 256 && W <= 384) || (W > 512 && W <= 580 && Nq >= 1024)) return split;
            const bool roomy = Nq >= 922 || (W >= 256 && full_rounds);      // (four 256-row blocks of fewer rows are padding)
            if (roomy && W <= 1024 && (avg_keys <= 4096 || W <= 768)) return fold;
            if (avg_keys > 2200 && W <= 1900) return split;
        } else if (avg_keys >= 1000 && nqt >= 2 && W <= 512) {
            return W <= 420 ? split : fold;
        } else if (avg_keys >= 2500 && W <= 390) {
            return split;
        }
        return avg_keys > 4096 ? wide : four;
    }
    if (causal && full_rounds) {
        if (avg_keys >= 8192 && (nqt >= 16 || 100ll * Nq >= 93ll * 256 * nqt)) return wide64;
        const bool even = 4ll * avg_keys >= 3ll * Nk && Nk % 64 == 0;      // no block much longer than the others
        if (avg_keys >= 2400 && even) return avg_keys >= 4096 ? wide64 : wide_rows64;
    }
    if (causal && nqt >= 4) {
        if (W >= 256 && W <= 1024 && full_rounds && Nq <= 4096) return W <= 256 || avg_keys >= 8192 ? fold : Decomposition{FA_MODE_WIDE_FOLD, 128};
        if (Nq > 4096 ? blocks <= 576 : Nq >= 2048 && W < 640) return split;
    }
    if (avg_keys >= 4096 && (full_rounds || W >= 6 * 256)) return wide64;
    if (!causal && Nk >= (Nk % 64 != 0 ? 2048 : W <= 256 ? 960 : 1216) && (W <= 256 || full_rounds || W >= 6 * 256)) return wide_rows64;
    if (!causal && Nk >= 1536 && W <= 256 && !full_rounds) return wide;
    return four;
}

// Whether an fp16 call on eight waves carries both row sums (TWO_SUMS in fa_attention_kernel.inc).  One sum is kept where the rows
// are long or the eight-wave forms are well ahead of the four-wave ones, which carry both in any case: long walks in few blocks,
// FOLD's whole rounds, SPLIT from 2048 rows on, walks over 4096 keys (full: 1535).  Whatever lies between, where either kind of
// workgroup is within some percent of the other, is as exact on eight waves as it is on four.
bool fp16_two_sums(int B, int H, int Nq, int Nk, int D, int causal) {
    const long long heads = (long long)B * H, blocks = heads * (((long long)Nq + 127) / 128);
    const long long nqt = ((long long)Nq + 255) / 256, W = heads * nqt, avg_keys = causal ? (long long)Nk - Nq / 2 : (long long)Nk;
    const bool full_rounds = (W + 255) / 256 * 256 * 100 <= W * 115;
    if (blocks <= 256) return Nk <= (!causal ? 1024 : D == 64 ? 512 : 768);
    if (causal && nqt >= 4) {
        if (W >= 256 && W <= (D == 64 ? 1024 : 256) && full_rounds && Nq <= (D == 64 ? 8192 : 4096)) return false;
        if (D == 64 && W < 256 && Nq > 1792 && Nq <= 8192) return false;
        if (Nq > 4096 ? blocks <= 512 : Nq >= 2048 && W < 640) return false;
    }
    if (D == 64) return avg_keys <= (causal ? 4096 : 1535);
    return causal ? avg_keys < 8192 : !(Nk >= 1536 && (full_rounds || W >= 6 * 256));
}

Decomposition choose_mode(const Options &opt, int B, int H, int Nq, int Nk, int D, int causal, int dtype) {
    Decomposition d = choose_form(opt[FA_OPT_FWD_MODE], B, H, Nq, Nk, D, causal, dtype);
    d.two_sums = opt[FA_OPT_FWD_MODE] == FA_AUTO && fp16_two_sums(B, H, Nq, Nk, D, causal);
    // (walks over 4096 keys have always been on WIDE64 with the one sum)
    if ((d.mode == FA_MODE_WIDE64 || d.rows64) && (causal ? (long long)Nk - Nq / 2 : (long long)Nk) >= 4096) d.two_sums = false;
    return d;
}

// Query rows of a workgroup under a descriptor mask: 128 (four waves), but for long walks 256, which load each tile for
// twice the rows.  A walk's length is the keys a row sees on average (padding counted as keys: the counts are on the
// device); the line lies later the more of its tiles are masked, which cost the four-wave form less, and at D = 64, where
// two 256-row workgroups share a compute unit, later still for rounds of 512 that are not filled, whose times are uneven
// both ways.  Less than a round of 256-row workgroups stays with 128.  us per call on 256 and 128 rows, bf16, D = 64 and
// 128: full with key counts 16 x 16 x 1024 39 37, 77 68; 8 x 16 x 2048 122 122, 203 199; 1 x 32 x 8192 343 348, 537 549;
// causal 4 x 16 x 4096 208 183, 305 289; 1 x 32 x 8192 335 336, 505 500; 1 x 16 x 16384 658 693, 922 943; 1 x 16 x 12000
// (1.5 rounds of 512) 351 358, 521 540; 1 x 20 x 12000 548 522, 736 716; window 4096 of 2 x 16 x 16384 545 542, 919 912;
// 8192 of 1 x 16 x 16384 465 478, 711 740; half a round, 1 x 2 x 16384, 247 179, 325 249.  fa_set_option(FA_OPT_FWD_MODE,
// FA_MODE_WIDE | FA_MODE_WIDE4) overrides (tests, tuning).
int masked_rows(int forced, const MaskGeom &g, long long heads, int Nq, int Nk, int D) {
    if (forced == FA_MODE_WIDE) return 256;
    if (forced == FA_MODE_WIDE4) return 128;
    const long long W = heads * (((long long)Nq + 255) / 256);
    if (W < 243 || (D == 64 && W > 256 && W < 480)) return 128;
    constexpr int SAMPLES = 16;
    long long keys = 0;
    for (int i = 0; i < SAMPLES; ++i) {
        const long long diag = g.off + (2ll * i + 1) * Nq / (2 * SAMPLES);
        const long long lo = diag - g.left > g.pfx ? diag - g.left : g.pfx, hi = diag + g.right < Nk - 1 ? diag + g.right : Nk - 1;
        keys += g.pfx + (hi >= lo ? hi - lo + 1 : 0);
    }
    const bool left_edge = (long long)g.off + Nq - 1 - g.left > g.pfx, right_edge = (long long)g.off + g.right < Nk - 1;
    int line = left_edge ? 5000 : right_edge ? (D == 128 ? 3500 : 4000) : 2100;
    if (D == 64 && W > 256 && W * 100 < (W + 511) / 512 * 512 * 93) line = 6500;
    return keys / SAMPLES > line ? 256 : 128;
}

// 64-key tiles the workgroup of query block qt walks (mirrors the kernel's kmax_wg)
long long tiles_walked(int mode, int BM, long long nqt, long long qt, int Nq, int Nk, int causal) {
    long long kmax = (long long)Nk - 1;
    if (causal) {
        long long last_row = qt * BM + BM - 1;
        if (last_row > (long long)Nq - 1) last_row = (long long)Nq - 1;
        if (mode == FA_MODE_WIDE_FOLD && BM == 256) {
            last_row = -1;
            for (int w = 0; w < 8; ++w) {
                const long long first = (long long)fold_block((int)nqt, (int)qt, w) * 32;
                if (first < Nq) {
                    const long long l = first + 31 < (long long)Nq - 1 ? first + 31 : (long long)Nq - 1;
                    if (l > last_row) last_row = l;
                }
            }
            if (last_row < 0) return 0;
        }
        const long long lim = last_row + ((long long)Nk - Nq);
        if (lim < kmax) kmax = lim;
    }
    return kmax >= 0 ? kmax / BN + 1 : 0;
}

// Split-KV launch shape.  nsplit_in > 0 is taken as given (clamped to the number of key tiles); otherwise runs of at least
// four tiles:
//  * a few queries (up to 16): as many as one round of workgroups holds -- one per compute unit at D = 128, two at D = 64,
//    whose tiles are half the bytes; the path is bound by HBM, which that many workgroups' loads in flight saturate.  A
//    round is counted per XCD: the work items go to the XCDs in runs of ceil(items / 8), and one run too many for an XCD's
//    32 compute units costs a second round (2 x 24 heads, 4 queries on 30000: 6 runs 193 us, 5 116); but two runs are kept
//    where one would leave a full round uneven, one run's and two's times at 4000 keys: D = 64, 288 heads 58 69, 352 70 70,
//    440 78 75, 504 92 87; D = 128, 192 heads 74 81, 228 83 83, 250 89 83; at 1000 keys one is 1.2 to 1.5 times as fast
//    throughout;
//  * more queries, where the number of workgroups alone asks for more than one run: the least of splitkv_cost, which prices
//    rounds, walks and the merge (us per call, chosen by the number of workgroups alone and by cost: 1 x 40 x 1000 on 20000
//    505, 393; 1 x 20 x 100 on 30000 107, 72; 3 x 8 x 225 on 6114 61, 40; 2 x 16 x 1000 on 9000 146, 134; 3 x 40 x 594 on
//    837, D = 64, 42, 27; and where an estimate that put one run too low had left them: 4 x 32 x 101 on 14122 179 in two
//    runs, 257 in one; 2 x 16 x 1042 on 24182, D = 64, 311 in four, 369 in one).
// The streaming kernel of the single-query case (fa_decode_kernel) does best with one four-wave workgroup per compute unit
// as well (each wave keeps 32 KiB of loads in flight): more of them only shorten the contiguous runs and add partial results
// to merge (measured: 512 workgroups 1-3% slower, 1024 5-10%). Where nobody asked for a number of runs and ceil(256 / heads)
// of them per head would leave compute units idle in a second round (up to 192 heads that do not divide 256), or one per
// head would (257 .. 320 heads), the tiles of all heads are cut into 256 equal pieces instead, given 20 tiles a piece (us
// per call, runs and pieces: 3 x 12 x 28949, D = 64: 57, 47; 2 x 24 x 32768: 156, 125; 10 x 32 x 3000: 88, 77; but 3 x 12 x
// 2000, D = 64, 4.5 tiles: 8.2, 9.7).  The lines in heads, equal runs' time over the pieces' at 20, 55 and 110 or more tiles
// a piece: 160 heads 1.08 1.12 1.15 at D = 64, 1.10 1.14 1.16 at 128; 192 heads 1.00 1.03 1.04, 0.98 1.05 1.03; 208 heads
// 1.00 1.00 0.99, 0.98 1.00 1.00; 224 heads 0.91 0.97 0.99, 0.97 0.97 0.99; 250 heads 0.96 0.98 0.84, 0.96 0.98 0.89; 257
// heads 1.10 1.25 1.29, 1.23 1.28 1.33; 320 heads 1.00 1.08 1.14, 1.07 1.12 1.19; 384 heads 0.87 0.96 1.02, 0.99 1.01 1.02.
constexpr int SPLITKV_MAX = 1024;
constexpr long long DECODE_WORKGROUPS = 256;
constexpr long long DECODE_PIECE_TILES = 20;
struct SplitChoice {
    int nsplit, stream_wgs;      // runs of a head (at most, with pieces); pieces of all heads laid end to end, 0: none
};
// Estimated microseconds of a call cut into n runs.  Fitted to 438 random shapes, each timed at 1 .. 48 runs: the number it
// picks takes 1.01 of the best one's time on average.  What the terms stand for: a single run is fa_fwd, 128-row workgroups in
// rounds of 256 (at D = 64 of whole ones, at D = 128 evened out by the list); several are 256-row work items in rounds of as many
// as an XCD holds, cheaper where half of the rows do not exist; a round of workgroups that start together takes as long as the
// longest walk, more of them as long as the average one; the merge moves every partial sum twice; and nothing is faster than
// reading K and V.
double splitkv_cost(long long heads, int Nq, int Nk, int D, long long n) {
    const double longest = (double)Nk / BN, average = Nk >= Nq ? (double)((long long)Nk - Nq / 2) / BN : longest;
    const double x = (double)(heads * (((long long)Nq + 127) / 128)) / 256;
    const double w = (double)((heads * (((long long)Nq + 255) / 256) + 7) / 8 * n);
    const double half = Nq <= 128 ? 0.7 / (double)n : 1.0 / (double)n, partial = (double)n * heads * Nq * D * 8;
    double t;
    if (D == 128) {
        if (n == 1) t = (x <= 1 ? longest * (0.6 + 0.42 * x) : fmax(average * (0.25 + 0.95 * x), longest * 1.02)) + 8;
        else t = ceil(w / 32) * ((w <= 32 ? longest : average) * half * 1.65 + 3.3) + 7.2 + partial / 5.5e6;
    } else {
        // (K and V that do not fit the 256 MiB cache slow many runs down more than one)
        const bool big = Nq > 128 && heads * Nk * D * 4 > (256ll << 20);
        if (n == 1) t = (x <= 1 ? longest * (0.47 + 0.17 * x) : fmax(average * 0.58 * ceil(x), longest * 0.64)) * (big ? 1.05 : 1.0) + 7;
        else if (w <= 32) t = longest * half * (big ? 1.34 : 1.12) + 2 + 7 + partial / 3.5e6;
        else t = ceil(w / 64) * ((w <= 64 ? longest : average) * half * (big ? 2.04 : 1.7) + 2) + 7 + partial / 3.5e6;
    }
    return fmax(t, (double)heads * Nk * D * 4 / 5.8e6 + 5);
}
// may_cut: the caller can take pieces (fa_decode_masked's shares are runs of equal numbers of VISIBLE keys instead)
SplitChoice choose_nsplit(int B, int H, int Nq, int Nk, int D, int nsplit_in, bool streaming, bool may_cut = true) {
    const long long heads = (long long)B * H, nwork = heads * (((long long)Nq + 255) / 256);
    const long long tiles_k = ((long long)Nk + BN - 1) / BN;
    long long n = nsplit_in;
    if (n <= 0) {
        const long long target = streaming ? DECODE_WORKGROUPS : (D == 128 ? 256 : 512);
        if (streaming && may_cut) {
            const long long total = nwork * tiles_k, wgs = DECODE_WORKGROUPS;
            const bool uneven = nwork <= 192 ? wgs % nwork != 0 : nwork > 256 && nwork <= 320;
            if (uneven && total >= wgs * DECODE_PIECE_TILES && (total + 1) * wgs < (1ll << 32)) {
                // a head's tiles begin at a multiple of 1/b of a piece and are a/b pieces long
                long long x = wgs, y = nwork;
                while (y) { const long long t = x % y; x = y; y = t; }
                const long long a = wgs / x, b = nwork / x;
                return {(int)((a + 2 * b - 2) / b), (int)wgs};
            }
        }
        n = (target + nwork - 1) / nwork;
        if (n > tiles_k / 4) n = tiles_k / 4;
        if (n < 1) n = 1;
        if (Nq > 1 && Nq <= 16) {
            const long long fit = target / 8 / ((nwork + 7) / 8);
            const bool nearly_full = tiles_k >= 60 && nwork * (D == 128 ? 9 : 11) >= target * 8;
            if (n > fit && !(nearly_full && n == 2)) n = fit;
        } else if (Nq > 16 && n > 1) {
            // (never past fa_fwd_splitkv_static's array where the number of workgroups alone stayed within it; priced as under
            // the causal mask either way, so that a plan holds for both)
            const long long row_bytes = heads * Nq * (D + 2) * 4;
            const long long cap = n * row_bytes > FA_STATIC_WORKSPACE_BYTES ? n * row_bytes : FA_STATIC_WORKSPACE_BYTES;
            double best = splitkv_cost(heads, Nq, Nk, D, 1);
            n = 1;
            for (long long i = 2; i <= 64 && i <= tiles_k / 4 && i * row_bytes <= cap; ++i) {
                const double t = splitkv_cost(heads, Nq, Nk, D, i);
                if (t < best) {
                    best = t;
                    n = i;
                }
            }
        }
    }
    if (n > tiles_k) n = tiles_k;
    if (n > SPLITKV_MAX) n = SPLITKV_MAX;
    if (n < 1) n = 1;
    return {(int)n, 0};
}

template <int DT, int D, bool TWO_SUMS = DT == FA_DTYPE_BF16>
hipError_t launch_pair(const FaParams &p, int nwork_padded, hipStream_t stream) {
    hipLaunchKernelGGL((fa_fwd_kernel<DT, D, true, true, false, false, true, 8, TWO_SUMS>), dim3(nwork_padded), dim3(512), 0, stream, p);
    return hipGetLastError();
}

// the plain instantiations: (split | wide) x dtype x head dimension x causal, the paired fold (causal only), and the
// four-wave forms of wide: persistent at D = 128, one workgroup per block at D = 64
hipError_t launch_attention(const FaParams &p, Decomposition dec, int D, int causal, int dtype, int grid, hipStream_t st) {
    hipError_t e;
    const int mode = dec.mode;
    if (dec.rows == 128 && mode != FA_MODE_SPLIT) {
        if (D == 128) return launch_rows(p, dtype, causal != 0, st);
        FaParams f = p;
        if (!causal) f.off = p.Nk - 1;             // the causal instantiation with the diagonal past every key
        return dtype == FA_DTYPE_F16 ? launch<0, 64, true, true, 4, true>(f, grid, st) : launch<1, 64, true, true, 4>(f, grid, st);
    }
    if (dtype == FA_DTYPE_F16 && dec.two_sums && mode != FA_MODE_WIDE64 && !dec.rows64) {
        // (full attention through the causal instantiations, with the diagonal past every key)
        FaParams f = p;
        if (!causal) f.off = p.Nk - 1;
        if (mode == FA_MODE_SPLIT) return D == 64 ? launch<0, 64, true, false, 8, true>(f, grid, st) : launch<0, 128, true, false, 8, true>(f, grid, st);
        if (mode == FA_MODE_WIDE) return D == 64 ? launch<0, 64, true, true, 8, true>(f, grid, st) : launch<0, 128, true, true, 8, true>(f, grid, st);
        if (causal && D == 64) return launch_pair<0, 64, true>(p, grid, st);
    }
    if (mode == FA_MODE_WIDE64 || dec.rows64) {
        if (D != 128) return hipErrorInvalidValue;
        if (dtype == 0 && dec.two_sums) {
            FaParams f = p;
            if (!causal) f.off = p.Nk - 1;         // the causal instantiation with the diagonal past every key
            hipLaunchKernelGGL((fa_fwd_wide64_kernel<0, true, false, true>), dim3(grid), dim3(256), 0, st, f);
        } else if (dtype == 0 && causal) hipLaunchKernelGGL((fa_fwd_wide64_kernel<0, true>), dim3(grid), dim3(256), 0, st, p);
        else if (dtype == 0) hipLaunchKernelGGL((fa_fwd_wide64_kernel<0, false>), dim3(grid), dim3(256), 0, st, p);
        else if (causal) hipLaunchKernelGGL((fa_fwd_wide64_kernel<1, true>), dim3(grid), dim3(256), 0, st, p);
        else hipLaunchKernelGGL((fa_fwd_wide64_kernel<1, false>), dim3(grid), dim3(256), 0, st, p);
        return hipGetLastError();
    }
    if (mode == FA_MODE_WIDE_FOLD && causal) {
        switch ((dtype << 1) | (D == 128)) {
            case 0: return launch_pair<0, 64>(p, grid, st);
            case 1: return launch_pair<0, 128>(p, grid, st);
            case 2: return launch_pair<1, 64>(p, grid, st);
            default: return launch_pair<1, 128>(p, grid, st);
        }
    }
    if (mode == FA_MODE_SPLIT) {
        // full attention is the causal instantiation with the diagonal past every key (at D = 64 it takes 120 registers
        // where one without the limit took 136, a fourth wave per SIMD)
        FaParams f = p;
        if (!causal) f.off = p.Nk - 1;
        switch ((dtype << 1) | (D == 128)) {
            case 0: return launch<0, 64, true, false>(f, grid, st);
            case 1: return launch<0, 128, true, false>(f, grid, st);
            case 2: return launch<1, 64, true, false>(f, grid, st);
            default: return launch<1, 128, true, false>(f, grid, st);
        }
    }
    switch ((dtype << 2) | ((D == 128) << 1) | (causal ? 1 : 0)) {
        case 0: e = launch<0, 64, false, true>(p, grid, st); break;
        case 1: e = launch<0, 64, true, true>(p, grid, st); break;
        case 2: {                                  // (the causal instantiation with the diagonal past every key)
            FaParams f = p;
            f.off = p.Nk - 1;
            e = launch<0, 128, true, true>(f, grid, st);
            break;
        }
        case 3: e = launch<0, 128, true, true>(p, grid, st); break;
        case 4: e = launch<1, 64, false, true>(p, grid, st); break;
        case 5: e = launch<1, 64, true, true>(p, grid, st); break;
        case 6: e = launch<1, 128, false, true>(p, grid, st); break;
        case 7: e = launch<1, 128, true, true>(p, grid, st); break;
        default: e = hipErrorInvalidValue; break;
    }
    return e;
}

struct LinearTile {
    int rows, cols;
};
// The projection's workgroup tile: the largest (rows x outputs; less LDS traffic per matrix instruction, more work per
// barrier) that gives every compute unit a workgroup, or, where even the smaller ones make at most 256, the smallest: a
// launch that leaves compute units idle takes as long as one workgroup's chain of k-tiles.  Two smaller tiles per compute
// unit are slower than one of the next size.  us per call with the attention, tiles 128 x 256, 128 x 128, 64 x 128 (number
// of workgroups of the chosen one), bf16, D = 128, 32 heads, outputs: 256 rows x 4096 65, 46, 38 (128); 512 rows x 4096, 40
// heads 83, 60, 52 (256); 768 rows x 4096 75, 56, 72 (192); 1024 x 4096 77, 62, 76 (256); 1280 x 4096 86, 101, 106 (160).
// `shared`: the next block's attention runs beside it.  64 x 128 tiles, whose workgroups take a compute unit's LDS to
// themselves, then leave it a quarter of the chip at least (D = 64, blocks of 1024 whose first has 512 rows: 1 x 20 x 2178,
// 3840 outputs, 240 of them 100 us, 120 of 128 x 128 95; 1 x 32 x 2093, 3584: 224 117, 112 111; 2 x 40 x 1031, 2560 in
// blocks of 512, 160 for the first 256 rows: 106, 111). FA_OPT_LINEAR_TILE overrides (tests, tuning).
LinearTile choose_linear_tile(int forced, int B, int rows, int N, bool shared) {
    const LinearTile forms[] = {{64, 128}, {128, 128}, {128, 256}, {256, 256}};
    auto tiles = [&](const LinearTile &t) { return (long long)B * (((long long)rows + t.rows - 1) / t.rows) * (N / t.cols); };
    switch (forced) {
        case 256: return forms[3];
        case 128: return forms[2];
        case 128128: return forms[1];
        case 64128: return forms[0];
        default: break;
    }
    if (tiles(forms[0]) <= (shared ? 192 : 256)) return forms[0];
    if (tiles(forms[1]) <= 256) return forms[1];
    return tiles(forms[3]) >= 256 ? forms[3] : forms[2];
}
template <int DT>
hipError_t launch_linear(const LinParams &p, LinearTile t, hipStream_t stream) {
    const dim3 grid(p.per_xcd * 8), block(512);
    if (t.rows == 256) hipLaunchKernelGGL((fa_linear_kernel<DT, 256, 256, 2>), grid, block, 0, stream, p);
    else if (t.cols == 256) hipLaunchKernelGGL((fa_linear_kernel<DT, 128, 256, 3>), grid, block, 0, stream, p);
    else if (t.rows == 128) hipLaunchKernelGGL((fa_linear_kernel<DT, 128, 128, 4>), grid, block, 0, stream, p);
    else hipLaunchKernelGGL((fa_linear_kernel<DT, 64, 128, 6>), grid, block, 0, stream, p);
    return hipGetLastError();
}

// Row tiles per panel of the projection's tile order.  The c = min(per_xcd, 32) workgroups an XCD runs at a
// time (one per compute unit) are consecutive tiles of its run: R row tiles by c / R column slices, for which
// its L2 fetches R * rows of o and (c / R) * cols of w, each K elements long: least for
// R = sqrt(c * cols / rows).  Measured: 4% on launches of several rounds, nothing on single-round ones.
int linear_panel(int per_xcd, LinearTile t, int m_tiles) {
    const int c = per_xcd < 32 ? per_xcd : 32;
    int R = 1;
    while ((R + 1) * (R + 1) * t.rows <= c * t.cols) ++R;
    if (R > m_tiles) R = m_tiles;
    return R < 1 ? 1 : R;
}

// The parameter block every entry point starts from: one launch over the whole of q (no row range,
// no split, no descriptor mask).
FaParams base_params(const void *q, const void *k, const void *v, void *o, float *lse, int H, int Nq, int Nk,
                     long long nqt, long long nwork, float scale) {
    FaParams p;
    p.q = (const uint16_t *)q;
    p.k = (const uint16_t *)k;
    p.v = (const uint16_t *)v;
    p.o = (uint16_t *)o;
    p.lse = lse;
    p.H = H;
    p.Nq = Nq;
    p.Nk = Nk;
    p.q_rows = Nq;
    p.kv_rows = Nk;
    p.off = Nk - Nq;
    p.nqt = (int)nqt;
    p.nwork = (int)nwork;
    p.per_xcd = (int)((nwork + 7) / 8);
    const float LOG2E = 1.4426950408889634f;
    p.qmode = scale > 0.f ? 0 : (scale < 0.f ? 1 : 2);
    p.c = scale == 0.f ? 1.f : fabsf(scale) * LOG2E;
    p.nsplit = 1;
    p.stream_wgs = 0;
    p.kv_stream = 0;
    p.part_o = nullptr;
    p.part_ml = nullptr;
    p.tag = 0;
    p.left = p.right = p.prefix = 0;
    p.anchor = 0;
    p.kv_len = nullptr;
    p.head_run = p.head_rest = p.grouped = p.group = 0;
    return p;
}

// Descriptor checks shared by the masked entry points; fills the geometry for `klen` valid keys.
int mask_geometry(const fa_mask_t *mask, int klen, int Nq, int Nk, MaskGeom *g) {
    if (!mask) return FA_ERR_NULL;
    if (Nq <= 0 || Nk <= 0) return FA_ERR_SHAPE;
    if ((long long)Nq + Nk >= MASK_NO_LIMIT) return FA_ERR_SHAPE;   // window arithmetic stays inside int
    if (mask->prefix < 0) return FA_ERR_MASK;
    if (klen < 0 || klen > Nk) return FA_ERR_MASK;
    if (mask->diag_from_kv_len != 0 && mask->diag_from_kv_len != 1) return FA_ERR_MASK;
    g->off = (mask->diag_from_kv_len ? klen : Nk) - Nq;
    g->left = mask->window_left < 0 || mask->window_left > MASK_NO_LIMIT ? MASK_NO_LIMIT : mask->window_left;
    g->right = mask->window_right < 0 || mask->window_right > MASK_NO_LIMIT ? MASK_NO_LIMIT : mask->window_right;
    g->pfx = mask->prefix < klen ? mask->prefix : klen;
    g->klen = klen;
    return FA_OK;
}

}  // namespace

extern "C" {

int fa_fwd_plan(int B, int H, int Nq, int Nk, int D, int causal, int dtype, fa_plan_t *plan) {
    if (!plan) return FA_ERR_NULL;
    const int rc = check_shape(B, H, Nq, Nk, D, dtype);
    if (rc != FA_OK) return rc;
    const long long tiles_k = ((long long)Nk + BN - 1) / BN;
    const Options opt = options_now();
    if (use_streaming_decode(opt, Nq)) {
        // one query per head (it sees every key, causal or not): fa_decode_kernel, one workgroup per (batch, head)
        plan->mode = FA_MODE_STREAM;
        plan->block_m = 1;
        plan->block_n = BN;
        plan->threads = DECODE_WAVES * 64;
        plan->grid = B * H;
        plan->work_items = (long long)B * H;
        plan->tiles_visited = plan->tiles_total = (long long)B * H * tiles_k;
        plan->lds_bytes = DECODE_WAVES * (512 / D) * (D + 2) * 4;     // one partial state per lane group
        return FA_OK;
    }
    const Decomposition dec = choose_mode(opt, B, H, Nq, Nk, D, causal, dtype);
    const int mode = dec.mode, BM = dec.rows;
    const bool four = BM == 128 && mode != FA_MODE_SPLIT;
    const long long nqt = ((long long)Nq + BM - 1) / BM;
    const long long nwork = (long long)B * H * nqt;
    long long visited = 0;
    for (long long qt = 0; qt < nqt; ++qt) visited += tiles_walked(mode, BM, nqt, qt, Nq, Nk, causal);
    plan->mode = mode;
    plan->block_m = BM;
    plan->block_n = BN;
    plan->threads = mode == FA_MODE_WIDE64 || dec.rows64 || four ? 256 : 512;
    plan->grid = four && D == 128 ? rows_grid((long long)B * H, nqt) : (int)(((nwork + 7) / 8) * 8);
    plan->work_items = nwork;
    plan->tiles_visited = visited * B * H;
    plan->tiles_total = nwork * tiles_k;
    plan->lds_bytes = (mode == FA_MODE_WIDE || four ? 1 : 2) * 4 * BN * D * 2;    // sets of 2+2 tiles
    if (mode == FA_MODE_WIDE64 || dec.rows64) plan->lds_bytes = 4 * (16 * 1088 + BN * D * 2);   // ring of four (padded K tile, V tile)
    return FA_OK;
}

static int fwd(const Options &opt, const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int Nq, int Nk,
               int D, float scale, int causal, int dtype, void *stream) {
    if (!q || !k || !v || !o || !lse) return FA_ERR_NULL;
    const int rc = check_shape(B, H, Nq, Nk, D, dtype);
    if (rc != FA_OK) return rc;
    if (!isfinite(scale)) return FA_ERR_SCALE;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return FA_ERR_ALIGN;
    if ((uintptr_t)lse & 3) return FA_ERR_ALIGN;

    const bool stream_kernel = use_streaming_decode(opt, Nq);
    const Decomposition dec = stream_kernel ? Decomposition{FA_MODE_STREAM, 256} : choose_mode(opt, B, H, Nq, Nk, D, causal, dtype);
    const int BM = dec.rows;
    const long long nqt = ((long long)Nq + BM - 1) / BM;
    const long long nwork = (long long)B * H * nqt;

    FaParams p = base_params(q, k, v, o, lse, H, Nq, Nk, nqt, nwork, scale);
    const int grid = p.per_xcd * 8;
    hipStream_t st = (hipStream_t)stream;

    hipError_t e;
    if (stream_kernel) {
        // a single query per head: the streaming kernel, one run per (batch, head), which stores o and lse itself
        switch ((dtype << 1) | (D == 128)) {
            case 0: e = launch_decode<0, 64>(p, (int)nwork, nwork, st); break;
            case 1: e = launch_decode<0, 128>(p, (int)nwork, nwork, st); break;
            case 2: e = launch_decode<1, 64>(p, (int)nwork, nwork, st); break;
            default: e = launch_decode<1, 128>(p, (int)nwork, nwork, st); break;
        }
    } else {
        e = launch_attention(p, dec, D, causal, dtype, grid, st);
    }
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return FA_ERR_LAUNCH;
    }
    return FA_OK;
}

int fa_fwd(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int Nq, int Nk,
           int D, float scale, int causal, int dtype, void *stream) {
    return fwd(options_now(), q, k, v, o, lse, B, H, Nq, Nk, D, scale, causal, dtype, stream);
}

// (causal or not, the plan is the same)
static int splitkv_plan(const Options &opt, int B, int H, int Nq, int Nk, int D, int dtype, int nsplit, fa_splitkv_plan_t *plan) {
    if (!plan) return FA_ERR_NULL;
    const int rc = check_shape(B, H, Nq, Nk, D, dtype);
    if (rc != FA_OK) return rc;
    if (nsplit > SPLITKV_MAX) return FA_ERR_NSPLIT;
    const long long nqt = ((long long)Nq + 255) / 256;
    const long long nwork = (long long)B * H * nqt;
    const bool streaming = use_streaming_decode(opt, Nq);
    const SplitChoice choice = choose_nsplit(B, H, Nq, Nk, D, nsplit, streaming);
    const int ns = choice.nsplit;
    const long long rows = (long long)B * H * Nq;
    plan->nsplit = ns;
    plan->streaming = streaming ? 1 : 0;
    plan->grid_x = choice.stream_wgs ? choice.stream_wgs : streaming ? (int)nwork : (int)(((nwork + 7) / 8) * 8);
    plan->grid_y = choice.stream_wgs ? 1 : ns;
    // (a single run is fa_fwd's launch; a single query's few runs are merged by the first kernel)
    plan->combine_grid = ns == 1 || (streaming && merges_itself(ns, D)) ? 0 : (int)((rows + (1024 / D) - 1) / (1024 / D));
    plan->work_items = nwork;
    plan->workspace_bytes = (long long)ns * rows * (D + 2) * 4;
    return FA_OK;
}

int fa_fwd_splitkv_plan(int B, int H, int Nq, int Nk, int D, int causal, int dtype, int nsplit,
                        fa_splitkv_plan_t *plan) {
    (void)causal;
    return splitkv_plan(options_now(), B, H, Nq, Nk, D, dtype, nsplit, plan);
}

static int splitkv(const Options &opt, const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int Nq,
                   int Nk, int D, float scale, int causal, int dtype, int nsplit, void *workspace, long long workspace_bytes,
                   void *stream) {
    if (!q || !k || !v || !o || !lse) return FA_ERR_NULL;
    fa_splitkv_plan_t pl;
    const int rc = splitkv_plan(opt, B, H, Nq, Nk, D, dtype, nsplit, &pl);
    if (rc != FA_OK) return rc;
    if (!isfinite(scale)) return FA_ERR_SCALE;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return FA_ERR_ALIGN;
    if ((uintptr_t)lse & 3) return FA_ERR_ALIGN;
    if (!workspace || workspace_bytes < pl.workspace_bytes) return FA_ERR_WORKSPACE;
    if ((uintptr_t)workspace & 15) return FA_ERR_ALIGN;
    const long long rows = (long long)B * H * Nq;
    if (rows > 0x7fffffffLL * 8) return FA_ERR_SHAPE;   // combine grid
    // a single run has nothing to merge: it is fa_fwd's launch (whose decompositions beat a one-run walk of
    // the split-KV kernel by about 5% when there are enough query blocks to fill the chip without splitting)
    if (pl.nsplit == 1) return fwd(opt, q, k, v, o, lse, B, H, Nq, Nk, D, scale, causal, dtype, stream);

    FaParams p = base_params(q, k, v, o, lse, H, Nq, Nk, ((long long)Nq + 255) / 256, pl.work_items, scale);
    p.nsplit = pl.nsplit;
    p.stream_wgs = pl.streaming && pl.grid_y == 1 ? pl.grid_x : 0;     // (a single run went to fa_fwd above)
    p.kv_stream = Nq <= 256;
    p.part_o = (float *)workspace;
    p.part_ml = p.part_o + (size_t)pl.nsplit * rows * D;
    hipStream_t st = (hipStream_t)stream;

    hipError_t e;
    if (pl.streaming) {
        if (pl.combine_grid == 0) p.tag = decode_tag();
        // one query sees every key under the bottom-right-aligned causal mask: causal or not is the same
        switch ((dtype << 1) | (D == 128)) {
            case 0: e = launch_decode<0, 64>(p, (int)pl.work_items, rows, st); break;
            case 1: e = launch_decode<0, 128>(p, (int)pl.work_items, rows, st); break;
            case 2: e = launch_decode<1, 64>(p, (int)pl.work_items, rows, st); break;
            default: e = launch_decode<1, 128>(p, (int)pl.work_items, rows, st); break;
        }
        if (e != hipSuccess) {
            g_last_hip_error = (int)e;
            return FA_ERR_LAUNCH;
        }
        return FA_OK;
    }
    // keys a query sees per run, on average (as in choose_mode): from 1400 the wide64 kernel is the faster one (us, tile kernel and
    // it, keys per run: 32 x 300 on 3300, 787, 38.5, 40.6; 12 x 1000 on 4000, 700, 41.5, 45.8; 12 x 1000 on 7000, 1300, 59.7, 58.4;
    // 32 x 512 on 6512, 1564, 78, 72; 32 x 300 on 6300, 1537, 62, 53; 32 x 1000 on 7000, 3250, 139, 114)
    const long long avg_keys = causal ? (long long)Nk - Nq / 2 : (long long)Nk;
    const bool long_runs = D == 128 && !p.kv_stream && opt[FA_OPT_FWD_MODE] != FA_MODE_WIDE &&
                           avg_keys / pl.nsplit >= 1400;
    const int key = (dtype << 2) | ((D == 128) << 1) | (causal ? 1 : 0);
    switch (key) {
        case 0: e = launch_splitkv<0, 64, false>(p, pl.grid_x, rows, long_runs, st); break;
        case 1: e = launch_splitkv<0, 64, true>(p, pl.grid_x, rows, long_runs, st); break;
        case 2: e = launch_splitkv<0, 128, false>(p, pl.grid_x, rows, long_runs, st); break;
        case 3: e = launch_splitkv<0, 128, true>(p, pl.grid_x, rows, long_runs, st); break;
        case 4: e = launch_splitkv<1, 64, false>(p, pl.grid_x, rows, long_runs, st); break;
        case 5: e = launch_splitkv<1, 64, true>(p, pl.grid_x, rows, long_runs, st); break;
        case 6: e = launch_splitkv<1, 128, false>(p, pl.grid_x, rows, long_runs, st); break;
        case 7: e = launch_splitkv<1, 128, true>(p, pl.grid_x, rows, long_runs, st); break;
        default: return FA_ERR_SHAPE;
    }
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return FA_ERR_LAUNCH;
    }
    return FA_OK;
}

int fa_fwd_splitkv(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int Nq, int Nk,
                   int D, float scale, int causal, int dtype, int nsplit, void *workspace, long long workspace_bytes,
                   void *stream) {
    return splitkv(options_now(), q, k, v, o, lse, B, H, Nq, Nk, D, scale, causal, dtype, nsplit, workspace, workspace_bytes, stream);
}

int fa_fwd_splitkv_static(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int Nq,
                          int Nk, int D, float scale, int causal, int dtype, int nsplit, void *stream) {
    const Options opt = options_now();
    // every argument check first (no HIP call before them), the size limit among them
    if (!q || !k || !v || !o || !lse) return FA_ERR_NULL;
    fa_splitkv_plan_t pl;
    const int rc = splitkv_plan(opt, B, H, Nq, Nk, D, dtype, nsplit, &pl);
    if (rc != FA_OK) return rc;
    if (!isfinite(scale)) return FA_ERR_SCALE;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return FA_ERR_ALIGN;
    if ((uintptr_t)lse & 3) return FA_ERR_ALIGN;
    if (pl.nsplit == 1) return fwd(opt, q, k, v, o, lse, B, H, Nq, Nk, D, scale, causal, dtype, stream);   // nothing to merge
    if (pl.workspace_bytes > FA_STATIC_WORKSPACE_BYTES) return FA_ERR_WORKSPACE;
    void *ws = nullptr;
    {
        // the array's device address on the current GPU, asked for once per device and kept
        constexpr int MAX_DEVICES = 64;
        static std::mutex lock;
        static void *address[MAX_DEVICES] = {};
        int dev = -1;
        hipError_t e = hipGetDevice(&dev);
        if (e == hipSuccess && (dev < 0 || dev >= MAX_DEVICES)) e = hipErrorInvalidDevice;
        if (e == hipSuccess) {
            std::lock_guard<std::mutex> guard(lock);
            if (!address[dev]) {
                void *ptr = nullptr;
                e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
                if (e == hipSuccess && !ptr) e = hipErrorInvalidSymbol;
                if (e == hipSuccess) address[dev] = ptr;
            }
            ws = address[dev];
        }
        if (e != hipSuccess) {
            g_last_hip_error = (int)e;
            return FA_ERR_LAUNCH;
        }
    }
    return splitkv(opt, q, k, v, o, lse, B, H, Nq, Nk, D, scale, causal, dtype, nsplit, ws, FA_STATIC_WORKSPACE_BYTES, stream);
}

int fa_fwd_masked(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int Nq, int Nk,
                  int D, float scale, const fa_mask_t *mask, int dtype, void *stream) {
    if (!q || !k || !v || !o || !lse || !mask) return FA_ERR_NULL;
    const int rc = check_shape(B, H, Nq, Nk, D, dtype);
    if (rc != FA_OK) return rc;
    if (!isfinite(scale)) return FA_ERR_SCALE;
    MaskGeom g;
    const int mrc = mask_geometry(mask, Nk, Nq, Nk, &g);
    if (mrc != FA_OK) return mrc;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return FA_ERR_ALIGN;
    if (((uintptr_t)lse | (uintptr_t)mask->kv_len) & 3) return FA_ERR_ALIGN;

    const Options opt = options_now();
    const int rows = masked_rows(opt[FA_OPT_FWD_MODE], g, (long long)B * H, Nq, Nk, D);
    const long long nqt = ((long long)Nq + rows - 1) / rows;
    const long long nwork = (long long)B * H * nqt;
    FaParams p = base_params(q, k, v, o, lse, H, Nq, Nk, nqt, nwork, scale);
    p.left = g.left;
    p.right = g.right;
    p.prefix = mask->prefix < Nk ? mask->prefix : Nk;
    p.kv_len = mask->kv_len;
    p.anchor = mask->diag_from_kv_len;
    const int grid = p.per_xcd * 8;
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;
    if (use_streaming_decode(opt, Nq)) {
        // one query per head: the streaming kernel walks the prefix and the window as runs of consecutive keys
        switch ((dtype << 1) | (D == 128)) {
            case 0: e = launch_decode_masked<0, 64>(p, (int)nwork, st); break;
            case 1: e = launch_decode_masked<0, 128>(p, (int)nwork, st); break;
            case 2: e = launch_decode_masked<1, 64>(p, (int)nwork, st); break;
            default: e = launch_decode_masked<1, 128>(p, (int)nwork, st); break;
        }
        if (e != hipSuccess) {
            g_last_hip_error = (int)e;
            return FA_ERR_LAUNCH;
        }
        return FA_OK;
    }
    switch ((dtype << 1) | (D == 128)) {
        case 0: e = launch_masked<0, 64>(p, rows, grid, st); break;
        case 1: e = launch_masked<0, 128>(p, rows, grid, st); break;
        case 2: e = launch_masked<1, 64>(p, rows, grid, st); break;
        default: e = launch_masked<1, 128>(p, rows, grid, st); break;
    }
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return FA_ERR_LAUNCH;
    }
    return FA_OK;
}

int fa_decode_masked(const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int Nk, int D,
                     float scale, const fa_mask_t *mask, int dtype, int nsplit, void *workspace,
                     long long workspace_bytes, void *stream) {
    if (!q || !k || !v || !o || !lse || !mask) return FA_ERR_NULL;
    fa_splitkv_plan_t pl;
    const int rc = splitkv_plan(options_now(), B, H, 1, Nk, D, dtype, nsplit, &pl);
    if (rc != FA_OK) return rc;
    if (!isfinite(scale)) return FA_ERR_SCALE;
    MaskGeom g;
    const int mrc = mask_geometry(mask, Nk, 1, Nk, &g);
    if (mrc != FA_OK) return mrc;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o) & 15) return FA_ERR_ALIGN;
    if (((uintptr_t)lse | (uintptr_t)mask->kv_len) & 3) return FA_ERR_ALIGN;
    const long long heads = (long long)B * H;
    // not the plan's number where that counts the pieces a head is cut into: equal runs of each head
    int shares = choose_nsplit(B, H, 1, Nk, D, nsplit, pl.streaming != 0, false).nsplit;
    if (shares > 1) {
        if (!workspace || workspace_bytes < shares * heads * (D + 2) * 4) return FA_ERR_WORKSPACE;
        if ((uintptr_t)workspace & 15) return FA_ERR_ALIGN;
    }
    FaParams p = base_params(q, k, v, o, lse, H, 1, Nk, 1, heads, scale);
    p.left = g.left;
    p.right = g.right;
    p.prefix = mask->prefix < Nk ? mask->prefix : Nk;
    p.kv_len = mask->kv_len;
    p.anchor = mask->diag_from_kv_len;
    // chosen by the library: a number of workgroups just past one per compute unit would take a second round for the few
    // (1 x 40 heads of 30000 keys: 320 workgroups 78 us, 240 68)
    if (nsplit <= 0 && heads * shares > 256 && heads * shares < 448 && 256 / heads * heads >= 192) shares = (int)(256 / heads);
    p.nsplit = shares;
    p.part_o = (float *)workspace;
    p.part_ml = p.part_o + (size_t)shares * heads * D;
    if (merges_itself(shares, D)) p.tag = decode_tag();
    hipStream_t st = (hipStream_t)stream;
    hipError_t e;
    switch ((dtype << 1) | (D == 128)) {
        case 0: e = launch_decode_masked<0, 64>(p, (int)heads, st); break;
        case 1: e = launch_decode_masked<0, 128>(p, (int)heads, st); break;
        case 2: e = launch_decode_masked<1, 64>(p, (int)heads, st); break;
        default: e = launch_decode_masked<1, 128>(p, (int)heads, st); break;
    }
    if (e != hipSuccess) {
        g_last_hip_error = (int)e;
        return FA_ERR_LAUNCH;
    }
    return FA_OK;
}

namespace {

int check_attn_linear(const void *q, const void *k, const void *v, const void *w, void *o, float *lse, float *y,
                      int B, int H, int Nq, int Nk, int D, int N, float scale, int dtype, int row_first, int row_count) {
    if (!q || !k || !v || !w || !o || !lse || !y) return FA_ERR_NULL;
    const int rc = check_shape(B, H, Nq, Nk, D, dtype);
    if (rc != FA_OK) return rc;
    if (N <= 0 || N % 256 != 0 || (long long)N * H * D * 2 > 0x7fffffffLL) return FA_ERR_SHAPE;
    if ((long long)Nq * D * 2 > 0x7fffffffLL) return FA_ERR_SHAPE;          // 32-bit offsets inside one head of o
    if (row_first < 0 || row_count <= 0 || (long long)row_first + row_count > Nq) return FA_ERR_SHAPE;
    if (!isfinite(scale)) return FA_ERR_SCALE;
    if (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)o | (uintptr_t)w) & 15) return FA_ERR_ALIGN;
    if (((uintptr_t)lse | (uintptr_t)y) & 3) return FA_ERR_ALIGN;
    return FA_OK;
}

// attention of one block of rows, every head: a launch over row_count rows whose diagonal is shifted by
// row_first; q, o, lse keep the full tensors' head pitch.  Arguments already checked.
int block_attention(const Options &opt, const void *q, const void *k, const void *v, void *o, float *lse, int B, int H, int Nq, int Nk,
                    int D, float scale, int causal, int dtype, int row_first, int row_count, hipStream_t st) {
    {
        // (the keys the block's rows can see end at its last row's diagonal)
        const int nk_seen = causal ? Nk - (Nq - row_first - row_count) : Nk;
        const Decomposition dec = choose_mode(opt, B, H, row_count, nk_seen > 0 ? nk_seen : 1, D, causal, dtype);
        const int BM = dec.rows;
        const long long nqt = ((long long)row_count + BM - 1) / BM;
        const long long nwork = (long long)B * H * nqt;
        FaParams p = base_params((const uint16_t *)q + (size_t)row_first * D, k, v, (uint16_t *)o + (size_t)row_first * D,
                                 lse + row_first, H, row_count, Nk, nqt, nwork, scale);
        p.q_rows = Nq;
        p.off = Nk - Nq + row_first;
        const hipError_t e = launch_attention(p, dec, D, causal, dtype, p.per_xcd * 8, st);
        if (e != hipSuccess) {
            g_last_hip_error = (int)e;
            return FA_ERR_LAUNCH;
        }
    }
    return FA_OK;
}

// the block's rows of y = (heads side by side) x w; `shared`: beside the next block's attention.  Arguments already checked.
int block_projection(const Options &opt, const void *w, const void *o, float *y, int B, int H, int Nq, int D, int N, int dtype,
                     int row_first, int row_count, bool shared, hipStream_t st) {
    {
        LinParams lp;
        lp.o = (const uint16_t *)o;
        lp.w = (const uint16_t *)w;
        lp.y = y;
        lp.H = H;
        lp.q_rows = Nq;
        lp.N = N;
        lp.s0 = row_first;
        lp.rows = row_count;
        lp.d_shift = D == 128 ? 7 : 6;
        const LinearTile t = choose_linear_tile(opt[FA_OPT_LINEAR_TILE], B, row_count, N, shared);
        lp.n_tiles = N / t.cols;
        lp.mt_per_b = (row_count + t.rows - 1) / t.rows;
        const long long tiles = (long long)B * lp.mt_per_b * lp.n_tiles;
        if (tiles > 0x7ffffff0LL) return FA_ERR_SHAPE;
        lp.ntile_total = (int)tiles;
        lp.per_xcd = (int)((tiles + 7) / 8);
        lp.panel = linear_panel(lp.per_xcd, t, B * lp.mt_per_b);
        if (const int v = opt[FA_OPT_LINEAR_PANEL]; v >= 1)   // tests, tuning
            lp.panel = v < B * lp.mt_per_b ? v : B * lp.mt_per_b;
        const hipError_t e = dtype == FA_DTYPE_F16 ? launch_linear<0>(lp, t, st) : launch_linear<1>(lp, t, st);
        if (e != hipSuccess) {
            g_last_hip_error = (int)e;
            return FA_ERR_LAUNCH;
        }
    }
    return FA_OK;
}

// fa_attn_linear's second stream (default priority) and the two events that tie it to the caller's stream, one
// set per device, created on the first call that may create them (not under stream capture) and kept until the
// process ends.  `busy` serialises the enqueueing of calls that share them.
struct SideStream {
    hipStream_t stream = nullptr;
    hipEvent_t attn_done = nullptr, joined = nullptr;
    bool ready = false;
    std::mutex busy;
};
SideStream g_side[64];

}  // namespace

int fa_attn_linear_block(const void *q, const void *k, const void *v, const void *w, void *o, float *lse, float *y,
                         int B, int H, int Nq, int Nk, int D, int N, float scale, int causal, int dtype,
                         int row_first, int row_count, void *stream) {
    int rc = check_attn_linear(q, k, v, w, o, lse, y, B, H, Nq, Nk, D, N, scale, dtype, row_first, row_count);
    if (rc != FA_OK) return rc;
    const Options opt = options_now();
    hipStream_t st = (hipStream_t)stream;
    rc = block_attention(opt, q, k, v, o, lse, B, H, Nq, Nk, D, scale, causal, dtype, row_first, row_count, st);
    if (rc != FA_OK) return rc;
    return block_projection(opt, w, o, y, B, H, Nq, D, N, dtype, row_first, row_count, false, st);
}

int fa_attn_linear(const void *q, const void *k, const void *v, const void *w, void *o, float *lse, float *y, int B,
                   int H, int Nq, int Nk, int D, int N, float scale, int causal, int dtype, int rows_per_block,
                   void *stream) {
    if (rows_per_block <= 0 || rows_per_block >= Nq)
        return fa_attn_linear_block(q, k, v, w, o, lse, y, B, H, Nq, Nk, D, N, scale, causal, dtype, 0, Nq, stream);
    int rc = check_attn_linear(q, k, v, w, o, lse, y, B, H, Nq, Nk, D, N, scale, dtype, 0, Nq);
    if (rc != FA_OK) return rc;
    const Options opt = options_now();
    hipStream_t st = (hipStream_t)stream;

    // The projection of block i and the attention of block i + 1 touch different rows, so the projections go to
    // a second stream behind an event recorded after each attention launch: the tail of one kernel (its last
    // workgroups, its stores) then overlaps the head of the next instead of leaving compute units idle between
    // ten short launches.  The caller's stream waits for the second stream at the end, so to the caller the call
    // behaves as if everything had been enqueued on `stream`.
    SideStream *side = nullptr;
    std::unique_lock<std::mutex> hold;
    if (opt[FA_OPT_LINEAR_OVERLAP] != 0) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess || dev < 0 || dev >= 64) {
            g_last_hip_error = (int)e;
            return FA_ERR_LAUNCH;
        }
        hold = std::unique_lock<std::mutex>(g_side[dev].busy);
        if (!g_side[dev].ready) {
            hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
            e = hipStreamIsCapturing(st, &cap);
            if (e != hipSuccess) {
                g_last_hip_error = (int)e;
                return FA_ERR_LAUNCH;
            }
            if (cap == hipStreamCaptureStatusNone) {     // nothing is created while a capture is in progress
                SideStream &n = g_side[dev];
                e = hipStreamCreateWithFlags(&n.stream, hipStreamNonBlocking);
                if (e == hipSuccess) e = hipEventCreateWithFlags(&n.attn_done, hipEventDisableTiming);
                if (e == hipSuccess) e = hipEventCreateWithFlags(&n.joined, hipEventDisableTiming);
                if (e != hipSuccess) {
                    g_last_hip_error = (int)e;
                    return FA_ERR_LAUNCH;
                }
                n.ready = true;
            }
        }
        if (g_side[dev].ready) side = &g_side[dev];
        else hold.unlock();
    }

    // the first block is half size (section 4.2: nothing overlaps with the first block's computation)
    const int first = rows_per_block / 2 > 0 ? rows_per_block / 2 : rows_per_block;
    bool forked = false;
    for (int r = 0; r < Nq && rc == FA_OK;) {
        const int n = r == 0 ? first : (Nq - r < rows_per_block ? Nq - r : rows_per_block);
        rc = block_attention(opt, q, k, v, o, lse, B, H, Nq, Nk, D, scale, causal, dtype, r, n, st);
        if (rc != FA_OK) break;
        hipStream_t lin_stream = st;
        if (side) {
            hipError_t e = hipEventRecord(side->attn_done, st);
            if (e == hipSuccess) e = hipStreamWaitEvent(side->stream, side->attn_done, 0);
            if (e != hipSuccess) {
                g_last_hip_error = (int)e;
                rc = FA_ERR_LAUNCH;
                break;
            }
            forked = true;
            lin_stream = side->stream;
        }
        rc = block_projection(opt, w, o, y, B, H, Nq, D, N, dtype, r, n, side && Nq - r - n >= n / 2, lin_stream);
        r += n;
    }
    if (forked) {      // also after an error: the second stream must rejoin (a capture could not end otherwise)
        hipError_t e = hipEventRecord(side->joined, side->stream);
        if (e == hipSuccess) e = hipStreamWaitEvent(st, side->joined, 0);
        if (e != hipSuccess && rc == FA_OK) {
            g_last_hip_error = (int)e;
            rc = FA_ERR_LAUNCH;
        }
    }
    return rc;
}

int fa_mask_tile_class(const fa_mask_t *mask, int kv_len, int Nq, int Nk, int row_first, int row_last, int key_first) {
    MaskGeom g;
    const int rc = mask_geometry(mask, kv_len, Nq, Nk, &g);
    if (rc != FA_OK) return rc;
    if (row_first < 0 || row_last < row_first || row_last >= Nq || key_first < 0 || key_first >= Nk) return FA_ERR_SHAPE;
    if (key_first % BN) return FA_ERR_SHAPE;
    return tile_class(row_tiles(g, row_first, row_last), key_first / BN);
}

int fa_mask_tile_walk(const fa_mask_t *mask, int kv_len, int Nq, int Nk, int row_first, int row_last, int *tiles,
                      int capacity, int *count) {
    if (!count || (capacity > 0 && !tiles)) return FA_ERR_NULL;
    MaskGeom g;
    const int rc = mask_geometry(mask, kv_len, Nq, Nk, &g);
    if (rc != FA_OK) return rc;
    if (row_first < 0 || row_last < row_first || row_last >= Nq || capacity < 0) return FA_ERR_SHAPE;
    const TileSeq sq = tile_sequence(g, row_first, row_last);
    *count = sq.count;
    for (int j = 0; j < sq.count && j < capacity; ++j) tiles[j] = sq.tile(j);   // the kernel's own position -> tile map
    return FA_OK;
}

int fa_mask_interior_run(const fa_mask_t *mask, int kv_len, int Nq, int Nk, int wg_row_first, int wg_row_last,
                         int row_first, int row_last, int *first, int *count) {
    if (!first || !count) return FA_ERR_NULL;
    MaskGeom g;
    const int rc = mask_geometry(mask, kv_len, Nq, Nk, &g);
    if (rc != FA_OK) return rc;
    if (wg_row_first < 0 || wg_row_last < wg_row_first || wg_row_last >= Nq) return FA_ERR_SHAPE;
    if (row_first < wg_row_first || row_last < row_first || row_last > wg_row_last) return FA_ERR_SHAPE;
    const Run r = interior_run(row_tiles(g, row_first, row_last), tile_sequence(g, wg_row_first, wg_row_last), Nk);
    *first = r.first;
    *count = r.count;
    return FA_OK;
}

int fa_set_option(int opt, int value) {
    bool ok = value == FA_AUTO;
    switch (opt) {
        case FA_OPT_FWD_MODE:
            ok = ok || value == FA_MODE_SPLIT || value == FA_MODE_WIDE || value == FA_MODE_WIDE_FOLD || value == FA_MODE_WIDE64 ||
                 value == FA_MODE_WIDE4;
            break;
        case FA_OPT_DECODE_KERNEL: ok = ok || value == 0 || value == 1; break;
        case FA_OPT_LINEAR_TILE: ok = ok || value == 128 || value == 256 || value == 128128 || value == 64128; break;
        case FA_OPT_LINEAR_PANEL: ok = ok || value >= 1; break;
        case FA_OPT_LINEAR_OVERLAP: ok = ok || value == 0 || value == 1; break;
        default: return FA_ERR_OPTION;
    }
    if (!ok) return FA_ERR_OPTION;
    return g_options[opt].exchange(value, std::memory_order_relaxed);
}

const char *fa_strerror(int code) {
    switch (code) {
        case FA_OK: return "success";
        case FA_ERR_NULL: return "a required pointer is NULL";
        case FA_ERR_SHAPE: return "B, H, Nq, Nk must be positive and the problem must be indexable";
        case FA_ERR_HEADDIM: return "head dimension D must be 64 or 128";
        case FA_ERR_DTYPE: return "dtype must be 0 (fp16) or 1 (bf16)";
        case FA_ERR_SCALE: return "scale must be finite";
        case FA_ERR_ALIGN: return "q, k, v, o must be 16-byte aligned and lse 4-byte aligned";
        case FA_ERR_LAUNCH: return "the HIP runtime rejected the kernel launch";
        case FA_ERR_WORKSPACE:
            return "workspace is NULL or smaller than fa_fwd_splitkv_plan reports (fa_fwd_splitkv_static: the problem needs "
                   "more than the library's 64 MiB)";
        case FA_ERR_NSPLIT: return "nsplit exceeds 1024";
        case FA_ERR_MASK: return "mask descriptor: prefix must be >= 0 and a key count within 0..Nk";
        case FA_ERR_OPTION: return "fa_set_option: unknown option, or a value it does not take";
        default: return "unknown error code";
    }
}

int fa_version(void) { return 300; }

int fa_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"
