// gfx950 kernels of the mixed block-decode / prefill attention call and the
// C-ABI forward entry point that launches them.
//
// What is computed (Sangam paper, Sec. 2.1 and Sec. 2.2): dLLM attention is
// bidirectional, so each query row of an item attends to all L positions of
// its sequence; a block decode recomputes only its 32 block rows and reuses
// the request's approximately cached KV for every other position, a prefill
// brings (and writes back) its whole sequence. Batches mix both kinds
// (Sec. 4.1, Alg. 1); the KV cache is paged with 16-token pages (Sec. 5,
// Sec. 6.1).
//
// Kernels:
//   attn_tiles_kernel one work-group per plan tile: a context range of one
//                     item and KV head against up to 8 x 32 query rows; one
//                     tile per item, KV head and row block also copies the
//                     fresh K/V rows into their cache pages.
//                     Per wave: S^T = K Q^T with v_mfma_f32_32x32x16_bf16
//                     (each lane holds the scores of one query, so row max /
//                     row sum need one cross-half exchange), online softmax
//                     in the exp2 domain, P^T rounded to bf16 feeds
//                     O^T += V^T P^T directly from the score registers.
//                     K/V stream global -> LDS with global_load_lds_dwordx4
//                     into XOR-swizzled tiles (double buffered); V^T operands
//                     come from ds_read_b64_tr_b16 transposing reads. Output
//                     rows leave through LDS, whole rows per 16 lanes.
//   attn_mixed_kernel the same tiles, prefill-shaped ones and block decodes of
//                     one query head per KV head in one launch.
//   merge_kernel      combines split-context partial (O, LSE) in split order,
//                     in calls whose tiles do not do so themselves.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <mutex>
#include <string>
#include <type_traits>

#include "../../include/sangam_attn.h"
#include "mixed_order.h"
#include "nonce.h"
#include "plan_format.h"

namespace sangam {
void set_error(const std::string& msg);
void clear_error();
const PlanHeader* check_plan(const void* plan);
}  // namespace sangam

using namespace sangam;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

#define LDS __attribute__((address_space(3)))

struct AttnArgs {
    const TileRec* tiles;
    const ItemRec* items;
    const int32_t* page_ids;
    const uint16_t* q;
    const uint16_t* k_new;
    const uint16_t* v_new;
    uint16_t* k_cache;  // read (cached rows) and written (the fresh rows' pages)
    uint16_t* v_cache;
    uint16_t* out;
    float* lse;
    float* ws;
    const int32_t* positions;    // rows of per-token cached decodes (kItemPosList items)
    const uint32_t* page_info;   // per page of such items: listed slots and earlier rows
    int32_t hq;
    int32_t hkv;
    float scale_log2;
    uint64_t nonce;  // marks this call's split partials as written (0: merge_kernel merges)
};

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Asynchronous copy of one K or V page (16 key rows of one head) from global
// memory into LDS by one wave: IPP global_load_lds_dwordx4, each moving 1 KiB
// (lane l's 16 bytes land at the instruction's LDS base + 16 l). The
// instruction adds its offset field to the global and to the LDS address, so
// one M0 write serves the page: instruction j lands at dst + 1024 j, and the
// lane offsets of instruction j are given less 1024 j. Issued through inline
// assembly so that the compiler does not track the LDS write: it would
// otherwise wait for every copy in flight before any later LDS read,
// including the copies that prefetch the next stage into another buffer,
// which serialises the prefetch with the compute it should overlap. The
// kernels order the copies themselves: s_waitcnt vmcnt and a barrier before a
// staged buffer is read, a barrier before it is overwritten. M0 is saved and
// restored around the copies, with the wait state the hardware needs between
// an M0 write and its use. Nor does the compiler count wait states into the
// block: a base it has just restored from a spill (v_readlane) is read five
// wait states after at the earliest, so the first copy stands behind that many.
__device__ __forceinline__ uint32_t lds_wave_base(LDS void* p) {
    return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)p);
}
// from a wave-uniform base plus per-lane 32-bit byte offsets
template <int IPP>
__device__ __forceinline__ void copy_page(const void* base, const uint32_t (&off)[IPP], LDS void* dst) {
    uint32_t saved;
    static_assert(IPP == 2 || IPP == 4, "a page is 2 or 4 KiB");
    if constexpr (IPP == 4)
        asm volatile(
            "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 2\n\t"
            "global_load_lds_dwordx4 %2, %6\n\tglobal_load_lds_dwordx4 %3, %6 offset:1024\n\t"
            "global_load_lds_dwordx4 %4, %6 offset:2048\n\tglobal_load_lds_dwordx4 %5, %6 offset:3072\n\t"
            "s_nop 0\n\ts_mov_b32 m0, %0"
            : "=&s"(saved)
            : "s"(lds_wave_base(dst)), "v"(off[0]), "v"(off[1]), "v"(off[2]), "v"(off[3]), "s"(base)
            : "memory");
    else
        asm volatile(
            "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 2\n\t"
            "global_load_lds_dwordx4 %2, %4\n\tglobal_load_lds_dwordx4 %3, %4 offset:1024\n\t"
            "s_nop 0\n\ts_mov_b32 m0, %0"
            : "=&s"(saved)
            : "s"(lds_wave_base(dst)), "v"(off[0]), "v"(off[1]), "s"(base)
            : "memory");
}
// the same from per-lane addresses
template <int IPP>
__device__ __forceinline__ void copy_page(const uint64_t (&addr)[IPP], LDS void* dst) {
    uint32_t saved;
    if constexpr (IPP == 4)
        asm volatile(
            "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
            "global_load_lds_dwordx4 %2, off\n\tglobal_load_lds_dwordx4 %3, off offset:1024\n\t"
            "global_load_lds_dwordx4 %4, off offset:2048\n\tglobal_load_lds_dwordx4 %5, off offset:3072\n\t"
            "s_nop 0\n\ts_mov_b32 m0, %0"
            : "=&s"(saved)
            : "s"(lds_wave_base(dst)), "v"(addr[0]), "v"(addr[1]), "v"(addr[2]), "v"(addr[3])
            : "memory");
    else
        asm volatile(
            "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\t"
            "global_load_lds_dwordx4 %2, off\n\tglobal_load_lds_dwordx4 %3, off offset:1024\n\t"
            "s_nop 0\n\ts_mov_b32 m0, %0"
            : "=&s"(saved)
            : "s"(lds_wave_base(dst)), "v"(addr[0]), "v"(addr[1])
            : "memory");
}

// Swizzle of 16-byte chunks inside a staged key row. K rows are read one key
// per lane (ds_read_b128), so 16 consecutive keys (4 KiB at D = 128; at
// D = 64 two keys share the 256 bytes of all banks) spread their chunks. V rows are
// read four keys at a time by ds_read_b64_tr_b16, so groups of four keys
// spread over the LDS banks.
template <int D>
__device__ __forceinline__ int swz_k(int r) {
    return D == 128 ? r & 15 : (r >> 1) & 7;
}
template <int D>
__device__ __forceinline__ int swz_v(int r) {
    return D == 128 ? ((r & 3) << 2) : (((r >> 1) & 1) << 2);
}

// Cross-half (lane l <-> l ^ 32) pair of a value: v_permlane32_swap with both
// operands x returns (x[l], x[l^32]) for the lower half and (x[l^32], x[l])
// for the upper half, so a symmetric combine of the two results is the pair's.
__device__ __forceinline__ float half_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float half_sum(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The running max moves only when a score exceeds it by more than this (log2
// units), so P <= 2^8 and O is rescaled rarely; the result is unchanged
// because O and l always share the same reference.
constexpr float kRescaleThreshold = 8.0f;

// Split partials cross the XCDs, whose L2s are not coherent: stores write
// through to memory and loads bypass the L2 (agent scope, sc1).
// The 16-byte store's data registers may be written again two wait states after
// it at the earliest, which the compiler does not see in assembly.
__device__ __forceinline__ void store_agent(float* p, float4 v) {
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(__builtin_bit_cast(u32x4, v)) : "memory");
}
__device__ __forceinline__ void store_agent(float* p, float v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float load_agent(const float* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
constexpr int kBufferAgent = 16;  // sc1 in a buffer load's cache policy

// Decode tiles of five to eight query heads at head dim 64 fit twice or three
// times on a CU with 128 registers a wave (four waves per SIMD), once or twice
// with the 165 they take otherwise. They get there with fragments read two steps
// ahead instead of four and with no more splits' sums than they merge. Measured
// with 165 -> 128 registers: 100 decodes of 1500 keys, 28/4 heads, 67.5 -> 61.2
// us, 150 of 20/4 95.0 -> 75.1, 250 of 64/8 304 -> 276; launches of up to one
// work-group per CU take the same time.
constexpr bool few_registers(int d, int qw, bool heads_across) { return d == 64 && heads_across && qw >= 5; }

// Waves per SIMD the register budget is sized for: two (256 registers) when a
// wave holds one query block.
constexpr int waves_per_simd(int qb, bool few) { return few ? 4 : qb == 1 ? 2 : 1; }

// LDS of a work-group
template <int BYTES>
struct TileShared {
    __attribute__((aligned(1024))) uint8_t stages[BYTES];  // K and V stage buffers
    int32_t wpages[kWaveRows];  // pages of the fresh rows this tile writes back
    int32_t fpos[kWaveRows];    // the listed positions (kItemPosList items)
    bool merging;               // this tile merges its rows' splits
};

// One work-group per plan tile: a context range [kv_begin, kv_end) of one
// item and KV head against QW query slots x QB blocks of 32 rows per slot.
//   D      head dim (64, 128)
//   QW     waves holding distinct query rows (query heads of a GQA group when
//          HEADS_ACROSS, else consecutive 32*QB-row blocks of one head)
//   KW     waves splitting each stage's keys (merged through LDS at the end)
//   QB     32-row query blocks per wave: every K and V fragment read from
//          LDS feeds QB MFMAs, so QB = 2 halves LDS traffic per flop
//   NB     32-key blocks per wave per stage
//   NSTAGE K/V stage buffers in LDS (NSTAGE - 1 stages in flight). 1: K and V
//          have one buffer each, and K of the next stage arrives while V of
//          this one is used, V while its K is
//   HELP   more waves, which only stage and write back
template <int D, int QW, int KW, int QB, int NB, int NSTAGE, bool HEADS_ACROSS, int HELP, typename Shared>
__device__ __forceinline__ void attn_tile(const AttnArgs& a, const TileRec t, const ItemRec it, Shared& shared) {
    constexpr int NT = 64 * (QW * KW + HELP);  // threads
    constexpr int KT = 32 * NB;          // keys per wave per stage
    constexpr int STEP = KT * KW;        // keys per stage
    constexpr int NC = D / 8;            // 16-byte chunks per key row
    constexpr int ROWB = D * 2;          // bytes per key row
    constexpr int TILE = STEP * ROWB;    // bytes of one staged K (or V) tile
    constexpr int NW = QW * KW + HELP;   // waves
    constexpr int SP = STEP / 16;        // 16-key pages per stage
    constexpr int PW = (SP + NW - 1) / NW;  // pages a wave copies per stage
    constexpr int RPI = 64 / NC;         // key rows per copy instruction
    constexpr int IPP = 16 / RPI;        // copy instructions per page
    constexpr int DS = D / 16;           // k-steps of the QK^T contraction
    constexpr int MB = D / 32;           // 32-dim blocks of O^T
    // MFMAs at raised wave priority: those of QK^T (1), of PV (2) or none (0).
    // Two waves share a SIMD. Measured: 128-key stages QK^T (long prefills
    // 6,510 us with PV, 6,480 with it), 64-key ones PV (Dream mixed batch 261
    // us with QK^T or none, 255 with it), D = 64 none (mixed batch 80.9 us
    // with PV, 76.4 without). Decode batches take the same time either way
    // (1 to 48 decodes, 14.8 to 78 us, within 0.2 %).
    constexpr int PRIO = D == 64 ? 0 : NB == 4 ? 1 : 2;
    constexpr bool FEW = few_registers(D, QW, HEADS_ACROSS);
    constexpr int RA = FEW ? 2 : 4;      // steps between a fragment's LDS read and its MFMA
    constexpr int MAXS = FEW ? max_merge_in_tile(QW) : kMaxMergeInTile;  // splits that a tile merges
    constexpr int MERGE_REGS = MB * 16 + 2;
    static_assert(KW == 1 || QB == 1, "context-splitting waves hold one query block");
    static_assert(!HEADS_ACROSS || QB == 1, "a decode block is 32 rows");
    static_assert(KW == 1 || (QW * KW * MERGE_REGS * 64 * 4) <= 2 * NSTAGE * TILE,
                  "cross-wave merge must fit in the stage buffers");
    static_assert(MB % KW == 0, "the waves of a query slot share its dims");
    static_assert(NSTAGE >= 1 && NSTAGE <= 4, "1 to 4 stage buffers");
    constexpr bool TURNS = NSTAGE == 1;  // K and V take turns
    static_assert(!TURNS || (KW == 1 && !HEADS_ACROSS && HELP == 0), "every wave meets the barrier between K and V");
    // pages a tile's write-back can touch: its rows at any offset, or one per listed row
    static_assert((32 * QB * QW + 15) / 16 + 1 <= kWaveRows && kWaveRows <= NT, "one thread per write-back page id");
    // with more than two buffers the wait counts loads, so every wave must
    // issue the same number per stage
    static_assert(NSTAGE <= 2 || SP % NW == 0, "deeper pipelines need whole staging rounds");
    static_assert(64 % SP == 0 && (NSTAGE - 1) * SP < 64, "a stage's page ids sit in one register of 64 lanes");

    static_assert(sizeof(shared.stages) >= 2 * NSTAGE * TILE, "the stage buffers");
    uint8_t* const smem = shared.stages;
    int32_t* const fpos = shared.fpos;
    int32_t* const wpages = shared.wpages;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = uniform(tid >> 6);
    const bool computes = HELP == 0 || wave < QW * KW;
    const int qs = computes ? wave % QW : 0;
    const int ks = computes ? wave / QW : 0;
    const int qn = lane & 31;   // query (column) this lane holds in each block
    const int hh = lane >> 5;   // half-wave

    // heads across the waves: a decode-shaped work-group, or a block decode
    // cut into a prefill-shaped one (whose last tile of a GQA group may hold
    // fewer heads than waves: the extra waves only stage K/V, write back and
    // meet the barriers; they compute and store nothing)
    const bool across = HEADS_ACROSS || (!TURNS && (t.flags & kTileHeadsAcross));
    const int head_want = across ? t.q_head0 + qs : t.q_head0;
    const bool head_ok = computes && head_want < (t.kv_head + 1) * (a.hq / a.hkv);
    const int head = head_ok ? head_want : t.q_head0;
    const int row_base = across ? t.row0 : t.row0 + 32 * QB * qs;
    const bool split_out = it.num_splits > 1;  // fp32 partials go to the workspace
    const bool merge_here = split_out && a.nonce != 0;
    const int kv_begin = t.kv_begin, kv_end = t.kv_end;
    const int nstages = (kv_end - kv_begin + STEP - 1) / STEP;
    // a whole prefill brings every position fresh: no page lookups
    const bool all_fresh = it.o == 0 && it.n == it.L;
    // a per-token cached decode: its rows sit at listed positions
    const bool plist = (it.flags & kItemPosList) != 0;
    const int pg0 = kv_begin >> 4;
    const int npg = ((kv_end + 15) >> 4) - pg0;
    // The tile's page ids (and page_info of kItemPosList items) sit in a
    // register, 64 at a time (lane l holds entry 64 c + l of chunk c): a stage
    // reads its ids with v_readlane, with no LDS or barrier in between.
    int32_t pv = 0;
    uint32_t iv = 0;
    auto load_pages = [&](int first) {
        const int k = it.page_start + pg0 + min(first + lane, npg - 1);
        pv = a.page_ids[k];
        if (plist) iv = a.page_info[k];
    };
    if (!all_fresh) load_pages(0);
    int32_t lpos = 0;  // the listed position of row `lane`, in every wave
    if (plist) lpos = a.positions[it.pos_start + min(lane, it.n - 1)];

    // ---- Q fragments (B operand: k = dims, n = query). Lanes past the last
    // row hold row 0 again: a query is a column of every product, so they
    // change no other row, and nothing of theirs is stored.
    bf16x8 qf[QB][DS];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int row = row_base + 32 * qb + qn;
        const uint16_t* qp = a.q + ((size_t)(it.q_start + (row < it.n ? row : 0)) * a.hq + head) * D;
#pragma unroll
        for (int s = 0; s < DS; ++s) qf[qb][s] = *(const bf16x8*)(qp + 16 * s + 8 * hh);
    }

    // ---- staging. A stage is SP pages of 16 key rows; wave w copies pages
    // w, w + NW, ... of it, K and V, IPP instructions each. Instruction j
    // covers rows RPI j + lane / NC; the lane's chunk of LDS row r is source
    // chunk (lane % NC) ^ swizzle(r). A work-group by itself is bound by its
    // serial chain of stages, and the scalar instructions of the copies stood
    // in it (about 110 per page; now about 20): one LLaDA decode 17.3 -> 16.6
    // us, a batch of 32 75.3 -> 74.1 us.
    const size_t row_stride = (size_t)a.hkv * D;                       // elements between positions
    const uint32_t row_bytes = uint32_t(row_stride * 2);
    const uint16_t* kfresh = a.k_new + ((size_t)(it.q_start - it.o) * a.hkv + t.kv_head) * D;
    const uint16_t* vfresh = a.v_new + ((size_t)(it.q_start - it.o) * a.hkv + t.kv_head) * D;
    const size_t page_stride = (size_t)a.hkv * 16 * D;
    const uint16_t* kcache = a.k_cache + (size_t)t.kv_head * 16 * D;
    const uint16_t* vcache = a.v_cache + (size_t)t.kv_head * 16 * D;

    // byte offsets of a lane's chunks from the first row of a page, less the
    // instruction's offset field: rows ROWB apart in the cache, row_bytes
    // apart among the fresh rows (row_bytes >= ROWB, so none is negative)
    uint32_t coff_k[IPP], coff_v[IPP], foff_k[IPP], foff_v[IPP];
#pragma unroll
    for (int j = 0; j < IPP; ++j) {
        const int r = RPI * j + lane / NC, pos = lane % NC;
        const uint32_t ck = uint32_t((pos ^ swz_k<D>(r)) << 4), cv = uint32_t((pos ^ swz_v<D>(r)) << 4);
        coff_k[j] = uint32_t(r * ROWB - 1024 * j) + ck;
        coff_v[j] = uint32_t(r * ROWB - 1024 * j) + cv;
        foff_k[j] = uint32_t(r) * row_bytes - 1024 * j + ck;
        foff_v[j] = uint32_t(r) * row_bytes - 1024 * j + cv;
    }

    // stages [mixed0, mixed1) may hold fresh rows beside cached ones (a block's,
    // or from the first to the last listed position), full_stages and on a
    // partial page
    const int last_pos = plist ? a.positions[it.pos_start + it.n - 1] : it.o + it.n - 1;
    const int full_stages = (kv_end - kv_begin) / STEP;
    const int mixed0 = all_fresh ? full_stages : min(full_stages, max(0, it.o - kv_begin) / STEP);
    const int mixed1 = all_fresh ? full_stages : last_pos < kv_begin ? 0 : (last_pos - kv_begin) / STEP + 1;
    const uint16_t* kfresh_w = kfresh + (int64_t)(kv_begin + wave * 16) * (int64_t)row_stride;
    const uint16_t* vfresh_w = vfresh + (int64_t)(kv_begin + wave * 16) * (int64_t)row_stride;
    const size_t stage_stride = STEP * row_stride;  // elements

    // do_k, do_v: whether to copy the stage's K rows and its V rows
    auto issue_stage = [&](int st, int buf, auto do_k, auto do_v) __attribute__((always_inline)) {
        uint8_t* kb = smem + buf * 2 * TILE;
        uint8_t* vb = kb + TILE;
        const int pl0 = st * SP & 63;  // lane holding the id of the stage's first page
        if (__builtin_expect(st < mixed0 || (st >= mixed1 && st < full_stages), 1)) {
            // a whole stage of one kind: wave-uniform bases, precomputed lane offsets
            const uint16_t* kf = kfresh_w + (size_t)unsigned(st) * stage_stride;
            const uint16_t* vf = vfresh_w + (size_t)unsigned(st) * stage_stride;
#pragma unroll
            for (int i = 0; i < PW; ++i) {
                const int k = wave + i * NW;  // page of the stage
                if (SP % NW != 0 && k >= SP) break;
                LDS void* kd = (LDS void*)(kb + k * 16 * ROWB);
                LDS void* vd = (LDS void*)(vb + k * 16 * ROWB);
                if (all_fresh) {
                    if (do_k) copy_page(kf + i * NW * 16 * row_stride, foff_k, kd);
                    if (do_v) copy_page(vf + i * NW * 16 * row_stride, foff_v, vd);
                } else {
                    const size_t off = size_t(uint32_t(__builtin_amdgcn_readlane(pv, pl0 + k))) * page_stride;
                    if (do_k) copy_page(kcache + off, coff_k, kd);
                    if (do_v) copy_page(vcache + off, coff_v, vd);
                }
            }
            return;
        }
        const int skey0 = kv_begin + st * STEP;
        for (int k = wave; k < SP; k += NW) {
            LDS void* kd = (LDS void*)(kb + k * 16 * ROWB);
            LDS void* vd = (LDS void*)(vb + k * 16 * ROWB);
            // a page past the range: the stage's first page again, masked later
            const bool past = skey0 + k * 16 >= kv_end;
            const int key0 = past ? skey0 : skey0 + k * 16;
            const int pl = past ? pl0 : pl0 + k;
            const uint32_t inf = plist ? uint32_t(__builtin_amdgcn_readlane(int(iv), pl)) : 0u;
            const size_t off = all_fresh ? 0 : (size_t)__builtin_amdgcn_readlane(pv, pl) * page_stride;
            if (key0 + 16 <= kv_end && !all_fresh &&
                (plist ? (inf & 0xFFFFu) == 0 : key0 + 16 <= it.o || key0 >= it.o + it.n)) {
                if (do_k) copy_page(kcache + off, coff_k, kd);
                if (do_v) copy_page(vcache + off, coff_v, vd);
                continue;
            }
            // fresh rows of a block, listed positions, the range's partial
            // last page (rows past its end repeat its last row)
            const int lim = min(16, kv_end - key0);
            // fresh rows of the page: row `first` onwards, in order
            const int64_t first = plist ? int64_t(it.q_start) + (inf >> kPageInfoRowShift)
                                        : int64_t(it.q_start) + key0 - it.o;
            const uint64_t fk = (uint64_t)(a.k_new + (size_t)t.kv_head * D) + uint64_t(first * int64_t(row_bytes));
            const uint64_t fv = (uint64_t)(a.v_new + (size_t)t.kv_head * D) + uint64_t(first * int64_t(row_bytes));
            uint64_t ak[IPP], av[IPP];
#pragma unroll
            for (int j = 0; j < IPP; ++j) {
                const int r = RPI * j + lane / NC, pos = lane % NC;
                const int rc = min(r, lim - 1);
                const bool fresh = plist ? (inf >> rc) & 1u : unsigned(key0 + rc - it.o) < unsigned(it.n);
                const uint32_t frow = plist ? __builtin_popcount(inf & ((1u << rc) - 1u)) : rc;
                const uint32_t ro = fresh ? frow * row_bytes : uint32_t(rc * ROWB);
                const int64_t lo = int64_t(ro) - 1024 * j;
                ak[j] = (fresh ? fk : (uint64_t)(kcache + off)) + uint64_t(lo + ((pos ^ swz_k<D>(r)) << 4));
                av[j] = (fresh ? fv : (uint64_t)(vcache + off)) + uint64_t(lo + ((pos ^ swz_v<D>(r)) << 4));
            }
            if (do_k) copy_page(ak, kd);
            if (do_v) copy_page(av, vd);
        }
    };

    // ---- write-back of the fresh K/V rows into their cache pages. Per item
    // and KV head, the tiles of the group's first query head copy the fresh
    // rows they stage (a prefill tile its own row block, a block decode its
    // rows) from LDS, right after the stage lands: no second read of k_new /
    // v_new. Every fresh position lies in exactly one such tile's row block
    // and context range. No tile reads these cache rows (fresh positions come
    // from k_new / v_new, and the planner rejects pages shared between items),
    // so the copy needs no ordering with the attention. The pages written are
    // kept in LDS (one per page of a block, one per listed row), so the copy
    // loop issues no global load whose wait would also drain the prefetch.
    const int group = a.hq / a.hkv;
    const bool wb_head = across ? t.q_head0 == t.kv_head * group : t.q_head0 % group == 0;
    // positions written: [wb_lo, wb_hi) for a block; for a position list (a
    // decode, so heads-across), its listed positions inside the span from the
    // first to the last listed position
    const int wb_lo = max(kv_begin, it.o + (across ? 0 : t.row0));
    const int wb_hi = min(kv_end, across ? last_pos + 1 : it.o + min(it.n, t.row0 + 32 * QB * QW));
    const bool writer = wb_head && wb_lo < wb_hi;
    const int wpg0 = wb_lo >> 4;
    const int wst0 = writer ? (wb_lo - kv_begin) / STEP : nstages;  // stages [wst0, wst1) hold such rows
    const int wst1 = writer ? (wb_hi - 1 - kv_begin) / STEP + 1 : 0;
    auto write_back = [&](int st, auto do_k, auto do_v) {
        const int key0 = kv_begin + st * STEP;
        const int lo = max(wb_lo, key0), hi = min(wb_hi, key0 + STEP);
        if (lo >= hi) return;
        const uint8_t* kb = smem + (st % NSTAGE) * 2 * TILE;
        const uint8_t* vb = kb + TILE;
        if (plist) {  // the listed positions inside [lo, hi): a run of the list
            const uint64_t in = __builtin_amdgcn_ballot_w64(lane < it.n && lpos >= lo && lpos < hi);
            const int first = __builtin_ctzll(in | 1ull << 63), count = __builtin_popcountll(in);
            for (int cidx = tid; cidx < count * NC; cidx += NT) {
                const int row = first + cidx / NC, p = fpos[row], pos = cidx % NC;
                const int r = p - key0;
                const u32x4 kv = *(const LDS u32x4*)(kb + r * ROWB + ((pos ^ swz_k<D>(r)) << 4));
                const u32x4 vv = *(const LDS u32x4*)(vb + r * ROWB + ((pos ^ swz_v<D>(r)) << 4));
                const size_t dst = (((size_t)wpages[row] * a.hkv + t.kv_head) * 16 + (p & 15)) * D + pos * 8;
                if (do_k) *(u32x4*)(a.k_cache + dst) = kv;
                if (do_v) *(u32x4*)(a.v_cache + dst) = vv;
            }
            return;
        }
        for (int cidx = tid; cidx < (hi - lo) * NC; cidx += NT) {
            const int p = lo + cidx / NC, pos = cidx % NC;
            const int r = p - key0;
            const u32x4 kv = *(const LDS u32x4*)(kb + r * ROWB + ((pos ^ swz_k<D>(r)) << 4));
            const u32x4 vv = *(const LDS u32x4*)(vb + r * ROWB + ((pos ^ swz_v<D>(r)) << 4));
            const size_t dst = (((size_t)wpages[(p >> 4) - wpg0] * a.hkv + t.kv_head) * 16 + (p & 15)) * D + pos * 8;
            if (do_k) *(u32x4*)(a.k_cache + dst) = kv;
            if (do_v) *(u32x4*)(a.v_cache + dst) = vv;
        }
    };

    // ---- stage-invariant LDS read offsets
    // K (A operand): lane reads key qn of each 32-key block, chunk 2k + hh of
    // k-step k: koff ^ (k << 5)
    const uint32_t koff = qn * ROWB + ((hh ^ swz_k<D>(qn)) << 4);
    // V^T (A operand) via transposing reads: 16-lane group g16 covers dims
    // mb*32 + (g16&1)*16 .. +15; lane (r4, j4) points at key row 4hh + r4 (+8),
    // dims 4 j4 .. 4 j4 + 3 of that group: voff ^ (mb << 6)
    const int g16 = lane >> 4;
    const int r4 = (lane >> 2) & 3;
    const int j4 = lane & 3;
    const int vdim = (g16 & 1) * 16 + 4 * j4;
    const uint32_t voff = (4 * hh + r4) * ROWB + (((vdim >> 3) ^ swz_v<D>(4 * hh + r4)) << 4) + (vdim & 7) * 2;
    const uint32_t lds0 = lds_wave_base((LDS void*)smem);

    f32x16 o[QB][MB];
    float m_used[QB];  // reference max (log2 domain) of this lane's query, per block
    float l_run[QB];   // sum of rounded P over this lane's half of the keys
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_used[qb] = -INFINITY;
        l_run[qb] = 0.0f;
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[qb][mb][i] = 0.0f;
    }
    const float c = a.scale_log2;

    // One stage of this wave: S^T = K Q^T (rows = keys, columns = queries; NB
    // 32-key blocks, each K fragment feeding the QB query blocks), online
    // softmax (exp2 domain), O^T += V^T P^T. tail: the stage may hold keys past
    // the range (set to -inf).
    //
    // The order of instructions is fixed here, MFMA by MFMA
    // (sched_barrier(0) after each step): the operand fragments form one
    // stream, K's then V's, each read from LDS RA steps before its MFMA; a
    // block's row max is taken beside the next block's QK^T and the
    // exponentials of the next 16 keys beside the PV of these. Left to the
    // compiler, most MFMAs sat right behind the LDS read they wait for (about
    // 130 cycles each), which a second wave on the SIMD hides in part only.
    // Measured per 64-key stage, K/V in L2, one 128-row work-group on the CU:
    // 1.30 -> 1.16 us at D = 128, 1.07 -> 0.85 us at D = 64; two: 1.98 -> 1.96
    // us and 1.32 -> 1.24 us (at D = 128 two work-groups draw the power limit:
    // the same MFMAs on random operands without the rest take 1.33 us).
    // between: called when the wave is done with the stage's K and is to read its V
    auto attend = [&](int st, auto tail, auto between) __attribute__((always_inline)) {
        constexpr bool TAIL = decltype(tail)::value;
        constexpr int NK = NB * DS;      // K fragments (and QK^T steps)
        constexpr int NV = NB * 2 * MB;  // V fragments (and PV steps)
        const uint32_t buf = lds0 + (st % NSTAGE) * 2 * TILE + ks * KT * ROWB;
        const uint32_t ka = buf + koff, va = buf + TILE + voff;
        auto read_frag = [&](int n) -> bf16x8 {
            if (n < NK) return *(const LDS bf16x8*)(uintptr_t)((ka ^ uint32_t((n % DS) << 5)) + (n / DS) * 32 * ROWB);
            const int v = n - NK;  // 16 keys v / MB, 32 dims v % MB
            const uint32_t vp = (va ^ uint32_t((v % MB) << 6)) + (v / MB) * 16 * ROWB;
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS bf16x4*)(uintptr_t)vp);
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((LDS bf16x4*)(uintptr_t)(vp + 8 * ROWB));
            return bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        };
        f32x16 s[QB][NB];
        float mx[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) mx[qb] = -INFINITY;
        // row max over scores [i0, i1) of block b
        auto take_max = [&](int b, int i0, int i1) {
#pragma unroll
            for (int i = i0; i < i1; ++i) {
                const int key = kv_begin + st * STEP + ks * KT + b * 32 + 8 * (i >> 2) + 4 * hh + (i & 3);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    if (TAIL && key >= kv_end) s[qb][b][i] = -INFINITY;
                    mx[qb] = fmaxf(mx[qb], s[qb][b][i]);
                }
            }
        };

        bf16x8 frag[RA];
#pragma unroll
        for (int n = 0; n < RA; ++n) frag[n] = read_frag(n);
        if (PRIO == 1) __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NK; ++n) {
            const int b = n / DS, k = n % DS;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                if (k == 0)
#pragma unroll
                    for (int i = 0; i < 16; ++i) s[qb][b][i] = 0.0f;
                s[qb][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[n % RA], qf[qb][k], s[qb][b], 0, 0, 0);
            }
            if (!TURNS || n + RA < NK) frag[n % RA] = read_frag(n + RA);
            // the previous block's scores are written two steps into this one
            if (b > 0 && k >= 2) take_max(b - 1, (k - 2) * 16 / (DS - 2), (k - 1) * 16 / (DS - 2));
            __builtin_amdgcn_sched_barrier(0);
        }
        if (PRIO == 1) __builtin_amdgcn_s_setprio(0);
        take_max(NB - 1, 0, 16);

        // The reference max moves (and O, l are rescaled) only when a score
        // exceeds it by more than kRescaleThreshold, which is rare after the
        // first stage.
        bool any_need = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            mx[qb] = half_max(mx[qb]) * c;
            any_need |= mx[qb] > m_used[qb] + kRescaleThreshold;
        }
        if (__builtin_amdgcn_ballot_w64(any_need)) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const bool need = mx[qb] > m_used[qb] + kRescaleThreshold;
                const float alpha = need ? __builtin_amdgcn_exp2f(m_used[qb] - mx[qb]) : 1.0f;
                m_used[qb] = need ? mx[qb] : m_used[qb];
                l_run[qb] *= alpha;
#pragma unroll
                for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                    for (int i = 0; i < 16; ++i) o[qb][mb][i] *= alpha;
            }
        }

        if constexpr (TURNS) {
            between();
#pragma unroll
            for (int n = NK; n < NK + RA; ++n) frag[n % RA] = read_frag(n);
            __builtin_amdgcn_sched_barrier(0);
        }

        // P = exp2(s c - m) rounded to bf16 (the PV operand); l += the rounded
        // values. Lane slot j of the P^T of 16 keys kk holds key
        // 16kk + 8(j/4) + 4hh + j%4.
        bf16x8 pf[QB][NB * 2];
        float mneg[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) mneg[qb] = m_used[qb] == -INFINITY ? 0.0f : -m_used[qb];
        auto exps = [&](int kk, int j0, int j1) {
#pragma unroll
            for (int j = j0; j < j1; j += 2)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    const f32x16& sb = s[qb][kk >> 1];
                    const int i = 8 * (kk & 1) + j;
                    const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sb[i], c, mneg[qb]));
                    const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sb[i + 1], c, mneg[qb]));
                    const bf16x2 pp = {(__bf16)p0, (__bf16)p1};
                    l_run[qb] = __builtin_amdgcn_fdot2_f32_bf16(pp, bf16x2{(__bf16)1.0f, (__bf16)1.0f}, l_run[qb], false);
                    pf[qb][kk][j] = pp[0];
                    pf[qb][kk][j + 1] = pp[1];
                }
        };
        exps(0, 0, 8);
        if (PRIO == 2) __builtin_amdgcn_s_setprio(1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int n = 0; n < NV; ++n) {
            const int kk = n / MB, mb = n % MB;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
                o[qb][mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(frag[(NK + n) % RA], pf[qb][kk], o[qb][mb], 0, 0, 0);
            if (n + RA < NV) frag[(NK + n) % RA] = read_frag(NK + n + RA);
            if (kk + 1 < NB * 2) exps(kk + 1, mb * 8 / MB, (mb + 1) * 8 / MB);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (PRIO == 2) __builtin_amdgcn_s_setprio(0);
    };

    // Stages st+1 .. st+NSTAGE-1 are in flight while stage st is computed.
    // Loads complete in order, so waiting for stage st leaves the later
    // stages outstanding.
    constexpr int LPS = 2 * IPP * PW;  // loads per stage per wave (K and V)
    auto wait_stage = [&](int st) {
        const int later = min(NSTAGE - 2, nstages - 1 - st);  // stages issued after st
        if (NSTAGE >= 4 && later >= 2)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * LPS) : "memory");
        else if (NSTAGE >= 3 && later >= 1)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LPS) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    // The compiler does not see the copies, so it would make the first use of
    // Q wait for every one in flight: Q is waited for here, with the page ids
    // or the first stage, which are needed at this point anyway.
    auto wait_q = [&]() {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int s = 0; s < DS; ++s) asm volatile("" : "+v"(qf[qb][s]));
    };
    if (NSTAGE > 2) wait_q();
    // the next 64 page ids, once stage st has read the last of these
    auto next_pages = [&](int st) {
        if (!all_fresh && ((st + 1) * SP & 63) == 0 && (st + 1) * SP < npg) load_pages((st + 1) * SP);
    };
    // the write-back's pages: loaded before the first copies, kept in LDS after
    const int nwp = writer ? plist ? it.n : ((wb_hi + 15) >> 4) - wpg0 : 0;
    int32_t wpage = 0;
    if (tid < nwp) wpage = a.page_ids[it.page_start + (plist ? lpos >> 4 : wpg0 + tid)];
    constexpr auto yes = std::true_type{};
    constexpr auto no = std::false_type{};
    for (int k = 0; k < NSTAGE - 1 && k < nstages; ++k) issue_stage(k, k, yes, yes);
    if (TURNS) issue_stage(0, 0, yes, no);
    if (NSTAGE <= 2) wait_q();
    if (tid < nwp) {
        wpages[tid] = wpage;
        if (plist) fpos[tid] = lpos;
    }
    int st = 0;
    if constexpr (TURNS) {
        // a stage: its K is there, V on its way under QK^T, the next K under PV
        auto stage = [&](auto tail) __attribute__((always_inline)) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            issue_stage(st, 0, no, yes);
            next_pages(st);
            if (st >= wst0 && st < wst1) write_back(st, yes, no);
            attend(st, tail, [&]() __attribute__((always_inline)) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if (st + 1 < nstages) issue_stage(st + 1, 0, yes, no);
                if (st >= wst0 && st < wst1) write_back(st, no, yes);
            });
        };
        for (; st < full_stages; ++st) stage(std::false_type{});
        if (st < nstages) stage(std::true_type{});
    } else {
        auto go_on = []() {};
        for (; st < full_stages; ++st) {
            wait_stage(st);
            __syncthreads();
            if (st + NSTAGE - 1 < nstages) {
                issue_stage(st + NSTAGE - 1, (st + NSTAGE - 1) % NSTAGE, yes, yes);
                next_pages(st + NSTAGE - 1);
            }
            if (st >= wst0 && st < wst1) write_back(st, yes, yes);
            if (head_ok) attend(st, std::false_type{}, go_on);  // a wave past its tile's GQA group only stages and writes back
        }
        if (st < nstages) {  // the last, partial stage
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            if (st >= wst0 && st < wst1) write_back(st, yes, yes);
            if (head_ok) attend(st, std::true_type{}, go_on);
        }
    }

    // ---- combine the context sub-ranges of the waves that share query rows:
    // each of the KW waves then holds MBW of the MB 32-dim blocks of O
    constexpr int MBW = MB / KW;
    const int mb0 = ks * MBW;  // first block of this wave
    if constexpr (KW > 1) {
        __syncthreads();
        float* mbuf = reinterpret_cast<float*>(smem) + (size_t)qs * KW * MERGE_REGS * 64;
        float* mine = mbuf + (size_t)ks * MERGE_REGS * 64;
        if (computes) {
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) mine[(mb * 16 + i) * 64 + lane] = o[0][mb][i];
            mine[(MB * 16) * 64 + lane] = m_used[0];
            mine[(MB * 16 + 1) * 64 + lane] = l_run[0];
        }
        __syncthreads();
        static_assert(KW == 2, "sums of two");
        const float* src[2] = {mbuf, mbuf + MERGE_REGS * 64};
        const float m_tot = fmaxf(src[0][(MB * 16) * 64 + lane], src[1][(MB * 16) * 64 + lane]);
        // wave ks = 0 always holds a valid key, so m_tot is finite
        float sc[2], l[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            sc[k] = __builtin_amdgcn_exp2f(src[k][(MB * 16) * 64 + lane] - m_tot);
            l[k] = src[k][(MB * 16 + 1) * 64 + lane];
        }
        // Which product of a sum is fused is written out: the compiler may
        // take either, and another build would differ in the last bits.
        const float l1 = sc[1] * l[1];
        l_run[0] = __builtin_fmaf(sc[0], l[0], l1);
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int at = ((mb0 + mb) * 16 + i) * 64 + lane;
                const float o0 = sc[0] * src[0][at];
                o[0][mb][i] = __builtin_fmaf(sc[1], src[1][at], o0);
            }
        m_used[0] = m_tot;
    }

    // ---- epilogue: O / l and the LSE, to the output or as a split's partial
    float lse_val[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const float l_tot = half_sum(l_run[qb]);
        const float inv = 1.0f / l_tot;
        lse_val[qb] = m_used[qb] * 0.69314718055994530942f + logf(l_tot);
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
            for (int i = 0; i < 16; ++i) o[qb][mb][i] *= inv;
    }
    if (split_out) {
        if (!merge_here) {
            // rows of D for merge_kernel: [split][row][head]
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                const int row = row_base + 32 * qb + qn;
                if (!head_ok || row >= it.n) continue;
                const size_t prow = (size_t)(t.split * it.n + row) * a.hq + head;
                float* po = a.ws + it.ws_o + prow * D;
#pragma unroll
                for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4)
                        *(float4*)(po + (mb0 + mb) * 32 + 8 * q4 + 4 * hh) =
                            float4{o[qb][mb][4 * q4], o[qb][mb][4 * q4 + 1], o[qb][mb][4 * q4 + 2], o[qb][mb][4 * q4 + 3]};
                if (hh == 0 && ks == 0) a.ws[it.ws_lse + prow] = lse_val[qb];
            }
            return;
        }
        // For a merge by a tile like this one: [split][head][rows of 32]
        // [D / 4][row] float4 and [split][head][row] LSE, so that a wave's
        // store, and its load by the merging wave, of one register is 16-byte
        // pieces of consecutive rows.
        const size_t rows0 = (size_t)(t.split * a.hq + head) * it.n;  // rows before this (split, head)
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int r0 = row_base + 32 * qb, nb = min(32, it.n - r0);
            if (!head_ok || qn >= nb) continue;
            float* po = a.ws + it.ws_o + (rows0 + r0) * D;
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const int d4 = (mb0 + mb) * 8 + q4 * 2 + hh;
                    const float4 v = {o[qb][mb][4 * q4], o[qb][mb][4 * q4 + 1], o[qb][mb][4 * q4 + 2], o[qb][mb][4 * q4 + 3]};
                    store_agent(po + (size_t)(d4 * nb + qn) * 4, v);
                }
            if (hh == 0 && ks == 0) store_agent(a.ws + it.ws_lse + rows0 + r0 + qn, lse_val[qb]);
        }
        // The tile that finds every split of its rows written merges them.
        // Each tile marks its split with the call's nonce, then looks at all
        // marks: both are read-modify-writes, complete before the next, so
        // the last tile to mark finds all of them. Two tiles may, and then
        // write the same bits. The merging tile clears the marks, so that a
        // replayed graph, whose nonce repeats, starts from none; whatever
        // else the workspace held is not this call's 64-bit nonce.
        uint64_t* marks = reinterpret_cast<uint64_t*>(a.ws + merge_marks(it, a.hq)) +
                          (size_t)((t.row0 / kWaveRows) * a.hq + t.q_head0) * it.num_splits;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's partials are in memory
        __syncthreads();
        if (wave == 0) {
            uint64_t before = 0, none = 0;
            if (lane == 0) before = __hip_atomic_exchange(marks + t.split, a.nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" : "+v"(before), "+v"(none)::"memory");
            bool there = true;
            if (lane < it.num_splits)
                there = __hip_atomic_fetch_or(marks + lane, none, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.nonce;
            const bool all = __builtin_amdgcn_ballot_w64(there) == ~0ull;
            if (all && lane < it.num_splits)
                __hip_atomic_store(marks + lane, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (lane == 0) shared.merging = all;
        }
        __syncthreads();
        if (!shared.merging) return;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            const int r0 = row_base + 32 * qb, nb = min(32, it.n - r0);
            if (!head_ok || nb <= 0) continue;
            const int row = min(qn, nb - 1);  // lanes past the last row repeat it
            const size_t step = (size_t)a.hq * it.n;  // rows between splits
            const size_t first = (size_t)head * it.n + r0;
            float ls[MAXS], mx = -INFINITY;
#pragma unroll
            for (int k = 0; k < MAXS; ++k)
                if (k < it.num_splits) ls[k] = load_agent(a.ws + it.ws_lse + k * step + first + row);
#pragma unroll
            for (int k = 0; k < MAXS; ++k)
                if (k < it.num_splits) mx = fmaxf(mx, ls[k]);
            f32x16 acc[MBW];
            float tot = 0.0f;
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc[mb][i] = 0.0f;
#pragma unroll 2
            for (int k = 0; k < it.num_splits; ++k) {
                const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(
                    a.ws + it.ws_o + (k * step + first) * D, 0, nb * D * 4, 0x00027000);
                u32x4 v[MBW * 4];
#pragma unroll
                for (int j = 0; j < MBW * 4; ++j) {
                    const int d4 = (mb0 + j / 4) * 8 + (j & 3) * 2 + hh;
                    v[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (d4 * nb + row) * 16, 0, kBufferAgent);
                }
                float w = 0.0f;
#pragma unroll
                for (int m = 0; m < MAXS; ++m)
                    if (m == k) w = __expf(ls[m] - mx);
                tot += w;
#pragma unroll
                for (int j = 0; j < MBW * 4; ++j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) acc[j / 4][4 * (j & 3) + e] += w * __uint_as_float(v[j][e]);
            }
            const float inv = 1.0f / tot;
#pragma unroll
            for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[qb][mb][i] = acc[mb][i] * inv;
            lse_val[qb] = mx + logf(tot);
        }
    }
    // Output rows leave through LDS where it holds them: each lane stages its
    // query's dims in 8-byte pieces, then 16 consecutive lanes store one whole
    // row in 16-byte pieces (stored directly, one instruction would leave
    // 16-byte fragments of 32 rows).
    constexpr int EROW = D * 2 + 16;  // bytes per staged row: 16-byte aligned, shifted by four banks
    constexpr int EBASE = KW > 1 ? QW * KW * MERGE_REGS * 64 * 4 : 0;  // past the waves' partials
    constexpr bool ESTAGE = EBASE + QW * QB * 32 * EROW <= 2 * NSTAGE * TILE;
    if constexpr (ESTAGE && KW == 1) {
        if (!split_out) __syncthreads();  // every wave is past its last stage's reads
    }
    uint8_t* ebuf = smem + EBASE + qs * (QB * 32 * EROW);
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int row = row_base + 32 * qb + qn;
        const bool stored = row < it.n && head_ok;
        uint16_t* op = a.out + ((size_t)(it.q_start + row) * a.hq + head) * D;
#pragma unroll
        for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                const int dim = (mb0 + mb) * 32 + 8 * q4 + 4 * hh;
                const bf16x4 v = {(__bf16)o[qb][mb][4 * q4], (__bf16)o[qb][mb][4 * q4 + 1],
                                  (__bf16)o[qb][mb][4 * q4 + 2], (__bf16)o[qb][mb][4 * q4 + 3]};
                if (ESTAGE && !computes) continue;
                if (ESTAGE) *(LDS u32x2*)(ebuf + (32 * qb + qn) * EROW + dim * 2) = __builtin_bit_cast(u32x2, v);
                else if (stored) *(u32x2*)(op + dim) = __builtin_bit_cast(u32x2, v);
            }
        if (stored && hh == 0 && ks == 0 && a.lse) a.lse[(size_t)(it.q_start + row) * a.hq + head] = lse_val[qb];
    }
    if constexpr (ESTAGE) {
        // with one wave per query slot a wave reads back only rows it staged
        if constexpr (KW > 1) __syncthreads();
        else asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (head_ok) {
            constexpr int CPR = D / 8;           // 16-byte pieces per row
            constexpr int NCE = QB * 32 * CPR;   // pieces per query slot
            static_assert(NCE % (64 * KW) == 0, "whole rounds of 64 lanes");
#pragma unroll
            for (int j = 0; j < NCE / (64 * KW); ++j) {
                const int c = (j * KW + ks) * 64 + lane;
                const int r = c / CPR, col = c % CPR;  // staged row r is row row_base + r
                if (row_base + r < it.n) {
                    const u32x4 v = *(const LDS u32x4*)(ebuf + r * EROW + col * 16);
                    *(u32x4*)(a.out + ((size_t)(it.q_start + row_base + r) * a.hq + head) * D + col * 8) = v;
                }
            }
        }
    }
}

template <int D, int QW, int KW, int QB, int NB, int NSTAGE, bool HEADS_ACROSS>
__global__ __launch_bounds__(64 * QW * KW, waves_per_simd(QB, few_registers(D, QW, HEADS_ACROSS))) void attn_tiles_kernel(AttnArgs a) {
    __shared__ TileShared<2 * NSTAGE * 32 * NB * KW * D * 2> shared;
    const TileRec t = a.tiles[blockIdx.x];
    attn_tile<D, QW, KW, QB, NB, NSTAGE, HEADS_ACROSS, 0>(a, t, a.items[t.item], shared);
}

// Prefill-shaped tiles and the block decodes of one query head per KV head
// (which no prefill-shaped tile takes) in one launch, where the planner finds
// that faster than one for each (launch_each_kind): the former are bound by
// the matrix cores and the latter by HBM, so they run beside each other, one
// of each per CU as far as they last. Both are four waves and hold 64 KiB of
// LDS; two waves of a decode only stage. Prefill tiles of 256 rows (WIDE) are
// taken as two of 128 that keep their 128-key stages, so that a prefill's sums
// are those of a launch without decodes, bit for bit: K and V have one buffer
// each and take turns (with two of 64 keys each, 16 decodes beside 1819 and
// 1201 rows, 32/32 heads, take 195 us instead of 199, but the sums differ by
// 2e-3).
// Order: `round` prefill tiles (one per CU), as many decodes, then groups of
// eight blocks (one per XCD) of either kind in the ratio of what is left.
// Measured on the same batch: 231 us in two launches, 198 in this one (the order
// was taken with the 64-key halves: 194 us, all prefill tiles first 206, all
// decodes first 212, no first round 197).
struct MixedArgs {
    AttnArgs a;                   // tiles: the prefill-shaped ones
    const TileRec* decode_tiles;
    MixedOrder order;
};

template <int D, bool WIDE>
__global__ __launch_bounds__(256, 2) void attn_mixed_kernel(MixedArgs m) {
    __shared__ TileShared<2 * 2 * 64 * D * 2> shared;
    const MixedBlock b = mixed_block(m.order, blockIdx.x);
    if (b.index < 0) return;
    if (b.decode) {
        const TileRec t = m.decode_tiles[b.index];
        attn_tile<D, 1, 2, 1, 1, 2, true, 2>(m.a, t, m.a.items[t.item], shared);
        return;
    }
    TileRec t = m.a.tiles[WIDE ? b.index >> 1 : b.index];
    const ItemRec it = m.a.items[t.item];
    if (WIDE) t.row0 += kPrefillRows * (b.index & 1);
    if (t.row0 < it.n) attn_tile<D, 4, 1, 1, WIDE ? 4 : 2, WIDE ? 1 : 2, false, 0>(m.a, t, it, shared);
}

// --------------------------------------------------------------- split merge
struct MergeArgs {
    const MergeRow* rows;
    const ItemRec* items;
    const float* ws;
    uint16_t* out;
    float* lse;
    int32_t hq;
    int32_t d;
};

// grid: (merge row, 256-element slice of the row's Hq x D/4 float4 outputs);
// one thread per float4 of one head, so that every partial of a row is
// loaded by a different thread in parallel.
__global__ __launch_bounds__(256) void merge_kernel(MergeArgs a) {
    const MergeRow mr = a.rows[blockIdx.x];
    const ItemRec it = a.items[mr.item];
    const int S = it.num_splits;
    const int d4n = a.d / 4;
    const int e = blockIdx.y * 256 + threadIdx.x;
    if (e >= a.hq * d4n) return;
    const int head = e / d4n;
    const int d4 = e - head * d4n;
    float mx = -INFINITY;
    for (int s = 0; s < S; ++s) mx = fmaxf(mx, a.ws[it.ws_lse + (size_t)(s * it.n + mr.row) * a.hq + head]);
    float tot = 0.0f;
    float4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int s = 0; s < S; ++s) {
        const size_t prow = (size_t)(s * it.n + mr.row) * a.hq + head;
        const float w = __expf(a.ws[it.ws_lse + prow] - mx);
        const float4 v = *(const float4*)(a.ws + it.ws_o + prow * a.d + 4 * d4);
        tot += w;
        acc.x += w * v.x;
        acc.y += w * v.y;
        acc.z += w * v.z;
        acc.w += w * v.w;
    }
    const float inv = 1.0f / tot;
    const bf16x4 v = {(__bf16)(acc.x * inv), (__bf16)(acc.y * inv), (__bf16)(acc.z * inv), (__bf16)(acc.w * inv)};
    const size_t orow = (size_t)(it.q_start + mr.row) * a.hq + head;
    *(u32x2*)(a.out + orow * a.d + 4 * d4) = __builtin_bit_cast(u32x2, v);
    if (d4 == 0 && a.lse) a.lse[orow] = mx + logf(tot);
}

// ------------------------------------------------------------------ launch
// Start / stop events attached to one launch (timed entry point), or none.
struct LaunchEvents {
    hipEvent_t start = nullptr;
    hipEvent_t stop = nullptr;
};

// A launch with events carries them in its dispatch (hipExtLaunchKernel), so
// their timestamps bracket the kernel itself, as a kernel trace does.
template <typename Args>
hipError_t launch(const void* fn, dim3 grid, unsigned threads, Args args, hipStream_t stream, LaunchEvents ev) {
    void* kargs[] = {&args};
    if (!ev.start && !ev.stop) return hipLaunchKernel(fn, grid, dim3(threads), kargs, 0, stream);
    return hipExtLaunchKernel(fn, grid, dim3(threads), kargs, 0, stream, ev.start, ev.stop, 0);
}

template <int D, int QW, int KW, int QB, int NB, bool HA, int NSTAGE = 2>
hipError_t launch_tiles(const AttnArgs& args, int n_tiles, hipStream_t stream, LaunchEvents ev) {
    return launch(reinterpret_cast<const void*>(&attn_tiles_kernel<D, QW, KW, QB, NB, NSTAGE, HA>),
                  dim3(unsigned(n_tiles)), unsigned(64 * QW * KW), args, stream, ev);
}

template <int D>
hipError_t launch_decode(const AttnArgs& args, int n_tiles, int qw, int kw, int nb, hipStream_t stream,
                         LaunchEvents ev, bool* supported) {
    *supported = true;
    if (qw == 1 && kw == 2 && nb == 1) return launch_tiles<D, 1, 2, 1, 1, true>(args, n_tiles, stream, ev);
    if (qw == 2 && kw == 2 && nb == 2) return launch_tiles<D, 2, 2, 1, 2, true>(args, n_tiles, stream, ev);
    if (kw == 1 && nb == 2) {
        switch (qw) {
            case 3: return launch_tiles<D, 3, 1, 1, 2, true>(args, n_tiles, stream, ev);
            case 4: return launch_tiles<D, 4, 1, 1, 2, true>(args, n_tiles, stream, ev);
            case 5: return launch_tiles<D, 5, 1, 1, 2, true>(args, n_tiles, stream, ev);
            case 6: return launch_tiles<D, 6, 1, 1, 2, true>(args, n_tiles, stream, ev);
            case 7: return launch_tiles<D, 7, 1, 1, 2, true>(args, n_tiles, stream, ev);
            case 8: return launch_tiles<D, 8, 1, 1, 2, true>(args, n_tiles, stream, ev);
            default: break;
        }
    }
    *supported = false;
    return hipSuccess;
}

sangam_status hip_fail(hipError_t e, const char* what) {
    set_error(std::string(what) + ": " + hipGetErrorString(e));
    return SANGAM_ERR_HIP;
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

// ---------------------------------------------------------- allocation-free
// Split-KV partial results of sangam_attn_forward_noalloc live in this array
// instead of a caller workspace. Each GPU the library runs on holds its own
// copy for the life of the process. In host code the name is only a stand-in
// for the symbol: kernels receive the device address that hipGetSymbolAddress
// returns for the current device, cached per device below.
namespace {
// beside them the merge marks of any plan with that many bytes of partials
// (at worst 256 bytes of marks to 768 of partials: two splits of one row)
constexpr size_t kScratchMarks = kScratchBytes / 3 + 4096;
static __device__ __align__(256) uint8_t scratch[kScratchBytes + kScratchMarks];

constexpr int kMaxScratchDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_dev[kMaxScratchDevices] = {};

// the scratch array's address on the device that runs `stream`, which must
// be the current device (the symbol is resolved with that device current)
sangam_status scratch_address(hipStream_t stream, void** addr) {
    int cur = -1;
    if (hipError_t e = hipGetDevice(&cur); e != hipSuccess) return hip_fail(e, "hipGetDevice");
    if (stream) {
        hipDevice_t sd = -1;
        if (hipError_t e = hipStreamGetDevice(stream, &sd); e != hipSuccess) return hip_fail(e, "hipStreamGetDevice");
        if (int(sd) != cur) {
            set_error("the stream belongs to device " + std::to_string(int(sd)) + ", the current device is " +
                      std::to_string(cur));
            return SANGAM_ERR_INVALID_ARG;
        }
    }
    if (cur < 0 || cur >= kMaxScratchDevices) {
        set_error("device ordinal " + std::to_string(cur) + " beyond the scratch table");
        return SANGAM_ERR_UNSUPPORTED;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_dev[cur]) {
        void* p = nullptr;
        if (hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)); e != hipSuccess)
            return hip_fail(e, "hipGetSymbolAddress(scratch)");
        g_scratch_dev[cur] = p;
    }
    *addr = g_scratch_dev[cur];
    return SANGAM_OK;
}
}  // namespace

static sangam_status forward_impl(const void* plan_host, const void* plan_dev, const void* q,
                                  const void* k_new, const void* v_new, void* k_cache, void* v_cache,
                                  int64_t pool_pages, const int32_t* page_ids_dev, int64_t num_page_ids,
                                  void* out, float* lse, void* workspace, size_t workspace_bytes,
                                  void* stream_ptr, void* const* events, bool use_scratch = false) {
    clear_error();
    const PlanHeader* h = check_plan(plan_host);
    if (!h) {
        set_error("plan_host is not a plan of this library version");
        return SANGAM_ERR_PLAN;
    }
    if (!plan_dev || !q || !k_new || !v_new || !k_cache || !v_cache || !page_ids_dev || !out) {
        set_error("plan_dev, q, k_new, v_new, k_cache, v_cache, page_ids_dev and out must not be NULL");
        return SANGAM_ERR_INVALID_ARG;
    }
    if (!aligned16(plan_dev) || !aligned16(q) || !aligned16(k_new) || !aligned16(v_new) ||
        !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out) ||
        (reinterpret_cast<uintptr_t>(page_ids_dev) & 3u) || (lse && (reinterpret_cast<uintptr_t>(lse) & 3u))) {
        set_error("tensors must be 16-byte aligned (page_ids and lse 4-byte aligned)");
        return SANGAM_ERR_ALIGN;
    }
    if (pool_pages < h->num_pool_pages) {
        set_error("the plan addresses " + std::to_string(h->num_pool_pages) + " pool pages, the cache holds " +
                  std::to_string(pool_pages));
        return SANGAM_ERR_BUFFER;
    }
    if (num_page_ids < h->total_pages) {
        set_error("the plan reads " + std::to_string(h->total_pages) + " page ids, page_ids_dev holds " +
                  std::to_string(num_page_ids));
        return SANGAM_ERR_BUFFER;
    }
    if (use_scratch && h->workspace_bytes > 0) {
        // the allocation-free entry point: split partials go to the scratch array
        if (size_t(h->workspace_bytes - h->mark_bytes) > kScratchBytes || size_t(h->mark_bytes) > kScratchMarks) {
            set_error("the plan's split partials need " + std::to_string(h->workspace_bytes - h->mark_bytes) +
                      " bytes; the allocation-free forward holds " + std::to_string(kScratchBytes));
            return SANGAM_ERR_BUFFER;
        }
        if (sangam_status st = scratch_address(static_cast<hipStream_t>(stream_ptr), &workspace); st != SANGAM_OK)
            return st;
        workspace_bytes = kScratchBytes + kScratchMarks;
    }
    if (h->workspace_bytes > 0) {
        if (!workspace || workspace_bytes < size_t(h->workspace_bytes)) {
            set_error("workspace needs " + std::to_string(h->workspace_bytes) + " bytes");
            return SANGAM_ERR_BUFFER;
        }
        if (!aligned16(workspace)) {
            set_error("workspace must be 16-byte aligned");
            return SANGAM_ERR_ALIGN;
        }
    }
    hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
    const uint8_t* pd = static_cast<const uint8_t*>(plan_dev);
    // events[2k], events[2k+1] bracket launch k (prefill-shaped, decode-shaped,
    // merge); a launch with no work records its pair back to back
    auto evs = [&](int k) {
        LaunchEvents ev;
        if (events) {
            ev.start = static_cast<hipEvent_t>(events[2 * k]);
            ev.stop = static_cast<hipEvent_t>(events[2 * k + 1]);
        }
        return ev;
    };
    auto mark_empty = [&](int k) -> hipError_t {
        const LaunchEvents ev = evs(k);
        for (hipEvent_t e : {ev.start, ev.stop})
            if (e)
                if (hipError_t r = hipEventRecord(e, stream); r != hipSuccess) return r;
        return hipSuccess;
    };
    const ItemRec* items = reinterpret_cast<const ItemRec*>(pd + h->off_items);

    AttnArgs args{nullptr,
                  items,
                  page_ids_dev,
                  static_cast<const uint16_t*>(q),
                  static_cast<const uint16_t*>(k_new),
                  static_cast<const uint16_t*>(v_new),
                  static_cast<uint16_t*>(k_cache),
                  static_cast<uint16_t*>(v_cache),
                  static_cast<uint16_t*>(out),
                  lse,
                  static_cast<float*>(workspace),
                  reinterpret_cast<const int32_t*>(pd + h->off_positions),
                  reinterpret_cast<const uint32_t*>(pd + h->off_page_info),
                  h->hq,
                  h->hkv,
                  h->scale_log2,
                  h->mark_bytes > 0 ? next_nonce() : 0};
    // 1. attention: prefill-shaped tiles (compute-bound) first, then
    // decode-shaped tiles; both also write the fresh rows into their pages
    const bool mixed = one_launch(*h);
    if (mixed) {
        const bool wide = h->prefill_rows == kWidePrefillRows;
        MixedArgs m{args, reinterpret_cast<const TileRec*>(pd + h->off_decode_tiles), {}};
        m.a.tiles = reinterpret_cast<const TileRec*>(pd + h->off_prefill_tiles);
        const int64_t round = h->cus > 0 ? h->cus : 256;  // one block of each kind per CU
        const int64_t blocks = mixed_order(&m.order, int64_t(h->n_prefill_tiles) << int(wide), h->n_decode_tiles, round);
        const void* fn = h->d == 64 ? reinterpret_cast<const void*>(&attn_mixed_kernel<64, false>)
                         : wide     ? reinterpret_cast<const void*>(&attn_mixed_kernel<128, true>)
                                    : reinterpret_cast<const void*>(&attn_mixed_kernel<128, false>);
        if (hipError_t e = launch(fn, dim3(unsigned(blocks)), 256u, m, stream, evs(0)); e != hipSuccess)
            return hip_fail(e, "mixed attention launch");
    } else if (h->n_prefill_tiles > 0) {
        args.tiles = reinterpret_cast<const TileRec*>(pd + h->off_prefill_tiles);
        hipError_t e;
        if (h->prefill_rows == kWidePrefillRows && h->d == 128)
            e = launch_tiles<128, kWidePrefillQWaves, 1, 1, 4, false>(args, h->n_prefill_tiles, stream, evs(0));
        else if (h->prefill_rows == kPrefillRows)
            e = h->d == 128
                    ? launch_tiles<128, kPrefillQWaves, 1, kPrefillQBlocks, 2, false>(args, h->n_prefill_tiles, stream, evs(0))
                    : launch_tiles<64, kPrefillQWaves, 1, kPrefillQBlocks, 2, false>(args, h->n_prefill_tiles, stream, evs(0));
        else {
            set_error("no prefill kernel for this tile shape");
            return SANGAM_ERR_UNSUPPORTED;
        }
        if (e != hipSuccess) return hip_fail(e, "prefill attention launch");
    } else if (hipError_t e = mark_empty(0); e != hipSuccess) {
        return hip_fail(e, "event record");
    }
    if (!mixed && h->n_decode_tiles > 0) {
        args.tiles = reinterpret_cast<const TileRec*>(pd + h->off_decode_tiles);
        bool ok = false;
        hipError_t e = h->d == 128 ? launch_decode<128>(args, h->n_decode_tiles, h->decode_qw, h->decode_kw,
                                                        h->decode_nb, stream, evs(1), &ok)
                                   : launch_decode<64>(args, h->n_decode_tiles, h->decode_qw, h->decode_kw,
                                                       h->decode_nb, stream, evs(1), &ok);
        if (!ok) {
            set_error("no decode kernel for this head grouping");
            return SANGAM_ERR_UNSUPPORTED;
        }
        if (e != hipSuccess) return hip_fail(e, "decode attention launch");
    } else if (hipError_t e = mark_empty(1); e != hipSuccess) {
        return hip_fail(e, "event record");
    }

    // 2. merge split contexts, unless the tiles do
    if (merge_launch(*h)) {
        MergeArgs m{reinterpret_cast<const MergeRow*>(pd + h->off_merge),
                    items,
                    static_cast<const float*>(workspace),
                    static_cast<uint16_t*>(out),
                    lse,
                    h->hq,
                    h->d};
        const unsigned slices = unsigned((h->hq * (h->d / 4) + 255) / 256);
        hipError_t e = launch(reinterpret_cast<const void*>(&merge_kernel), dim3(unsigned(h->n_merge_rows), slices),
                              256u, m, stream, evs(2));
        if (e != hipSuccess) return hip_fail(e, "merge launch");
    } else if (hipError_t e = mark_empty(2); e != hipSuccess) {
        return hip_fail(e, "event record");
    }
    return SANGAM_OK;
}

extern "C" sangam_status sangam_attn_forward(const void* plan_host, const void* plan_dev, const void* q,
                                             const void* k_new, const void* v_new, void* k_cache,
                                             void* v_cache, int64_t pool_pages, const int32_t* page_ids_dev,
                                             int64_t num_page_ids, void* out, float* lse, void* workspace,
                                             size_t workspace_bytes, void* stream) {
    clear_error();
    return forward_impl(plan_host, plan_dev, q, k_new, v_new, k_cache, v_cache, pool_pages, page_ids_dev,
                        num_page_ids, out, lse, workspace, workspace_bytes, stream, nullptr);
}

extern "C" size_t sangam_noalloc_scratch_bytes(void) { return kScratchBytes; }

extern "C" sangam_status sangam_attn_forward_noalloc(const void* plan_host, const void* plan_dev, const void* q,
                                                     const void* k_new, const void* v_new, void* k_cache,
                                                     void* v_cache, int64_t pool_pages,
                                                     const int32_t* page_ids_dev, int64_t num_page_ids,
                                                     void* out, float* lse, void* stream) {
    clear_error();
    return forward_impl(plan_host, plan_dev, q, k_new, v_new, k_cache, v_cache, pool_pages, page_ids_dev,
                        num_page_ids, out, lse, nullptr, 0, stream, nullptr, true);
}

extern "C" sangam_status sangam_attn_forward_timed(const void* plan_host, const void* plan_dev,
                                                   const void* q, const void* k_new, const void* v_new,
                                                   void* k_cache, void* v_cache, int64_t pool_pages,
                                                   const int32_t* page_ids_dev, int64_t num_page_ids,
                                                   void* out, float* lse, void* workspace,
                                                   size_t workspace_bytes, void* stream, void* const* events) {
    clear_error();
    if (!events) {
        set_error("events must not be NULL");
        return SANGAM_ERR_INVALID_ARG;
    }
    return forward_impl(plan_host, plan_dev, q, k_new, v_new, k_cache, v_cache, pool_pages, page_ids_dev,
                        num_page_ids, out, lse, workspace, workspace_bytes, stream, events);
}
