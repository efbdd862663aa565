// Device code of libmts.
//
//   k_arrivals  (mts_arrivals.hip) samples every arrival of a chunk of ticks
//               and sorts each tick's arrivals by tier.
//   k_step      the scheduling tick, a workgroup of one, four or eight waves
//               per replica for a whole chunk of ticks: per-instance summaries live in LDS, per-instance
//               O(1) work is lane-parallel (lane i <-> instance i), slot
//               state lives in HBM and is touched only by events.
//   k_init      empty clusters; k_digest the canonical state digest.
//
// Slot record (uint4 per slot): x = slot word, y = meta (in the kernels with a
// queue cache with a running request's place in its finish bucket from bit 8
// on), z = seq, w = arrival tick, so that an event reads or writes one 16-byte
// record.  Slot word (u32, bits 31..30 = status):
//   waiting   01 | rem (14 bits) | len (16 bits)
//   running   10 | fin mod 2^14  | final length (16 bits)
//   inbound   11 | 0 (with meta; seq and arrival tick keep whatever the slot
//             held last and are read as zero by the export and the digest)
//   empty     0 (the word alone marks an empty slot: meta, seq and arrival
//             tick keep whatever the slot held last; the export and the
//             digest read them as zero)
// A running request's word never changes while it runs: the tick at which it
// emits its last token (fin) and its final length determine its length at
// any tick t (final - (fin - t + 1) before the decode of t), so decoding
// writes nothing.  Its KV growth falls on ticks t with
// (final - fin - 1 + t) mod block = 0: per instance, counters indexed by that
// residue give the number of requests that need a new block at tick t in
// O(1).  A request that starts running is filed under its finish tick in a
// per-replica timing wheel, so a tick visits exactly the requests that
// finish in it.  The head of line of every instance is cached in LDS (slot,
// key, slot word, meta, arrival tick), so admission reads no HBM.
#include <hip/hip_runtime.h>

#include "mts_internal.h"
#include "mts_wave.h"

namespace mts {
namespace {

constexpr int kNstat = MTS_NSTAT;
constexpr int kTiers = MTS_MAX_TIERS;
constexpr unsigned long long kNone = ~0ull;
constexpr uint32_t kWaitW = 1u << 30, kRunW = 2u << 30, kInbW = 3u << 30;
constexpr uint32_t kFin = 0x3FFFu;
constexpr int kNoHol = -1, kHolUnknown = -2;
constexpr int kFlagAbort = 1, kFlagBusy = 2, kFlagIntf = 4;

__device__ __forceinline__ uint32_t wst(uint32_t v) { return v >> 30; }
__device__ __forceinline__ uint32_t wlo(uint32_t v) { return v & 0xFFFFu; }
__device__ __forceinline__ uint32_t wmid(uint32_t v) { return (v >> 16) & kFin; }

// ---------------------------------------------------------------------------
// LDS of one replica
// ---------------------------------------------------------------------------
constexpr int kInts = 18;
// placements of the previous tick's dispatch kept in LDS (at most one wave's worth)
constexpr int kLast = 64;
// requests preempted in the current tick, listed for the prefetched finish visit
constexpr int kVic = 16;
// kernels for more than 64 instances: up to this many pairs are picked one by one
// (about 450 cycles each; the whole order takes 11K)
constexpr int kPickPairs = 16;
// Section 6.5 extensions: words of the device table (u32; the addresses of
// the per-replica headroom and snapshot arrays as u64 at the end)
enum { kXSlo = 0, kXAge = 10, kXPromoMin = 20, kXPromoPeriod, kXAdaptEpoch, kXAdaptUp, kXAdaptDown, kXAdaptMax,
       kXAdaptMargin, kXZeroLowest, kXHqr = 28, kXHsnap = 30, kXWords = 32 };
static_assert(kXWords == MTS_EXT_WORDS, "extension table size");

struct LdsLayout {
    uint32_t stats, occ, holk, fd, ht, ints, res, tcnt, mig, last, vic, wc, wov, inf, qt, qn, xn, ext, blk, rsel, total;
};

// Waves per replica (NW): eight in the kernels for more than 64 instances
// (IM 128 and 256; the per-instance phases are spread over the waves, the
// serial ones stay on wave 0); one or, for overloaded clusters that leave the
// chip room, four in the others.

__host__ __device__ inline uint32_t al8(uint32_t x) { return (x + 7u) & ~7u; }

// Per-instance arrays are sized for IM instances (a power of two >= I, at
// least 16) and come first, so that their offsets are compile-time constants
// of the kernel instantiation; the arrays whose size depends on S, the block
// size or the wheel follow.
__host__ __device__ constexpr uint32_t imax_for(uint32_t I)
{
    return I <= 16 ? 16 : I <= 32 ? 32 : I <= 64 ? 64 : I <= 128 ? 128 : 256;
}

__host__ __device__ inline LdsLayout lds_layout(uint32_t IM, uint32_t I, uint32_t W, uint32_t RB, uint32_t wsz,
                                                uint32_t policy, uint32_t qdepth, bool ext, uint32_t nw)
{
    const bool wide = IM >= 128;
    LdsLayout L;
    uint32_t o = 0;
    L.stats = o; o += kNstat * 8;
    L.holk = o;  o += IM * 8;
    L.fd = o;    o += IM * 8;
    L.ht = o;    o += 64 * 4;
    L.ints = o;  o += IM * kInts * 4;
    L.tcnt = o;  o += IM * kTiers / 2 * 4;
    L.mig = o;   o += IM * 16;
    L.last = o;  o += kLast * 12 + 8;
    L.vic = o;   o += kVic * 4 + 8;
    L.occ = o;   o += I * W * 8;
    L.res = o;   o += ((I * RB + 1) / 2) * 4;
    L.wc = o;    o += (wsz / 2) * 4;
    L.wov = o;   o += ((wsz + 31) / 32) * 4;
    // INFaaS only: per instance this tick's finished end-to-end sum (u64), the
    // service-time estimate (i64), the finish count and the state penalty
    o = al8(o);
    L.inf = o;   o += policy == MTS_POLICY_INFAAS ? IM * 24 : 0;
    // queue cache: per instance the qdepth waiting requests after the head of
    // line, in (tier, seq) order, 16 bytes each, and their number
    o = (o + 15u) & ~15u;
    L.qt = o;    o += IM * qdepth * 16;
    L.qn = o;    o += qdepth ? IM * 8 : 0;
    // kernels for more than 64 instances: per instance the queue cache extension's head << 16 | count
    L.xn = o;    o += wide ? IM * 4 : 0;
    // adaptive headroom / promotion: the ticks left to the next promotion
    // pass and headroom update, and per instance a lower bound on the
    // arrival ticks of its waiting requests (the rest of their state stays
    // in HBM: it is touched only on pass and update ticks)
    o = al8(o);
    L.ext = o;   o += ext ? 8 + IM * 4 : 0;
    // multi-wave kernels: values the waves combine (the auto-scaling sum, an
    // abort flag, the work lists' lengths and next entries)
    o = al8(o);
    L.blk = o;   o += nw > 1 ? 40 : 0;
    // kernels for more than 64 instances: per wave 64 (key, slot | demand) pairs, the rescan's
    // selected requests before they are ranked (the dispatch's deferred
    // bursts and the pairing's sorted blocks of 64 (key, index) pairs use the
    // same bytes later in the tick)
    o = (o + 15u) & ~15u;
    L.rsel = o;  o += wide ? nw * 64 * 8 : 0;
    L.total = (o + 15u) & ~15u;
    return L;
}

struct Ctx {
    // LDS
    unsigned long long* stats;
    unsigned long long* occ;   // [I][W] slot not empty
    unsigned long long* holk;  // [I] head-of-line key tier << 32 | seq
    double* fd;                // [I] freeness num / max(B, 1) (exact order for S <= 2048)
    int* ht;                   // [64] headroom sums: [m] of tiers 0-4 in mask m, [32 + m] of tiers 5-9
    int *freeb, *B, *live, *nwait, *hols, *hold, *num, *held, *inb, *tmask, *flags, *gtmp, *order;
    int* drn;                  // [I] draining (infinite virtual-usage sentinel)
    int* frs;                  // [I] 1: every waiting request was placed by the previous tick's dispatch
    unsigned *lw, *lsl, *lsq;  // [kLast] previous tick's placements in dispatch order: slot word,
                               // instance << 16 | tier << 12 | slot, seq
    int* lastn;                // number of those placements
    unsigned* vic;             // [kVic] instance << 16 | slot of this tick's preemption victims
    int* nvic;                 // their number (above kVic: more than the list holds)
    unsigned *hwd, *hmt, *hta; // [I] head of line: slot word, meta, arrival tick
    unsigned* res;             // [RB][I] running requests per growth residue (u16 pairs)
    unsigned* tcnt;            // [I][10] running requests per tier (u16 pairs)
    int* mig;                  // [I][4] dst, src slot, dst slot, copied
    unsigned* wc;              // [wsz / 2] entries filed per wheel bucket, two u16 per word
    unsigned* wov;             // [wsz / 32] bucket overflowed since its last visit
    // INFaaS policy only (null otherwise), per instance
    unsigned long long* fsum;  // [I] end-to-end ticks of this tick's finishes
    long long* svc;            // [I] service-time estimate, 1/256 tick
    int *fcnt, *pen;           // [I] this tick's finishes; state penalty in ticks
    // queue cache behind the head of line (td entries per instance; td = 0: none):
    // entry {seq, slot word, arrival tick, slot | tier << 12 | admitted << 16}
    uint4* qt;                 // [I][td] a ring: entry k at (qh + k) mod td
    int* qn;                   // [I] cached entries
    int* qh;                   // [I] ring position of the first entry
    // kernels for more than 64 instances (null otherwise): behind the ring, further
    // waiting requests of the instance in order, a ring of xd entries in HBM
    int* xn;                   // [I] first entry << 16 | count
    uint4* qx;                 // [I][xd] this replica's extensions
    int xd;
    int td;
    uint32_t blind;            // 1: tiers order nothing (tier-blind scheduling)
    // adaptive headroom and promotion (null when both are off): the LDS
    // region read through the accessors below
    unsigned char* ext;
    // multi-wave kernels only (null otherwise): the block area, a 64-bit sum
    // and a flag the waves combine, the admission work list's length and the
    // next entry to hand out (the list itself is kept in order[])
    long long* bsum;
    int* bflag;
    int* wln;
    int* wlnext;
    int* e2go;                 // pairing runs this tick (set by wave 0)
    int* e2n2;                 // staged copies to start
    int* kcnt;                 // entries that stay in the visited finish bucket
    int *gln, *glnext;         // four-wave kernels: the preempting instances' list
                               // (in order[] too), its next entry
    uint2* rsel;               // this wave's 64 entries of the rescan selection buffer
    // HBM: timing wheel of this replica, slot arrays, latency histograms
    uint32_t* wheel;           // [wsz][wcap] instance << 16 | slot
    uint32_t* hist;            // [2][10][MTS_HIST_BINS] queue delay, end-to-end
    uint32_t wmask, wcap;
    uint4* slot;               // [I][S] slot records of this replica
    uint32_t I, S, W, RB, shift, bmask, M, K;
};

// Section 6.5 extension state in LDS, at fixed offsets from C.ext: the
// ticks left to the next promotion pass and headroom update, then per
// instance a lower bound lb on the arrival ticks of its waiting requests
// (0: unknown, the next pass reads the instance)
__device__ __forceinline__ int* xleft(const Ctx& C) { return reinterpret_cast<int*>(C.ext); }
__device__ __forceinline__ unsigned* wlb(const Ctx& C) { return reinterpret_cast<unsigned*>(C.ext + 8); }
// fields of slot record x
__device__ __forceinline__ uint32_t& s_word(const Ctx& C, size_t x) { return reinterpret_cast<uint32_t*>(C.slot + x)[0]; }
__device__ __forceinline__ uint32_t& s_meta(const Ctx& C, size_t x) { return reinterpret_cast<uint32_t*>(C.slot + x)[1]; }
__device__ __forceinline__ uint32_t& s_tarr(const Ctx& C, size_t x) { return reinterpret_cast<uint32_t*>(C.slot + x)[3]; }
// word and meta of slot record x in one 8-byte store
__device__ __forceinline__ void s_set_wm(const Ctx& C, size_t x, uint32_t w, uint32_t m)
{
    *reinterpret_cast<uint2*>(C.slot + x) = make_uint2(w, m);
}

// addresses of the per-replica headroom and snapshot arrays (null: static headroom)
__device__ __forceinline__ int32_t* ext_hqr(const Params& P)
{
    return reinterpret_cast<int32_t*>(reinterpret_cast<const unsigned long long*>(P.ext + kXHqr)[0]);
}
__device__ __forceinline__ unsigned long long* ext_hsnap(const Params& P)
{
    return reinterpret_cast<unsigned long long*>(reinterpret_cast<const unsigned long long*>(P.ext + kXHsnap)[0]);
}

template <int IM, bool INF, bool EXT, bool QC, int NW>
__device__ inline Ctx carve(char* base, const Params& P)
{
    const LdsLayout Y = lds_layout(IM, P.I, P.W, P.RB, P.wsz, P.policy, P.qdepth, EXT, NW);
    Ctx C;
    C.stats = reinterpret_cast<unsigned long long*>(base + Y.stats);
    C.occ = reinterpret_cast<unsigned long long*>(base + Y.occ);
    C.holk = reinterpret_cast<unsigned long long*>(base + Y.holk);
    C.fd = reinterpret_cast<double*>(base + Y.fd);
    C.ht = reinterpret_cast<int*>(base + Y.ht);
    int* p = reinterpret_cast<int*>(base + Y.ints);
    C.freeb = p; p += IM;
    C.B = p; p += IM;
    C.live = p; p += IM;
    C.nwait = p; p += IM;
    C.hols = p; p += IM;
    C.hold = p; p += IM;
    C.num = p; p += IM;
    C.held = p; p += IM;
    C.inb = p; p += IM;
    C.tmask = p; p += IM;
    C.flags = p; p += IM;
    C.gtmp = p; p += IM;
    C.order = p; p += IM;
    C.drn = p; p += IM;
    C.frs = p; p += IM;
    C.hwd = reinterpret_cast<unsigned*>(p); p += IM;
    C.hmt = reinterpret_cast<unsigned*>(p); p += IM;
    C.hta = reinterpret_cast<unsigned*>(p); p += IM;
    C.res = reinterpret_cast<unsigned*>(base + Y.res);
    C.tcnt = reinterpret_cast<unsigned*>(base + Y.tcnt);
    C.mig = reinterpret_cast<int*>(base + Y.mig);
    C.lw = reinterpret_cast<unsigned*>(base + Y.last);
    C.lsl = C.lw + kLast;
    C.lsq = C.lsl + kLast;
    C.lastn = reinterpret_cast<int*>(C.lsq + kLast);
    C.vic = reinterpret_cast<unsigned*>(base + Y.vic);
    C.nvic = reinterpret_cast<int*>(C.vic + kVic);
    C.wc = reinterpret_cast<unsigned*>(base + Y.wc);
    C.wov = reinterpret_cast<unsigned*>(base + Y.wov);
    C.td = QC ? int(P.qdepth) : 0;
    C.blind = P.blind;
    C.qt = reinterpret_cast<uint4*>(base + Y.qt);
    C.qn = reinterpret_cast<int*>(base + Y.qn);
    C.qh = C.qn + IM;
    C.xn = IM >= 128 ? reinterpret_cast<int*>(base + Y.xn) : nullptr;
    C.qx = nullptr;  // per replica, set with the slot records
    C.xd = int(P.qxd);
    if (INF) {
        C.fsum = reinterpret_cast<unsigned long long*>(base + Y.inf);
        C.svc = reinterpret_cast<long long*>(base + Y.inf + IM * 8);
        C.fcnt = reinterpret_cast<int*>(base + Y.inf + IM * 16);
        C.pen = C.fcnt + IM;
    } else {
        C.fsum = nullptr; C.svc = nullptr; C.fcnt = nullptr; C.pen = nullptr;
    }
    C.ext = EXT ? reinterpret_cast<unsigned char*>(base + Y.ext) : nullptr;
    C.bsum = NW > 1 ? reinterpret_cast<long long*>(base + Y.blk) : nullptr;
    C.bflag = NW > 1 ? reinterpret_cast<int*>(base + Y.blk + 8) : nullptr;
    C.wln = NW > 1 ? reinterpret_cast<int*>(base + Y.blk + 12) : nullptr;
    C.wlnext = NW > 1 ? reinterpret_cast<int*>(base + Y.blk + 16) : nullptr;
    C.e2go = NW > 1 ? reinterpret_cast<int*>(base + Y.blk + 20) : nullptr;
    C.e2n2 = NW > 1 ? reinterpret_cast<int*>(base + Y.blk + 24) : nullptr;
    C.kcnt = NW > 1 ? reinterpret_cast<int*>(base + Y.blk + 28) : nullptr;
    C.gln = NW > 1 ? reinterpret_cast<int*>(base + Y.blk + 32) : nullptr;
    C.glnext = NW > 1 ? reinterpret_cast<int*>(base + Y.blk + 36) : nullptr;
    C.rsel = IM >= 128 ? reinterpret_cast<uint2*>(base + Y.rsel) + 64 * (threadIdx.x >> 6) : nullptr;
    C.I = P.I; C.S = P.S; C.W = P.W; C.RB = P.RB;
    C.shift = P.blk_shift;
    C.bmask = (1u << P.blk_shift) - 1u;
    C.M = P.M;
    C.wmask = P.wsz - 1u;
    C.wcap = P.wcap;
    return C;
}

using namespace wave;

// Wave reductions and scans through DPP lane moves and lane reads (no LDS
// round trip): four row steps leave every lane of a 16-lane row with the
// row's reduction (quad_perm 1,0,3,2; quad_perm 2,3,0,1; row_half_mirror;
// row_mirror), the four rows are combined from lanes 0, 16, 32, 48.
template <int kCtrl>
__device__ __forceinline__ int dpp_row(int x)
{
    return __builtin_amdgcn_mov_dpp(x, kCtrl, 0xF, 0xF, false);
}
template <int kCtrl>
__device__ __forceinline__ unsigned long long dpp_row64(unsigned long long x)
{
    const unsigned lo = unsigned(dpp_row<kCtrl>(int(unsigned(x))));
    const unsigned hi = unsigned(dpp_row<kCtrl>(int(unsigned(x >> 32))));
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}
__device__ __forceinline__ int wsum(int x)
{
    x += dpp_row<0xB1>(x);
    x += dpp_row<0x4E>(x);
    x += dpp_row<0x141>(x);
    x += dpp_row<0x140>(x);
    return rl(x, 0) + rl(x, 16) + rl(x, 32) + rl(x, 48);
}
__device__ __forceinline__ unsigned long long wsum64(unsigned long long x)
{
    x += dpp_row64<0xB1>(x);
    x += dpp_row64<0x4E>(x);
    x += dpp_row64<0x141>(x);
    x += dpp_row64<0x140>(x);
    return rl64(x, 0) + rl64(x, 16) + rl64(x, 32) + rl64(x, 48);
}
template <typename T>
__device__ __forceinline__ T tmax(T a, T b) { return a > b ? a : b; }
template <typename T>
__device__ __forceinline__ T tmin(T a, T b) { return a < b ? a : b; }
__device__ __forceinline__ unsigned long long wmax64(unsigned long long x)
{
    x = tmax(x, dpp_row64<0xB1>(x));
    x = tmax(x, dpp_row64<0x4E>(x));
    x = tmax(x, dpp_row64<0x141>(x));
    x = tmax(x, dpp_row64<0x140>(x));
    return tmax(tmax(rl64(x, 0), rl64(x, 16)), tmax(rl64(x, 32), rl64(x, 48)));
}
__device__ __forceinline__ unsigned long long wmin64(unsigned long long x)
{
    x = tmin(x, dpp_row64<0xB1>(x));
    x = tmin(x, dpp_row64<0x4E>(x));
    x = tmin(x, dpp_row64<0x141>(x));
    x = tmin(x, dpp_row64<0x140>(x));
    return tmin(tmin(rl64(x, 0), rl64(x, 16)), tmin(rl64(x, 32), rl64(x, 48)));
}
__device__ __forceinline__ uint32_t wmin32(uint32_t x)
{
    x = tmin(x, uint32_t(dpp_row<0xB1>(int(x))));
    x = tmin(x, uint32_t(dpp_row<0x4E>(int(x))));
    x = tmin(x, uint32_t(dpp_row<0x141>(int(x))));
    x = tmin(x, uint32_t(dpp_row<0x140>(int(x))));
    return tmin(tmin(rlu(x, 0), rlu(x, 16)), tmin(rlu(x, 32), rlu(x, 48)));
}
__device__ __forceinline__ uint32_t wmax32(uint32_t x)
{
    x = tmax(x, uint32_t(dpp_row<0xB1>(int(x))));
    x = tmax(x, uint32_t(dpp_row<0x4E>(int(x))));
    x = tmax(x, uint32_t(dpp_row<0x141>(int(x))));
    x = tmax(x, uint32_t(dpp_row<0x140>(int(x))));
    return tmax(tmax(rlu(x, 0), rlu(x, 16)), tmax(rlu(x, 32), rlu(x, 48)));
}

// wave-wide max of a double through DPP lane moves; every lane gets the result
template <int kCtrl, int kRowMask>
__device__ __forceinline__ double dpp_f64(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const int lo2 = __builtin_amdgcn_update_dpp(lo, lo, kCtrl, kRowMask, 0xF, false);
    const int hi2 = __builtin_amdgcn_update_dpp(hi, hi, kCtrl, kRowMask, 0xF, false);
    return __hiloint2double(hi2, lo2);
}
// a lane move in which every lane reads a lane of its own row (no old value)
template <int kCtrl>
__device__ __forceinline__ double dpp_row_f64(double v)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), kCtrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), kCtrl, 0xF, 0xF, false);
    return __hiloint2double(hi, lo);
}
// Maximum over the first NL lanes (NL = 16, 32 or 64) for every lane; the
// other lanes must not exceed it.  (The file is compiled without NaN
// support: no operand needs quieting before v_max_f64.)
template <int NL>
__device__ __forceinline__ double wave_max_f64(double v)
{
    v = fmax(v, dpp_row_f64<0xB1>(v));    // quad_perm 1,0,3,2
    v = fmax(v, dpp_row_f64<0x4E>(v));    // quad_perm 2,3,0,1
    v = fmax(v, dpp_row_f64<0x141>(v));   // row_half_mirror
    v = fmax(v, dpp_row_f64<0x140>(v));   // row_mirror: every lane of a row holds its maximum
    if (NL > 16) v = fmax(v, dpp_f64<0x142, 0xA>(v));  // row_bcast:15
    if (NL > 32) v = fmax(v, dpp_f64<0x143, 0xC>(v));  // row_bcast:31
    const int lo = __builtin_amdgcn_readlane(__double2loint(v), NL - 1);
    const int hi = __builtin_amdgcn_readlane(__double2hiint(v), NL - 1);
    return __hiloint2double(hi, lo);
}

// Sum over the first NL lanes (NL = 16, 32 or 64) of doubles whose sums are
// exact, for every lane; the other lanes hold 0.
template <int NL>
__device__ __forceinline__ double wsum_f64(double x)
{
    x += dpp_row_f64<0xB1>(x);
    x += dpp_row_f64<0x4E>(x);
    x += dpp_row_f64<0x141>(x);
    x += dpp_row_f64<0x140>(x);
    auto row = [&](int l) {
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), l), __builtin_amdgcn_readlane(__double2loint(x), l));
    };
    double r = row(0);
    if (NL > 16) r += row(16);
    if (NL > 32) r += row(32) + row(48);
    return r;
}

__device__ __forceinline__ int blocks_of(uint32_t len, uint32_t shift)
{
    return int((len + (1u << shift) - 1u) >> shift);
}

// full finish tick of a running word, given that it has not finished before t
__device__ __forceinline__ uint32_t fin_of(uint32_t v, uint32_t t) { return t + ((wmid(v) - t) & kFin); }

// Headroom of the tiers in mask tm (Eq. 4), 1/256 block: two reads of the
// replica's table of sums instead of a term per tier, whose ten values would
// stay in registers through the tick loop.
__device__ __forceinline__ int headroom_sum(const Ctx& C, int tm) { return C.ht[tm & 31] + C.ht[32 + (tm >> 5)]; }
// The table of headroom values hq[0..9], by one wave.
__device__ inline void headroom_table(const Ctx& C, const int32_t* hq, int lane)
{
    int v = 0;
#pragma unroll
    for (int p = 0; p < 5; ++p) v += (lane >> p) & 1 ? (lane < 32 ? hq[p] : hq[5 + p]) : 0;
    C.ht[lane] = v;
}

// a / den for an integer a (exact in a double) and a divisor den whose
// correctly rounded reciprocal is rd: the correctly rounded quotient
// (Markstein 1990: with r = RN(1/den), q = RN(a r) and the exact remainder
// a - q den, RN(q + remainder r) is RN(a/den)), in three operations where
// the full division takes eleven.
__device__ __forceinline__ double quot(double a, double den, double rd)
{
    const double q = a * rd;
    return __builtin_fma(__builtin_fma(-q, den, a), rd, q);
}

// Freeness of instance i (Eq. 1-4): num = 256 (free - hol demand) - sum of H_p
// over the tiers with a running request, over max(B, 1).
__device__ inline void set_f(const Ctx& C, int i)
{
    const int tm = C.tmask[i], b = C.B[i], fr = C.freeb[i], hd = C.hold[i];
    const int num = 256 * (fr - hd) - headroom_sum(C, tm);
    C.num[i] = num;
    C.fd[i] = double(num) / double(b > 0 ? b : 1);
}

// running requests of instance i whose length is r mod block_tokens: laid out
// residue-major, so that the lanes of one residue read consecutive counters
__device__ __forceinline__ uint32_t res_idx(const Ctx& C, int i, uint32_t r) { return r * C.I + uint32_t(i); }

// Counters of running requests, two u16 per LDS word (an instance holds at
// most 2048 running requests, so no half ever carries into the other).  All
// updates are atomic: lanes that work on different instances may share a word.
__device__ __forceinline__ uint32_t c16_get(const unsigned* a, uint32_t idx)
{
    return (a[idx >> 1] >> ((idx & 1u) * 16u)) & 0xFFFFu;
}
__device__ __forceinline__ uint32_t c16_inc(unsigned* a, uint32_t idx)
{
    const uint32_t sh = (idx & 1u) * 16u;
    return (atomicAdd(&a[idx >> 1], 1u << sh) >> sh) & 0xFFFFu;
}
__device__ __forceinline__ uint32_t c16_dec(unsigned* a, uint32_t idx)
{
    const uint32_t sh = (idx & 1u) * 16u;
    return (atomicSub(&a[idx >> 1], 1u << sh) >> sh) & 0xFFFFu;
}

__device__ __forceinline__ void tier_dec(const Ctx& C, int i, int tier)
{
    if (c16_dec(C.tcnt, uint32_t(i * kTiers + tier)) == 1u) atomicAnd(&C.tmask[i], ~(1 << tier));
}
__device__ __forceinline__ void tier_inc(const Ctx& C, int i, int tier)
{
    c16_inc(C.tcnt, uint32_t(i * kTiers + tier));
    atomicOr(&C.tmask[i], 1 << tier);
}

__device__ __forceinline__ void stat(const Ctx& C, int idx, unsigned long long v) { atomicAdd(&C.stats[idx], v); }

// Latency histograms in ticks: a value below 16 has its own bin; a larger
// value v with 2^e <= v < 2^(e+1) falls into one of eight sub-ranges of
// width 2^(e-3), bin 16 + 8 (e - 4) + (v >> (e - 3)) - 8.
__device__ __forceinline__ uint32_t hist_bin(uint32_t v)
{
    if (v < 16u) return v;
    const uint32_t e = 31u - uint32_t(__builtin_clz(v));
    return 8u * e - 24u + (v >> (e - 3u));
}
__device__ __forceinline__ void hist_add(const Ctx& C, int metric, int tier, uint32_t v)
{
    atomicAdd(&C.hist[(metric * kTiers + tier) * MTS_HIST_BINS + hist_bin(v)], 1u);
}

// INFaaS cost of instance i in 1/256 tick with extra queued requests:
// alpha q + beta s + gamma penalty, q = waiting + extra.  Below 2^51 by the
// configuration limits, so exact as a double.
__device__ __forceinline__ double infaas_cost(const Ctx& C, const Params& P, int i, int extra)
{
    const long long c = P.alpha256 * (C.nwait[i] + extra) + P.beta * C.svc[i] + P.gamma256 * C.pen[i];
    return double(c);
}

// number of 64-slot chunks of instance i up to its highest non-empty one; uniform
__device__ __forceinline__ int live_chunks(const Ctx& C, int i, int lane)
{
    const unsigned long long w = lane < int(C.W) ? C.occ[i * C.W + lane] : 0ull;
    const unsigned long long nz = ballot(w != 0);
    return nz ? 64 - __clzll(static_cast<long long>(nz)) : 0;
}

// position of the k-th (from 0) set bit of m; m has more than k set bits.  The
// half is chosen first, so that the rest works on one 32-bit register.
__device__ __forceinline__ int kth_set_bit(unsigned long long m, int k)
{
    const uint32_t lo = uint32_t(m);
    const int cl = __popc(lo);
    const bool up = k >= cl;
    uint32_t x = up ? uint32_t(m >> 32) : lo;
    int pos = up ? 32 : 0;
    k -= up ? cl : 0;
#pragma unroll
    for (int w = 16; w >= 1; w >>= 1) {
        const uint32_t part = x & ((1u << w) - 1u);
        const int c = __popc(part);
        const bool skip = k >= c;
        x = skip ? x >> w : part;
        k -= skip ? c : 0;
        pos += skip ? w : 0;
    }
    return pos;
}

// inclusive prefix sum over the lanes of the wave, by DPP: row_shr 1, 2, 4,
// 8 (lanes reading before their row's start get 0) scan each row, then
// row_bcast:15 adds row 0's total into row 1 and row 2's into row 3, and
// row_bcast:31 adds the total of rows 0-1 into rows 2 and 3
__device__ __forceinline__ int wscan(int x, int lane)
{
    (void)lane;
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);
    return x;
}

// ---------------------------------------------------------------------------
// per-instance event handlers (uniform: the whole wave works on instance i)
// ---------------------------------------------------------------------------

__device__ __forceinline__ void qx_clear(const Ctx& C, int i)
{
    if (C.xn) C.xn[i] = 0;
}
__device__ __forceinline__ int qx_count(const Ctx& C, int i) { return C.xn ? (C.xn[i] & 0xFFFF) : 0; }
// entry k of instance i's extension whose first entry is at xh (k <= xd)
__device__ __forceinline__ uint4* qx_at(const Ctx& C, int i, int xh, int k)
{
    const int x = xh + k;
    return C.qx + size_t(i) * C.xd + (x >= C.xd ? x - C.xd : x);
}


__device__ __forceinline__ void clear_hol(const Ctx& C, int i)
{
    C.hols[i] = kNoHol; C.holk[i] = kNone; C.hold[i] = 0;
    if (C.td) C.qn[i] = 0;
    qx_clear(C, i);
}

__device__ __forceinline__ void set_hol(const Ctx& C, int i, int slot, unsigned long long key, uint32_t word,
                                        uint32_t meta, uint32_t tarr)
{
    C.hols[i] = slot; C.holk[i] = key; C.hold[i] = blocks_of(wlo(word), C.shift);
    C.hwd[i] = word; C.hmt[i] = meta; C.hta[i] = tarr;
}

// Queue cache.  Invariant: the head of line, the qn[i] cached entries and
// (kernels for more than 64 instances) the extension's entries are the smallest
// (tier, seq) keys among instance i's waiting requests, in order.  The functions below are per lane (lane-private
// instance i) and keep it: popping the head promotes the first cached entry
// (or leaves the head unknown, to be found by a rescan), a new waiting
// request becomes the head or enters the cache at its place when it is
// smaller than the last cached entry (or follows it, when every waiting
// request is listed).  Arrivals enter it too (qc_arrive and the dispatch's
// run): dropping the cache of every instance that takes an ordinary arrival
// cost the overloaded gauss10 workload 1.57 rescans per tick where 0.22
// remain, 24.6 ms per 1000 ticks against 18.9 (4096 replicas).
// the rank a tier gives in every ordering (queue, preemption, migration
// candidate): the tier itself, or 0 for all when scheduling is tier-blind
__device__ __forceinline__ unsigned long long rank_of(const Ctx& C, uint32_t tier)
{
    return C.blind ? 0ull : static_cast<unsigned long long>(tier);
}

__device__ __forceinline__ uint4 qc_pack(unsigned long long key, int slot, uint32_t word, uint32_t meta, uint32_t tarr)
{
    return make_uint4(uint32_t(key), word, tarr,
                      uint32_t(slot) | (((meta >> 2) & 15u) << 12) | (((meta >> 6) & 1u) << 16));
}
__device__ __forceinline__ unsigned long long qc_key(const Ctx& C, uint4 e)
{
    return (rank_of(C, (e.w >> 12) & 15u) << 32) | e.x;
}
__device__ __forceinline__ int qc_at(const Ctx& C, int i, int k)
{
    const int x = C.qh[i] + k;
    return i * C.td + (x >= C.td ? x - C.td : x);
}
// insert e at position p of instance i's cache (the last entry drops out when full)
__device__ inline void qc_insert_at(const Ctx& C, int i, int p, uint4 e)
{
    const int n = C.qn[i];
    if (C.xn && n >= C.td) {
        // the last entry drops out of the ring, to the front of the extension
        // (it is the smallest request behind the ring)
        const int xv = C.xn[i], xc = xv & 0xFFFF, xh = xv >> 16;
        if (xc < C.xd) {
            const int h = xc == 0 ? 0 : xh == 0 ? C.xd - 1 : xh - 1;
            *qx_at(C, i, h, 0) = C.qt[qc_at(C, i, n - 1)];
            C.xn[i] = (h << 16) | (xc + 1);
        } else {
            C.xn[i] = 0;
        }
    }
    if (p == 0) {
        // in front: the ring start moves back (over the last entry when full)
        const int h = C.qh[i];
        C.qh[i] = h == 0 ? C.td - 1 : h - 1;
        C.qt[qc_at(C, i, 0)] = e;
        C.qn[i] = n < C.td ? n + 1 : C.td;
        return;
    }
    const int last = n < C.td ? n : C.td - 1;
    for (int k = last; k > p; --k) C.qt[qc_at(C, i, k)] = C.qt[qc_at(C, i, k - 1)];
    C.qt[qc_at(C, i, p)] = e;
    C.qn[i] = last + 1;
}
// the head of line of i left the queue (admitted or moved)
__device__ inline void hol_pop(const Ctx& C, int i)
{
    if (C.nwait[i] == 0) { clear_hol(C, i); return; }
    const int n = C.td ? C.qn[i] : 0;
    if (n == 0) {
        const int xv = C.xn ? C.xn[i] : 0;
        if ((xv & 0xFFFF) == 0) { C.hols[i] = kHolUnknown; return; }
        // the extension's first entry becomes the head of line
        const int xh = xv >> 16;
        const uint4 e = *qx_at(C, i, xh, 0);
        const uint32_t tier = (e.w >> 12) & 15u;
        set_hol(C, i, int(e.w & 0xFFFu), qc_key(C, e), e.y, kWaiting | (tier << 2) | (((e.w >> 16) & 1u) << 6), e.z);
        // (an empty extension starts at its first entry again)
        C.xn[i] = (xv & 0xFFFF) == 1 ? 0 : ((xh + 1 == C.xd ? 0 : xh + 1) << 16) | ((xv & 0xFFFF) - 1);
        return;
    }
    const uint4 e = C.qt[qc_at(C, i, 0)];
    const uint32_t tier = (e.w >> 12) & 15u;
    set_hol(C, i, int(e.w & 0xFFFu), qc_key(C, e), e.y, kWaiting | (tier << 2) | (((e.w >> 16) & 1u) << 6), e.z);
    const int h = C.qh[i] + 1;
    C.qh[i] = h == C.td ? 0 : h;
    C.qn[i] = n - 1;
}
// what the dispatch knows of an instance's queue cache (kept in order[] while
// its arrivals enter): nothing to do, the head of line and the cache are the
// smallest of the waiting requests, or all of them; with the flags that the
// head of line is one of this batch's arrivals, and that the batch's other
// arrivals follow the cached entries as one run
constexpr int kQcSkip = 0, kQcPart = 1, kQcAll = 2, kQcHead = 4, kQcRun = 8;
__device__ __forceinline__ unsigned long long arr_key(const Ctx& C, int tier, uint32_t seq)
{
    return (rank_of(C, uint32_t(tier)) << 32) | seq;
}
// The arrivals of mask em (one per lane, ascending keys, entries en), all
// larger than instance i's head of line, enter its ring in one merge: lane l
// holds entry l, each arrival finds its place by a ballot and the entries
// behind it move up.  An arrival behind the last entry enters only when the
// head and the ring list every waiting request (all); the first one without a
// place ends the merge, the rest being larger still.  Entries that drop out of
// a full ring go to the front of the extension; it is dropped when an arrival
// that got no place belongs in front of its end (inside: such arrivals).  Uniform.
// (Entering the arrivals one after the other by their own lanes took the
// overloaded study 12-13K cycles a tick.)
__device__ inline void qc_merge(const Ctx& C, int i, unsigned long long em, unsigned long long key, uint4 en, bool all,
                                unsigned long long inside, int lane)
{
    const int n = C.qn[i], h = C.qh[i], xv = C.xn ? C.xn[i] : 0, xc = xv & 0xFFFF;
    uint4 e = make_uint4(0u, 0u, 0u, 0u);
    unsigned long long ke = kNone;
    if (lane < n) {
        const int x = h + lane;
        e = C.qt[i * C.td + (x >= C.td ? x - C.td : x)];
        ke = qc_key(C, e);
    }
    int up = 0, ins = 0, at = -1;
    bool split = false;  // an arrival without a place is smaller than some entry
    unsigned long long m = em;
    for (; m; m &= m - 1) {
        const int l = ffs64(m);
        const unsigned long long kj = rl64(key, l);
        const int p = __popcll(ballot(ke < kj));  // (lanes without an entry hold the largest key)
        if (p + ins >= C.td) { split = p < n; break; }
        if (p == n && !(all && xc == 0)) break;
        up += ke > kj ? 1 : 0;
        at = lane == l ? p + ins : at;
        ++ins;
    }
    const int to = lane + up, total = n + ins;
    if (lane < n && to < C.td) C.qt[i * C.td + to] = e;
    if (at >= 0) C.qt[i * C.td + at] = en;
    if (C.xn) {
        const int o = total > C.td ? total - C.td : 0;
        const bool drop = split || (inside & m) || xc + o > C.xd;
        int xh = (xv >> 16) - o;
        xh += xh < 0 ? C.xd : 0;
        if (!drop && lane < n && to >= C.td) *qx_at(C, i, xh, to - C.td) = e;
        if (lane == 0 && (drop || o > 0)) C.xn[i] = drop ? 0 : (xh << 16) | (xc + o);
    }
    if (lane == 0) {
        C.qn[i] = min(total, C.td);
        C.qh[i] = 0;
    }
    wave_sync();
}
// a new waiting request of i (nwait already counts it); returns true when it
// falls behind the ring of an instance with an extension: the caller's wave
// then puts it in its place there (qx_insert)
__device__ inline bool hol_insert(const Ctx& C, int i, unsigned long long key, int slot, uint32_t word, uint32_t meta,
                                  uint32_t tarr)
{
    const int h = C.hols[i];
    if (h == kHolUnknown) return false;
    if (h == kNoHol) { set_hol(C, i, slot, key, word, meta, tarr); if (C.td) C.qn[i] = 0; qx_clear(C, i); return false; }
    if (key < C.holk[i]) {
        if (C.td) qc_insert_at(C, i, 0, qc_pack(C.holk[i], h, C.hwd[i], C.hmt[i], C.hta[i]));
        set_hol(C, i, slot, key, word, meta, tarr);
        return false;
    }
    if (!C.td) return false;
    const int n = C.qn[i];
    int p = 0;
    while (p < n && qc_key(C, C.qt[qc_at(C, i, p)]) < key) ++p;
    if (p < n) qc_insert_at(C, i, p, qc_pack(key, slot, word, meta, tarr));
    else if (qx_count(C, i) > 0) return true;
    else if (n < C.td && C.nwait[i] == n + 2) {
        // the head and the cache listed every other waiting request: it is the last
        C.qt[qc_at(C, i, n)] = qc_pack(key, slot, word, meta, tarr);
        C.qn[i] = n + 1;
    }
    return false;
}

// Puts waiting request e at its place in the extension of instance i (which
// has one): the entries after it move up by one, read and written from the
// end 256 at a time, so the place in a queue of 2000 costs a few memory round
// trips instead of the rescans that a dropped extension brings (3.2 rescans of
// 2048 slots per tick on the wide workload, 0.65 with it; 23.6 ms per 300
// ticks against 21.5).  When nothing lies behind it, it is the last known
// request only if every other waiting one is listed; else it stays out.
// Uniform.
__device__ inline void qx_insert(const Ctx& C, int i, uint4 e, int lane)
{
    constexpr int GX = 4;
    const int xv = C.xn[i], xc = xv & 0xFFFF, xh = xv >> 16;
    const unsigned long long key = qc_key(C, e);
    if (xc >= C.xd) { wave_sync(); if (lane == 0) C.xn[i] = 0; wave_sync(); return; }
    int p = xc;  // the place of e: everything from p on is larger
    for (int hi = xc; hi > 0; hi -= 64 * GX) {
        uint4 v[GX];
        bool up[GX];
#pragma unroll
        for (int g = 0; g < GX; ++g) {
            const int k = hi - 1 - g * 64 - lane;
            v[g] = k >= 0 ? *qx_at(C, i, xh, k) : make_uint4(0u, 0u, 0u, 0u);
        }
        int moved = 0;
#pragma unroll
        for (int g = 0; g < GX; ++g) {
            const int k = hi - 1 - g * 64 - lane;
            up[g] = k >= 0 && qc_key(C, v[g]) > key;
            moved += __popcll(ballot(up[g]));
        }
#pragma unroll
        for (int g = 0; g < GX; ++g)
            if (up[g]) *qx_at(C, i, xh, hi - g * 64 - lane) = v[g];
        wave_sync();
        p -= moved;
        if (moved < 64 * GX) break;
    }
    const bool all = C.nwait[i] == 2 + C.qn[i] + xc;  // head, ring, extension, e
    wave_sync();
    if (lane == 0 && (p < xc || all)) {
        *qx_at(C, i, xh, p) = e;
        C.xn[i] = (xh << 16) | (xc + 1);
    }
    wave_sync();
}

// File a running request under its finish tick.  In the kernels with a queue
// cache, whose workloads preempt, it returns its place in the bucket (kNoPlace:
// the bucket is full) as the bits 8.. of the slot's meta, so that a request
// that leaves early finds its entry without reading the bucket (overloaded
// study: preemption 51K -> 41K cycles a tick).  The others keep no places:
// moving them with the entries that stay in a bucket cost the sweep 1.5 %,
// and the few requests that leave early there search their bucket.
constexpr uint32_t kNoPlace = 0xFFFu, kPlaceShift = 8;
static_assert(MTS_HIST_BINS > 0 && kMaxSlots < kNoPlace, "a place fits 12 bits");
__device__ __forceinline__ uint32_t wheel_put(const Ctx& C, uint32_t fin, int i, int s)
{
    const uint32_t b = fin & C.wmask;
    const uint32_t sh = (b & 1u) * 16u;
    const uint32_t k = (atomicAdd(&C.wc[b >> 1], 1u << sh) >> sh) & 0xFFFFu;
    if (k < C.wcap) {
        C.wheel[size_t(b) * C.wcap + k] = (uint32_t(i) << 16) | uint32_t(s);
        return C.td ? k << kPlaceShift : 0u;
    } else {
        // full: keep the count at wcap and mark the bucket for an exact rebuild
        atomicSub(&C.wc[b >> 1], 1u << sh);
        atomicOr(&C.wov[b >> 5], 1u << (b & 31u));
        return C.td ? kNoPlace << kPlaceShift : 0u;
    }
}

// A running request that leaves its slot before its finish tick (preempted,
// or moved out by a committed migration) loses its wheel entry: the entry is
// overwritten with a tombstone, so every entry of the wheel names a distinct
// running request.  A bucket that overflowed is rebuilt from the slots at its
// visit and needs nothing here.  Per lane, with a place in the slot's meta m.
constexpr uint32_t kTomb = 0xFFFFFFFFu;
__device__ __forceinline__ void wheel_erase(const Ctx& C, uint32_t fin, uint32_t m)
{
    const uint32_t b = fin & C.wmask, k = m >> kPlaceShift;
    if ((C.wov[b >> 5] >> (b & 31u)) & 1u) return;
    if (k < C.wcap) C.wheel[size_t(b) * C.wcap + k] = kTomb;
}
// The same without places: the whole wave searches the bucket for slot s of i.
__device__ inline void wheel_erase_search(const Ctx& C, uint32_t fin, int i, int s, int lane)
{
    const uint32_t b = fin & C.wmask;
    if ((C.wov[b >> 5] >> (b & 31u)) & 1u) return;
    const uint32_t n = (C.wc[b >> 1] >> ((b & 1u) * 16u)) & 0xFFFFu;
    uint32_t* ent = C.wheel + size_t(b) * C.wcap;
    const uint32_t key = (uint32_t(i) << 16) | uint32_t(s);
    for (uint32_t e0 = 0; e0 < n; e0 += 64) {
        const bool hit = e0 + lane < n && ent[e0 + lane] == key;
        if (hit) ent[e0 + lane] = kTomb;
        if (ballot(hit)) break;
    }
}

// memory pressure: preempt the largest (tier, seq) running request until the
// growth of this tick fits (Section 2.2; recompute semantics)
template <int GR, int MK, bool kArr>
__device__ inline bool preempt(const Ctx& C, int i, uint32_t t, int lane)
{
    const size_t b = size_t(i) * C.S;
    // (MK: a call takes one victim nearly always, since a victim frees tens of
    // blocks and a tick's growth is a few; a second key per lane only spares the
    // second scan of a call with more.  One key instead of two: overloaded study
    // 21.08 -> 20.70 ms, gauss10 14.84 -> 14.56, with extensions 4.39 -> 4.26,
    // INFaaS sweep 6.59 -> 6.44, tiny run 6.45 -> 6.34; wide, whose bursts take
    // more victims a call, 15.20 -> 15.66, keeps two.)
    // (kArr: a victim's arrival tick comes with the scan; 16 chunks a round trip
    // leave it no registers, and without a queue cache its spills cost the
    // INFaaS sweep 4 %)
    int G = C.gtmp[i], fr = C.freeb[i];
    bool aborted = false;
    bool scan = G > fr;
    while (scan) {
        // Each lane keeps the MK largest (tier, seq) keys of its running slots,
        // descending, with the slot, its word and its meta (a running
        // request's word and meta do not change while it runs); GR chunks of
        // 64 slots are read per memory round trip.
        const int nch = live_chunks(C, i, lane);
        unsigned long long k[MK];
        uint32_t kw[MK], km[MK], ka[MK];
        int ks[MK];
#pragma unroll
        for (int x = 0; x < MK; ++x) { k[x] = 0; kw[x] = 0; km[x] = 0; ka[x] = 0; ks[x] = 0; }
        int cnt = 0;
        for (int c0 = 0; c0 < nch; c0 += GR) {
            uint32_t v[GR], m[GR], q[GR], a[GR];
#pragma unroll
            for (int g = 0; g < GR; ++g) {
                const bool in = c0 + g < nch;
                const uint4 rr = in ? C.slot[b + (c0 + g) * 64 + lane] : make_uint4(0u, 0u, 0u, 0u);
                v[g] = rr.x; m[g] = rr.y; q[g] = rr.z; a[g] = kArr ? rr.w : 0u;
            }
#pragma unroll
            for (int g = 0; g < GR; ++g) {
                if (wst(v[g]) != 2u) continue;
                ++cnt;
                unsigned long long ck = ((rank_of(C, (m[g] >> 2) & 15u) + 1ull) << 32) | q[g];
                if (ck <= k[MK - 1]) continue;
                uint32_t cw = v[g], cm = m[g], ca = a[g];
                int cs = (c0 + g) * 64 + lane;
#pragma unroll
                for (int x = 0; x < MK; ++x) {
                    if (ck > k[x]) {
                        const unsigned long long tk = k[x]; k[x] = ck; ck = tk;
                        const uint32_t tw = kw[x]; kw[x] = cw; cw = tw;
                        const uint32_t tm = km[x]; km[x] = cm; cm = tm;
                        const uint32_t ta = ka[x]; ka[x] = ca; ca = ta;
                        const int ts = ks[x]; ks[x] = cs; cs = ts;
                    }
                }
            }
        }
        const bool more = cnt > MK;
        int taken = 0;
        scan = false;
        while (G > fr) {
            const unsigned long long mx = wmax64(k[0]);
            if (mx == 0) break;  // nothing runs
            const int wl = ffs64(ballot(k[0] == mx));
            const int vs = rl(ks[0], wl);
            const uint32_t v = rlu(kw[0], wl), m = rlu(km[0], wl), vta = kArr ? rlu(ka[0], wl) : s_tarr(C, b + vs);
            const bool win = lane == wl;
#pragma unroll
            for (int x = 0; x + 1 < MK; ++x) {
                k[x] = win ? k[x + 1] : k[x];
                kw[x] = win ? kw[x + 1] : kw[x];
                km[x] = win ? km[x + 1] : km[x];
                ka[x] = win ? ka[x + 1] : ka[x];
                ks[x] = win ? ks[x + 1] : ks[x];
            }
            k[MK - 1] = win ? 0ull : k[MK - 1];
            taken += win ? 1 : 0;
            const bool unknown = ballot(win && more && taken >= MK) != 0;
            // the victim returns to the queue (recompute semantics: len, rem and
            // seq kept, its blocks freed)
            const uint32_t lenf = wlo(v), fin = fin_of(v, t);
            const uint32_t remb = fin - t + 1u, lenb = lenf - remb;
            const uint32_t vw = kWaitW | (remb << 16) | lenb;
            const uint32_t vmeta = (m & 0xFFu & ~(3u | kMigrating)) | kWaiting;
            const int vb = blocks_of(lenb, C.shift);
            const int vg = (lenb & C.bmask) == 0;
            const int vt = int((m >> 2) & 15u);
            const int vr = int((lenf - fin - 1u) & C.bmask);
            const bool vm = (m & kMigrating) != 0;
            if (lane == 0) {
                s_set_wm(C, b + vs, vw, vmeta);
                if (C.td) wheel_erase(C, fin, m);
            }
            if (!C.td) wheel_erase_search(C, fin, i, vs, lane);
            fr += vb;
            G -= vg;
            aborted = aborted || vm;
            bool deep = false;
            if (lane == 0) {
                C.held[i] -= vb;
                C.B[i] -= 1;
                C.nwait[i] += 1;
                C.frs[i] = 0;
                if (C.fsum) C.flags[i] |= kFlagIntf;  // (INFaaS state)
                // (several waves may preempt at once; a count above kVic means
                // the list missed some)
                const int nv = atomicAdd(C.nvic, 1);
                if (nv < kVic) C.vic[nv] = (uint32_t(i) << 16) | uint32_t(vs);
                c16_dec(C.res, res_idx(C, i, vr));
                tier_dec(C, i, vt);
                stat(C, vt * 8 + kPreempted, 1);
                if (vm) C.flags[i] |= kFlagAbort;
                const unsigned long long key = (rank_of(C, uint32_t(vt)) << 32) | static_cast<unsigned>(mx);
                deep = hol_insert(C, i, key, vs, vw, vmeta, vta);
                if (C.ext) wlb(C)[i] = vta < wlb(C)[i] ? vta : wlb(C)[i];
            }
            wave_sync();
            if (C.xn && ballot(deep))
                qx_insert(C, i, qc_pack((rank_of(C, uint32_t(vt)) << 32) | static_cast<unsigned>(mx), vs, vw, vmeta, vta), lane);
            if (unknown) { scan = G > fr; break; }  // the winner's next key is unknown: read again
        }
    }
    // this tick's growth, now that it fits
    if (lane == 0) { C.freeb[i] = fr - G; C.held[i] += G; }
    wave_sync();
    return aborted;
}

// Exact finish scan of instance i, used when a wheel bucket overflowed:
// finishes the requests whose last token is at t and files again the running
// requests that share the bucket of t but finish later.
__device__ inline void finish_scan(const Ctx& C, int i, uint32_t t, int lane, bool& abort_any)
{
    const size_t b = size_t(i) * C.S;
    const int nch = live_chunks(C, i, lane);
    const uint32_t bk = t & C.wmask;
    int freed = 0, nf = 0;
    bool ab = false;
    for (int c = 0; c < nch; ++c) {
        const int s = c * 64 + lane;
        const uint4 rec = C.slot[b + s];
        const uint32_t v = rec.x;
        const bool run = wst(v) == 2u;
        const uint32_t fin = fin_of(v, t);
        const bool f = run && fin == t;
        if (f) {
            const uint32_t lenf = wlo(v);
            freed += blocks_of(lenf, C.shift);
            const uint32_t m = rec.y;
            const int tier = int((m >> 2) & 15u);
            stat(C, tier * 8 + kFinished, 1);
            const uint32_t e2e = t - rec.w;
            stat(C, tier * 8 + kE2e, e2e);
            hist_add(C, kHistE2e, tier, e2e);
            if (C.fsum) { atomicAdd(&C.fsum[i], static_cast<unsigned long long>(e2e)); atomicAdd(&C.fcnt[i], 1); }
            c16_dec(C.res, res_idx(C, i, (lenf - t - 1u) & C.bmask));
            tier_dec(C, i, tier);
            // being copied out: the source of its instance's migration record
            // (the same test as the wheel visit's)
            if (C.mig[4 * i] >= 0 && C.mig[4 * i + 1] == s) ab = true;
            s_word(C, b + s) = 0;  // the word alone marks the slot empty
        } else if (run && (fin & C.wmask) == bk) {
            const uint32_t place = wheel_put(C, fin, i, s);
            if (C.td) s_meta(C, b + s) = (rec.y & 0xFFu) | place;
        }
        const unsigned long long fb = ballot(f);
        const unsigned long long ow = ballot(v != 0 && !f);
        nf += __popcll(fb);
        if (lane == 0) C.occ[i * C.W + c] = ow;
    }
    freed = wsum(freed);
    const bool any_ab = ballot(ab) != 0;
    abort_any = abort_any || any_ab;
    if (lane == 0) {
        C.freeb[i] += freed;
        C.held[i] -= freed;
        C.B[i] -= nf;
        C.live[i] -= nf;
        if (any_ab) C.flags[i] |= kFlagAbort;
    }
    wave_sync();
}

// One batch of up to 64 entries of bucket t mod wsz (lanes with inb set),
// each with its slot's word, meta and arrival tick: entries with fin = t
// finish, those with a later fin stay in the bucket (compacted in place from
// position kept on, or from the one that counter gives when several waves
// visit the bucket; returns the new kept count), tombstones and entries whose
// slot changed since are dropped.
__device__ inline uint32_t finish_batch(const Ctx& C, uint32_t t, int lane, uint32_t* ent, uint32_t kept, bool inb,
                                        uint32_t e, uint32_t v, uint32_t m, uint32_t ta, bool& abort_any,
                                        int* counter = nullptr)
{
    const uint32_t bk = t & C.wmask;
    const int i = int(e >> 16), s = int(e & 0xFFFFu);
    const bool valid = inb && uint32_t(i) < C.I && uint32_t(s) < C.S;
    if (!valid) v = 0;
    const int2 mg = *reinterpret_cast<const int2*>(&C.mig[valid ? 4 * i : 0]);
    const uint32_t fin = fin_of(v, t);
    // entries name distinct running requests (wheel_erase)
    const bool f = valid && wst(v) == 2u && fin == t;
    const bool k = valid && wst(v) == 2u && fin != t && (fin & C.wmask) == bk;
    const unsigned long long km = ballot(k);
    if (counter && km) {
        int b = 0;
        if (lane == 0) b = atomicAdd(counter, __popcll(km));
        kept = uint32_t(rl(b, 0));
    }
    if (k) {
        // a later finish that shares the bucket: its entry moves to its new place
        // (m may predate a migration's start: the flag comes from the record)
        const uint32_t at = kept + __popcll(km & lanemask_lt());
        ent[at] = e;
        if (C.td)
            s_meta(C, size_t(i) * C.S + s) = (m & 0x7Fu) | (mg.x >= 0 && mg.y == s ? kMigrating : 0u) | (at << kPlaceShift);
    }
    kept += __popcll(km);
    bool ab = false;
    if (f) {
        const size_t idx = size_t(i) * C.S + s;
        const uint32_t lenf = wlo(v);
        const int bl = blocks_of(lenf, C.shift);
        const int tier = int((m >> 2) & 15u);
        stat(C, tier * 8 + kFinished, 1);
        stat(C, tier * 8 + kE2e, t - ta);
        hist_add(C, kHistE2e, tier, t - ta);
        if (C.fsum) { atomicAdd(&C.fsum[i], static_cast<unsigned long long>(t - ta)); atomicAdd(&C.fcnt[i], 1); }
        c16_dec(C.res, res_idx(C, i, (lenf - t - 1u) & C.bmask));
        tier_dec(C, i, tier);
        // being copied out: the source of its instance's migration record (the
        // slot's meta may predate the migration's start)
        ab = mg.x >= 0 && mg.y == s;
        if (ab) atomicOr(&C.flags[i], kFlagAbort);
        atomicAnd(&C.occ[i * C.W + (s >> 6)], ~(1ull << (s & 63)));
        atomicAdd(&C.freeb[i], bl);
        atomicSub(&C.held[i], bl);
        atomicSub(&C.B[i], 1);
        atomicSub(&C.live[i], 1);
        s_word(C, idx) = 0;  // the word alone marks the slot empty
    }
    abort_any = abort_any || ballot(ab) != 0;
    wave_sync();
    return kept;
}

// A bucket of more than one batch, by all NW waves: batch b of 64 entries is
// wave b mod NW's.  Every entry and its slot is read before any entry moves
// (two memory round trips for the whole bucket where one wave after the other
// batch took two each: 8.6K cycles of the wide workload's tick).  *kcnt is 0
// before; the caller sets the bucket's count to it after a barrier.
template <int NW>
__device__ inline void finish_wide(const Ctx& C, uint32_t t, int lane, int wid, uint32_t n, bool& abort_any)
{
    // kMaxSlots caps the entries of a bucket
    constexpr int NB = int(kMaxSlots) / (64 * NW);
    uint32_t* ent = C.wheel + size_t(t & C.wmask) * C.wcap;
    uint32_t e[NB], v[NB], m[NB], ta[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint32_t k = uint32_t(b * NW + wid) * 64u + uint32_t(lane);
        e[b] = k < n ? ent[k] : kTomb;
    }
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const uint32_t i = e[b] >> 16, s = e[b] & 0xFFFFu;
        const uint4 rec = i < C.I && s < C.S ? C.slot[size_t(i) * C.S + s] : make_uint4(0u, 0u, 0u, 0u);
        v[b] = rec.x; m[b] = rec.y; ta[b] = rec.w;
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (uint32_t(b * NW + wid) * 64u >= n) break;
        finish_batch(C, t, lane, ent, 0, true, e[b], v[b], m[b], ta[b], abort_any, C.kcnt);
    }
}

__device__ __forceinline__ void wheel_set_count(const Ctx& C, uint32_t b, uint32_t n, int lane)
{
    const uint32_t sh = (b & 1u) * 16u;
    if (lane == 0) C.wc[b >> 1] = (C.wc[b >> 1] & ~(0xFFFFu << sh)) | (n << sh);
    wave_sync();
}

// Requests that emit their last token at tick t: the bucket t mod wsz lists
// every running request with fin = t (mod wsz).
__device__ inline void finish_tick(const Ctx& C, uint32_t t, int lane, bool& abort_any)
{
    const uint32_t bk = t & C.wmask;
    const uint32_t sh = (bk & 1u) * 16u;
    const uint32_t n = (C.wc[bk >> 1] >> sh) & 0xFFFFu;
    if ((C.wov[bk >> 5] >> (bk & 31u)) & 1u) {
        // the bucket overflowed: rebuild it by scanning every instance with running requests
        if (lane == 0) {
            C.wc[bk >> 1] &= ~(0xFFFFu << sh);
            C.wov[bk >> 5] &= ~(1u << (bk & 31u));
            stat(C, kWheelRebuilds, 1);
        }
        wave_sync();
        for (uint32_t j = 0; j < (C.I + 63) / 64; ++j) {
            const uint32_t i = lane + 64 * j;
            for (unsigned long long m = ballot(i < C.I && C.B[i] > 0); m; m &= m - 1)
                finish_scan(C, int(64 * j + ffs64(m)), t, lane, abort_any);
        }
        return;
    }
    uint32_t* ent = C.wheel + size_t(bk) * C.wcap;
    uint32_t kept = 0;
    for (uint32_t e0 = 0; e0 < n; e0 += 64) {
        const bool inb = e0 + lane < n;
        const uint32_t e = inb ? ent[e0 + lane] : 0u;
        const int i = int(e >> 16), s = int(e & 0xFFFFu);
        const bool valid = inb && uint32_t(i) < C.I && uint32_t(s) < C.S;
        const size_t idx = size_t(i) * C.S + s;
        uint32_t v = 0, m = 0, ta = 0;
        if (valid) { const uint4 rec = C.slot[idx]; v = rec.x; m = rec.y; ta = rec.w; }
        kept = finish_batch(C, t, lane, ent, kept, inb, e, v, m, ta, abort_any);
    }
    wheel_set_count(C, bk, kept, lane);
}

// Admits the longest prefix of w ranked waiting requests of instance i (lane
// r holds the request of rank r: key, slot word, meta, arrival tick, slot)
// whose summed demand fits the free blocks, and makes the next one the head
// of line (Section 3.1: the local queue is served in priority order while
// the head fits; the result equals admitting the head of line one request at
// a time).  The list holds every waiting request of i (complete) or the w
// smallest keys of a longer queue; when all w of those fit, the head of line
// is unknown afterwards (the next rescan finds it).
// xn0 >= 0: the list is the head of line, the xn0 cached entries and the
// extension (xc0 entries from xh0 on) as far as it fits the wave
// (admit_cached): the new extension is then a suffix of the stored one (the
// cache never holds more than qdepth), so only its head moves; when the whole
// list is admitted, its first entry becomes the head of line (go_on: the
// caller admits from there on, the head of line stays unknown).
__device__ inline void admit_ranked(const Ctx& C, int i, uint32_t t, int lane, int w, unsigned long long key,
                                    uint32_t word, uint32_t meta, uint32_t ta, int slot, bool complete = true,
                                    int xn0 = -1, int xh0 = 0, int xc0 = 0, bool go_on = false)
{
    const size_t b = size_t(i) * C.S;
    const int dem = lane < w ? blocks_of(wlo(word), C.shift) : 0;
    const int pre = wscan(dem, lane);
    const int fr = C.freeb[i];
    const bool adm = lane < w && pre <= fr && uint32_t(slot) < C.S;
    const int na = __popcll(ballot(adm));
    if (adm) {
        const uint32_t len = wlo(word), rem = wmid(word);
        const uint32_t fin = t + rem;
        const size_t hb = b + slot;
        const uint32_t place = wheel_put(C, fin, i, slot);
        s_set_wm(C, hb, kRunW | ((fin & kFin) << 16) | (len + rem), (meta & 0xFCu) | kRunning | kAdmitted | place);
        const int tier = int((meta >> 2) & 15u);
        if (!(meta & kAdmitted)) {
            stat(C, tier * 8 + kAdmittedCnt, 1);
            stat(C, tier * 8 + kQdelay, t - ta);
            hist_add(C, kHistQdelay, tier, t - ta);
        }
        c16_inc(C.res, res_idx(C, i, (len - t - 1u) & C.bmask));
        tier_inc(C, i, tier);
    }
    const int used = na > 0 ? rl(pre, na - 1) : 0;
    const int hs = rl(slot, na < w ? na : 0);
    const unsigned long long hk = rl64(key, na < w ? na : 0);
    const uint32_t hw = rlu(word, na < w ? na : 0), hm = rlu(meta, na < w ? na : 0),
                   ht = rlu(ta, na < w ? na : 0);
    if (lane == 0) {
        C.freeb[i] -= used;
        C.held[i] += used;
        C.B[i] += na;
        C.nwait[i] -= na;
        if (complete ? w != C.nwait[i] + na : w >= C.nwait[i] + na) stat(C, kInvariant, 1);
        if (na < w) {
            set_hol(C, i, hs, hk, hw, hm, ht);
        } else if (complete) {
            clear_hol(C, i);
        } else {
            C.hols[i] = kHolUnknown;
            if (C.td) C.qn[i] = 0;
        }
        if (C.td && na < w) { C.qn[i] = min(w - na - 1, C.td); C.qh[i] = 0; }
        if (C.xn) {
            if (xn0 < 0) {
                C.xn[i] = C.td && na < w && w - na - 1 > C.td ? w - na - 1 - C.td : 0;
            } else {
                // entries before the new extension: the admitted ones and the new ring's
                // (behind the new head of line, or, when all were admitted, none)
                const int used = na + (na < w ? min(w - na - 1, C.td) : -1) - xn0;
                const int xc = xc0 - used;
                const int xh = xh0 + used;
                C.xn[i] = xc > 0 ? ((xh >= C.xd ? xh - C.xd : xh) << 16) | xc : 0;
                if (na == w && xc > 0 && !go_on) hol_pop(C, i);
            }
        }
    }
    // the ranked list holds the smallest keys: the ones after the new head fill
    // the cache, and the ones after those its extension
    if (C.td && lane > na && lane < w && lane - na - 1 < C.td)
        C.qt[i * C.td + lane - na - 1] = qc_pack(key, slot, word, meta, ta);
    if (C.xn && C.td && xn0 < 0 && lane > na + C.td && lane < w)
        *qx_at(C, i, 0, lane - na - 1 - C.td) = qc_pack(key, slot, word, meta, ta);
    wave_sync();
}

// The ranked prefix of a rescan, taken minimum by minimum from the lanes'
// ascending lists k (MK each, with slot | demand << 12 in sd): lane r
// receives the key and sd of rank r.  The extraction stops when nothing is
// left, after 64 requests, qdepth requests after the first one whose summed
// demand exceeds the free blocks fr (the new head of line and the cache
// behind it), or when the winning lane had more waiting slots than it kept
// (more: its next key is unknown).  Returns the number taken.  KT is the key
// type: the 64-bit keys or an order-preserving 32-bit form of them, with
// all-ones as "none".
__device__ __forceinline__ uint32_t wmin_k(uint32_t x) { return wmin32(x); }
__device__ __forceinline__ unsigned long long wmin_k(unsigned long long x) { return wmin64(x); }

template <typename KT, int MK>
__device__ inline int rank_extract(KT (&k)[MK], uint32_t (&sd)[MK], bool more, int fr, int td, int lane, KT& myk,
                                   uint32_t& mysd)
{
    const KT none = static_cast<KT>(~static_cast<KT>(0));
    myk = none;
    mysd = 0;
    int got = 0, taken = 0, cum = 0, lim = 64;
    for (int r = 0; r < lim; ++r) {
        const KT mn = wmin_k(k[0]);
        if (mn == none) break;
        const int wl = ffs64(ballot(k[0] == mn));
        const uint32_t wsd = rlu(sd[0], wl);
        myk = lane == r ? mn : myk;
        mysd = lane == r ? wsd : mysd;
        got = r + 1;
        cum += int(wsd >> 12);
        if (cum > fr && lim == 64) lim = min(64, r + 1 + td);
        const bool win = lane == wl;
#pragma unroll
        for (int x = 0; x + 1 < MK; ++x) {
            k[x] = win ? k[x + 1] : k[x];
            sd[x] = win ? sd[x + 1] : sd[x];
        }
        k[MK - 1] = win ? none : k[MK - 1];
        taken += win ? 1 : 0;
        if (ballot(win && more && taken >= MK)) break;  // the winner's next key is unknown
    }
    return got;
}

// The same ranked prefix as rank_extract on 32-bit keys, found by selection
// instead of minimum by minimum: the candidates the extraction can reach are
// the keys up to the smallest last kept key of a lane with more waiting slots
// (bnd, from the caller; all keys when no lane has more).  Of those, the 64
// smallest are the keys up to a threshold found by bisection over key values
// (the keys are distinct, counted by ballots); they are gathered into this
// wave's buffer, taken out of the lists (set to none), ranked by counting and
// sent to the lane of their rank, and the prefix stops qdepth requests after
// the first one whose summed demand exceeds fr.  The latency chain is a few
// dozen scalar steps instead of one wave reduction per request.
template <int MK>
__device__ inline int rank_select(const Ctx& C, uint32_t (&k)[MK], uint32_t (&sd)[MK], uint32_t bnd, int fr, int lane,
                                  uint32_t& myk, uint32_t& mysd)
{
    constexpr uint32_t none = 0xFFFFFFFFu;
    bool vx[MK];
    int nvalid = 0;
#pragma unroll
    for (int x = 0; x < MK; ++x) {
        vx[x] = k[x] != none && k[x] <= bnd;
        nvalid += __popcll(ballot(vx[x]));
    }
    myk = none;
    mysd = 0;
    const int want = min(64, nvalid);
    if (want == 0) return 0;
    uint32_t thr = none;
    if (nvalid > 64) {
        // the smallest value with 64 candidates at or below it (a lane's
        // candidates need not start at k[0]: taken keys are none)
        uint32_t lo = none, hi = 0;
#pragma unroll
        for (int x = 0; x < MK; ++x) {
            lo = vx[x] ? tmin(lo, k[x]) : lo;
            hi = vx[x] ? tmax(hi, k[x]) : hi;
        }
        lo = wmin32(lo);
        hi = wmax32(hi);
        while (lo < hi) {
            const uint32_t mid = lo + ((hi - lo) >> 1);
            int c = 0;
#pragma unroll
            for (int x = 0; x < MK; ++x) c += __popcll(ballot(vx[x] && k[x] <= mid));
            if (c >= 64) hi = mid;
            else lo = mid + 1;
        }
        thr = lo;
    }
    // gather the want selected candidates (and take them out of the lists)
    int base = 0;
#pragma unroll
    for (int x = 0; x < MK; ++x) {
        const bool sel = vx[x] && k[x] <= thr;
        const unsigned long long m = ballot(sel);
        const int at = base + __popcll(m & lanemask_lt());  // < want <= 64
        if (sel && at < 64) C.rsel[at] = make_uint2(k[x], sd[x]);
        if (sel) k[x] = none;
        base += __popcll(m);
    }
    wave_sync();
    uint32_t ck = none, cs = 0;
    if (lane < want) { const uint2 e = C.rsel[lane]; ck = e.x; cs = e.y; }
    wave_sync();
    // (four independent counts, so that the lane reads overlap)
    int rank = 0, r1 = 0, r2 = 0, r3 = 0, j = 0;
    for (; j + 4 <= want; j += 4) {
        rank += int(rlu(ck, j) < ck);
        r1 += int(rlu(ck, j + 1) < ck);
        r2 += int(rlu(ck, j + 2) < ck);
        r3 += int(rlu(ck, j + 3) < ck);
    }
    for (; j < want; ++j) rank += int(rlu(ck, j) < ck);
    rank += r1 + r2 + r3;
    if (lane >= want) rank = lane;
    const uint32_t sk = uint32_t(__builtin_amdgcn_ds_permute(rank * 4, int(ck)));
    const uint32_t ss = uint32_t(__builtin_amdgcn_ds_permute(rank * 4, int(cs)));
    const int cum = wscan(lane < want ? int(ss >> 12) : 0, lane);
    const unsigned long long over = ballot(lane < want && cum > fr);
    // (with the extension every selected request is kept: the head of line,
    // the cache and the extension take them)
    const int got = over && !C.xn ? min(want, ffs64(over) + 1 + C.td) : want;
    if (lane < got) { myk = sk; mysd = ss; }
    return got;
}

// Head of line of instance i from its slots, with admission (Section 3.1:
// the local queue is served in (tier, seq) order while the head fits).  Each
// lane keeps the MK smallest keys of its slots, with their demand; the wave
// then takes minima round by round, lane r receiving the request of rank r,
// and stops when the winning lane had more waiting slots than it kept (its
// next key is unknown), after 64 requests, or qdepth requests after the first
// one whose cumulative demand exceeds the free blocks (the new head of line
// and the cache behind it).  A second read fetches the fields of the requests
// taken, and the longest fitting prefix is admitted at once (admit_ranked).
// The minima are taken on 32-bit keys when the candidates' seqs allow
// (rank_extract); with SEL (the kernels for more than 64 instances) the same prefix
// is found by selection (rank_select), and when every request taken fits the
// candidates left up to the exhaustion bound are taken next without reading
// the slots again.  GR chunks of 64 slots are read per memory round trip.
// Returns true when every request taken was admitted and more wait (the head
// of line is still unknown).  Uniform.
template <int GR, int MK, bool SEL = false>
__device__ inline bool rescan_admit(const Ctx& C, int i, uint32_t t, int lane)
{
    const size_t b = size_t(i) * C.S;
    const int nch = live_chunks(C, i, lane);
    // per lane: its MK smallest keys, ascending, each with slot | demand << 12
    // (slot < 4096, demand < 2^16 blocks)
    unsigned long long k[MK];
    uint32_t sd[MK];
#pragma unroll
    for (int x = 0; x < MK; ++x) { k[x] = kNone; sd[x] = 0; }
    int cnt = 0;
    for (int c0 = 0; c0 < nch; c0 += GR) {
        uint32_t v[GR], m[GR], q[GR];
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            const bool in = c0 + g < nch;
            const uint4 rr = in ? C.slot[b + (c0 + g) * 64 + lane] : make_uint4(0u, 0u, 0u, 0u);
            v[g] = rr.x; m[g] = rr.y; q[g] = rr.z;
        }
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            if (wst(v[g]) != 1u) continue;
            ++cnt;
            unsigned long long ck = (rank_of(C, (m[g] >> 2) & 15u) << 32) | q[g];
            if (ck >= k[MK - 1]) continue;
            uint32_t cs = uint32_t((c0 + g) * 64 + lane) | (uint32_t(blocks_of(wlo(v[g]), C.shift)) << 12);
            // insertion into the lane's sorted list (the largest drops out)
#pragma unroll
            for (int x = 0; x < MK; ++x) {
                if (ck < k[x]) {
                    const unsigned long long tk = k[x]; k[x] = ck; ck = tk;
                    const uint32_t ts = sd[x]; sd[x] = cs; cs = ts;
                }
            }
        }
    }
    // rank extraction on 32-bit keys rank << 27 | (seq - lowest seq) when the
    // candidates' seqs span less than 2^27 (the order is the same; a 32-bit
    // wave minimum is a third of the 64-bit one), else on the keys themselves
    const int fr = C.freeb[i];
    const bool more = cnt > MK;
    uint32_t slo = 0xFFFFFFFFu, shi = 0;
#pragma unroll
    for (int x = 0; x < MK; ++x) {
        if (k[x] != kNone) { slo = tmin(slo, uint32_t(k[x])); shi = tmax(shi, uint32_t(k[x])); }
    }
    slo = wmin32(slo);
    shi = wmax32(shi);
    const bool c32 = shi - slo < (1u << 27) || slo > shi;
    uint32_t k32[MK];
#pragma unroll
    for (int x = 0; x < MK; ++x)
        k32[x] = k[x] == kNone ? 0xFFFFFFFFu : (uint32_t(k[x] >> 32) << 27) | (uint32_t(k[x]) - slo);
    const uint32_t bnd = SEL && c32 ? wmin32(more ? k32[MK - 1] : 0xFFFFFFFFu) : 0u;
    for (;;) {
        unsigned long long myk;
        uint32_t mysd;
        int got;
        if (c32) {
            uint32_t my32;
            if (SEL) got = rank_select<MK>(C, k32, sd, bnd, C.freeb[i], lane, my32, mysd);
            else got = rank_extract<uint32_t, MK>(k32, sd, more, fr, C.td, lane, my32, mysd);
            myk = my32 == 0xFFFFFFFFu
                      ? kNone
                      : (static_cast<unsigned long long>(my32 >> 27) << 32) | ((my32 & 0x7FFFFFFu) + slo);
        } else {
            got = rank_extract<unsigned long long, MK>(k, sd, more, fr, C.td, lane, myk, mysd);
        }
        if (got == 0) {
            if (lane == 0) clear_hol(C, i);
            wave_sync();
            return false;
        }
        const int mys = int(mysd & 0xFFFu);
        uint32_t w = 0, mt = 0, ta = 0;
        if (lane < got) { const uint4 rec = C.slot[b + mys]; w = rec.x; mt = rec.y; ta = rec.w; }
        const bool complete = got >= C.nwait[i];
        if (lane == 0) C.frs[i] = 0;
        admit_ranked(C, i, t, lane, got, myk, w, mt, ta, mys, complete);
        // (selection) every request taken was admitted and more wait: the
        // candidates left up to bnd are the next smallest keys of the queue,
        // and are taken without reading the slots again
        if (!(SEL && c32) || C.hols[i] != kHolUnknown) break;
        bool left = false;
#pragma unroll
        for (int x = 0; x < MK; ++x) left = left || (k32[x] != 0xFFFFFFFFu && k32[x] <= bnd);
        if (!ballot(left)) break;
    }
    return C.hols[i] == kHolUnknown;
}

// Admission of instance i when its head of line fits and 2..64 requests wait
// (Section 3.1: the local queue is served in priority order while the head
// fits).  The waiting requests are gathered into lanes, ranked by (tier, seq),
// and the longest prefix of the ranked list whose summed demand fits is
// admitted in one step; the next ranked request becomes the head of line.
// The result equals admitting the head of line one request at a time.  GR
// chunks of 64 slots are read per memory round trip.
template <int GR>
__device__ inline void admit_batch(const Ctx& C, int i, uint32_t t, int lane)
{
    const size_t b = size_t(i) * C.S;
    const int nch = live_chunks(C, i, lane);
    unsigned long long key = kNone;
    uint32_t word = 0, meta = 0, ta = 0;
    int slot = 0, w = 0;
    for (int c0 = 0; c0 < nch; c0 += GR) {
        uint32_t v[GR], m[GR], q[GR], a[GR];
        // all loads of the group are issued together (one memory round trip)
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            const bool in = c0 + g < nch;
            const size_t sb = b + (c0 + g) * 64 + lane;
            const uint4 rr = in ? C.slot[sb] : make_uint4(0u, 0u, 0u, 0u);
            v[g] = rr.x; m[g] = rr.y; q[g] = rr.z; a[g] = rr.w;
        }
#pragma unroll
        for (int g = 0; g < GR; ++g) {
            const unsigned long long wm = ballot(wst(v[g]) == 1u);
            if (!wm) continue;
            const int cnt = __popcll(wm);
            const int k = lane - w;
            const bool take = k >= 0 && k < cnt;
            const int src = kth_set_bit(wm, take ? k : 0);
            const uint32_t pv = __shfl(v[g], src), pm = __shfl(m[g], src), pq = __shfl(q[g], src),
                           pa = __shfl(a[g], src);
            if (take) {
                word = pv; meta = pm; ta = pa;
                key = (rank_of(C, (pm >> 2) & 15u) << 32) | pq;
                slot = (c0 + g) * 64 + src;
            }
            w += cnt;
        }
    }
    if (w > 64) w = 64;  // callers guarantee at most 64 waiting requests
    // rank among the gathered keys (all distinct: seq is unique per replica)
    int rank = 0;
    for (int j = 0; j < w; ++j) rank += rl64(key, j) < key ? 1 : 0;
    if (lane >= w) rank = lane;
    // sort: lane r receives the request of rank r
    const int ad = rank * 4;
    const uint32_t k_lo = uint32_t(__builtin_amdgcn_ds_permute(ad, int(uint32_t(key))));
    const uint32_t k_hi = uint32_t(__builtin_amdgcn_ds_permute(ad, int(uint32_t(key >> 32))));
    word = uint32_t(__builtin_amdgcn_ds_permute(ad, int(word)));
    meta = uint32_t(__builtin_amdgcn_ds_permute(ad, int(meta)));
    ta = uint32_t(__builtin_amdgcn_ds_permute(ad, int(ta)));
    slot = __builtin_amdgcn_ds_permute(ad, slot);
    key = (static_cast<unsigned long long>(k_hi) << 32) | k_lo;
    admit_ranked(C, i, t, lane, w, key, word, meta, ta, slot);
}

// Admission of instance i from its head of line and the requests cached behind
// it, which are the smallest keys of its queue in order: the longest fitting
// prefix is admitted at once (admit_ranked).  When all of them fit and more
// wait, the head of line is unknown afterwards.
template <bool XT>
__device__ inline void admit_cached(const Ctx& C, int i, uint32_t t, int lane)
{
    const int n = C.qn[i];
    // (XT, the kernels for more than 64 instances) the extension follows the ring
    const int xv = XT ? C.xn[i] : 0, xc = xv & 0xFFFF, xh = xv >> 16;
    const int w = min(64, n + xc + 1);
    unsigned long long key = kNone;
    uint32_t word = 0, meta = 0, ta = 0;
    int slot = 0;
    if (lane == 0) {
        key = C.holk[i]; word = C.hwd[i]; meta = C.hmt[i]; ta = C.hta[i]; slot = C.hols[i];
    } else if (lane < w) {
        const uint4 e = !XT || lane <= n ? C.qt[qc_at(C, i, lane - 1)] : *qx_at(C, i, xh, lane - n - 1);
        const uint32_t tier = (e.w >> 12) & 15u;
        key = qc_key(C, e);
        word = e.y;
        meta = kWaiting | (tier << 2) | (((e.w >> 16) & 1u) << 6);
        ta = e.z;
        slot = int(e.w & 0xFFFu);
    }
    if constexpr (!XT) {
        admit_ranked(C, i, t, lane, w, key, word, meta, ta, slot, C.nwait[i] == w);
    } else {
    // While whole windows fit, the next 64 entries of the extension are on
    // their way when a window is admitted: one memory round trip per window, and
    // none for the head of line in between.
    int nr = n, x0 = xh, xr = xc, wn = w;
    for (;;) {
        const int at = x0 + (wn - 1 - nr);  // of the entries behind the window
        const int x1 = at >= C.xd ? at - C.xd : at, rest = xr - (wn - 1 - nr);
        const int dem = lane < wn ? blocks_of(wlo(word), C.shift) : 0;
        const bool all = rl(wscan(dem, lane), 63) <= C.freeb[i] && rest > 0;
        uint4 nx = make_uint4(0u, 0u, 0u, 0u);
        if (all && lane < rest) nx = *qx_at(C, i, x1, lane);
        admit_ranked(C, i, t, lane, wn, key, word, meta, ta, slot, C.nwait[i] == wn, nr, x0, xr, all);
        if (!all) return;
        // (the window's first entry stands for the head of line)
        wn = min(64, rest);
        nr = 0;
        x0 = x1 + 1 == C.xd ? 0 : x1 + 1;
        xr = rest - 1;
        const uint32_t tier = (nx.w >> 12) & 15u;
        key = lane < wn ? qc_key(C, nx) : kNone;
        word = nx.y;
        meta = kWaiting | (tier << 2) | (((nx.w >> 16) & 1u) << 6);
        ta = nx.z;
        slot = int(nx.w & 0xFFFu);
    }
    }
}

// Admission of instance i whose waiting requests all arrived in the previous
// tick (kept in LDS by the dispatch): they are listed in dispatch order,
// which is (tier, seq) order, so no HBM read and no ranking is needed.
__device__ inline void admit_fresh(const Ctx& C, int i, uint32_t t, int lane)
{
    const int n = *C.lastn;
    const bool mine = lane < n && (C.lsl[lane] >> 16) == uint32_t(i);
    const unsigned long long mm = ballot(mine);
    const int w = __popcll(mm);
    // lane r receives the list index of the r-th request of i
    const int dest = mine ? __popcll(mm & lanemask_lt()) : w + __popcll(~mm & lanemask_lt());
    const int idx = __builtin_amdgcn_ds_permute(dest * 4, lane);
    unsigned long long key = kNone;
    uint32_t word = 0, meta = 0, ta = 0;
    int slot = 0;
    if (lane < w) {
        const uint32_t e = C.lsl[idx];
        const uint32_t tier = (e >> 12) & 15u;
        word = C.lw[idx];
        meta = kWaiting | (tier << 2);
        ta = t - 1u;
        slot = int(e & 0xFFFu);
        key = (rank_of(C, tier) << 32) | C.lsq[idx];
    }
    admit_ranked(C, i, t, lane, w, key, word, meta, ta, slot);
}

// Admission of every instance whose waiting requests all arrived in the
// previous tick and whose head of line fits (one-wave kernels).  The dispatch's
// list in LDS holds those requests in (tier, seq) order, one per lane; each
// instance admits the longest prefix of its own requests whose summed demand
// fits, and its next request becomes the head of line.  One pass over the list
// serves all instances, whatever their number: a lane writes its own request,
// and an instance's totals are combined by LDS atomics.  (A pass per instance
// and a lane-parallel round for the instances with one request took the sweep
// 10.85 ms per 1000 ticks, this one 10.2.)
__device__ inline void admit_fresh_all(const Ctx& C, uint32_t t, int lane)
{
    const bool in = lane < *C.lastn;
    const uint32_t e = in ? C.lsl[lane] : 0u;
    const uint32_t word = in ? C.lw[lane] : 0u, seq = in ? C.lsq[lane] : 0u;
    const int i = int(e >> 16), slot = int(e & 0xFFFu), tier = int((e >> 12) & 15u);
    const int fr = C.freeb[i], fs = C.frs[i], h = C.hols[i], hd = C.hold[i], nwi = C.nwait[i];
    const bool act = in && fs && h >= 0 && hd <= fr;
    const int dem = act ? blocks_of(wlo(word), C.shift) : 0;
    // per instance: the running sum of the demands and the lanes of its requests
    // (an instance with one request is done at once)
    const int nw = act ? nwi : 0;
    int pre = dem;
    unsigned long long own = act ? 1ull << lane : 0ull;
    for (unsigned long long m = ballot(act && nw > 1); m;) {
        const int ii = rl(i, ffs64(m));
        const bool mine = act && i == ii;
        const unsigned long long mm = ballot(mine);
        const int p = wscan(mine ? dem : 0, lane);
        if (mine) { pre = p; own = mm; }
        m &= ~mm;
    }
    const bool adm = act && pre <= fr;
    const unsigned long long am = ballot(adm) & own;
    const int na = __popcll(am), cnt = __popcll(own), idx = __popcll(own & lanemask_lt());
    wave_sync();
    if (adm) {
        const uint32_t len = wlo(word), rem = wmid(word), fin = t + rem;
        const uint32_t place = wheel_put(C, fin, i, slot);
        s_set_wm(C, size_t(i) * C.S + slot, kRunW | ((fin & kFin) << 16) | (len + rem),
                 (uint32_t(tier) << 2) | kRunning | kAdmitted | place);
        // (a request's first admission, one tick after it arrived)
        stat(C, tier * 8 + kAdmittedCnt, 1);
        stat(C, tier * 8 + kQdelay, 1);
        hist_add(C, kHistQdelay, tier, 1);
        c16_inc(C.res, res_idx(C, i, (len - t - 1u) & C.bmask));
        tier_inc(C, i, tier);
        atomicSub(&C.freeb[i], dem);
        atomicAdd(&C.held[i], dem);
    }
    if (act) {
        const uint32_t meta = kWaiting | (uint32_t(tier) << 2);
        if (idx == 0) {
            atomicAdd(&C.B[i], na);
            atomicSub(&C.nwait[i], na);
            if (cnt != nw) stat(C, kInvariant, 1);
            if (na == cnt) clear_hol(C, i);
            else if (C.td) { C.qn[i] = min(cnt - na - 1, C.td); C.qh[i] = 0; }
        }
        if (idx == na) set_hol(C, i, slot, (rank_of(C, uint32_t(tier)) << 32) | seq, word, meta, t - 1u);
        else if (C.td && idx > na && idx - na - 1 < C.td)
            C.qt[i * C.td + idx - na - 1] = qc_pack(seq, slot, word, meta, t - 1u);
    }
    wave_sync();
}

// Admission of instance i's known head of line, which fits (per lane: the
// lane-parallel rounds call it for their lanes' instances; the next head of
// line comes from the queue cache or is left unknown).
__device__ inline void admit_head(const Ctx& C, int i, uint32_t t)
{
    const int h = C.hols[i], dem = C.hold[i];
    const uint32_t w = C.hwd[i], m = C.hmt[i];
    const uint32_t len = wlo(w), rem = wmid(w);
    const uint32_t fin = t + rem;
    const size_t hb = size_t(i) * C.S + h;
    const uint32_t place = wheel_put(C, fin, i, h);
    s_set_wm(C, hb, kRunW | ((fin & kFin) << 16) | (len + rem), (m & 0xFCu) | kRunning | kAdmitted | place);
    const int tier = int((m >> 2) & 15u);
    if (!(m & kAdmitted)) {
        stat(C, tier * 8 + kAdmittedCnt, 1);
        stat(C, tier * 8 + kQdelay, t - C.hta[i]);
        hist_add(C, kHistQdelay, tier, t - C.hta[i]);
    }
    C.freeb[i] -= dem;
    C.held[i] += dem;
    C.B[i] += 1;
    C.nwait[i] -= 1;
    c16_inc(C.res, res_idx(C, i, (len - t - 1u) & C.bmask));
    tier_inc(C, i, tier);
    hol_pop(C, i);
}

// The whole admission of instance i (uniform): requests are admitted in
// (tier, seq) order while the head of line fits (Section 3.1), through the
// same steps as the lane-parallel rounds -- a rescan when the head of line
// is unknown, the previous tick's placements, a gather of a short queue, a
// cached run, or one head of line -- until the head of line does not fit or
// nothing waits.  Every step admits at least one request, or finds the head
// of line, so the loop ends.  (The multi-wave kernels hand instances to waves
// dynamically with it.)
template <int GR, int MK, bool SEL>
__device__ inline void admit_all(const Ctx& C, int i, uint32_t t, int lane)
{
    for (;;) {
        const int h = C.hols[i];
        if (h == kHolUnknown) {
            rescan_admit<GR, MK, SEL>(C, i, t, lane);
            continue;
        }
        if (h < 0 || C.hold[i] > C.freeb[i]) break;
        const int nw = C.nwait[i];
        const bool cached = C.td && (C.qn[i] > 0 || qx_count(C, i) > 0);
        if (nw >= 2 && nw <= 64 && C.frs[i]) {
            admit_fresh(C, i, t, lane);
        } else if (nw >= 2 && nw <= 64 && !cached) {
            admit_batch<GR>(C, i, t, lane);
        } else if (cached) {
            admit_cached<SEL>(C, i, t, lane);
        } else {
            if (lane == 0) admit_head(C, i, t);
            wave_sync();
        }
    }
}

// ---------------------------------------------------------------------------
// Section 6.5 extensions, run at the start of a tick (uniform)
// ---------------------------------------------------------------------------

// Promotion pass: every waiting request of tier p >= 1 whose age t - tarr
// has reached the tier's quota (non-zero) moves to tier p - 1.  An instance
// with a promoted request loses its list of fresh placements and its queue
// cache; its head of line stays when it was not promoted and every promoted
// key is still larger, else it is found again by the admission rescan.
// lb <= the arrival tick of every waiting request of the instance, and every
// such tick is at most t (requests start to wait at the current tick or
// keep an older one): when t - lb is below the smallest quota no request can
// be old enough and the instance is not read.  lb = 0 means unknown (a
// launch that reads the slots starts so, as does an instance holding a request
// that arrived after t, possible only after the clock was moved back; a launch
// that resumes from the replica's image keeps lb).
template <int NW>
__device__ inline void promote_waiting(const Ctx& C, const Params& P, uint32_t t, int lane, int wid)
{
    const uint32_t qmin = P.ext[kXPromoMin];
    for (uint32_t i = uint32_t(wid); i < C.I; i += NW) {
        if (C.nwait[i] == 0) continue;
        const uint32_t lb = wlb(C)[i];
        if (lb != 0 && t - lb < qmin) continue;
        const size_t b = size_t(i) * C.S;
        const int nch = live_chunks(C, i, lane);
        const int h = C.hols[i];
        bool any = false, late = false, head = false;
        uint32_t lo = 0xFFFFFFFFu;
        unsigned long long kmin = kNone;
        // four chunks of 64 slots per memory round trip (one at a time took the
        // passes of the overloaded gauss10 workload 10.7K cycles a tick)
        for (int c0 = 0; c0 < nch; c0 += 4) {
            uint4 rr[4];
#pragma unroll
            for (int g = 0; g < 4; ++g) rr[g] = c0 + g < nch ? C.slot[b + (c0 + g) * 64 + lane] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint4 rec = rr[g];
                if (wst(rec.x) != 1u) continue;
                const int s = (c0 + g) * 64 + lane;
                const uint32_t m = rec.y, tier = (m >> 2) & 15u, ta = rec.w;
                lo = ta < lo ? ta : lo;
                late = late || ta > t;
                if (tier == 0) continue;
                const uint32_t q = P.ext[kXAge + tier];
                if (q != 0 && t - ta >= q) {
                    s_meta(C, b + s) = m - 4u;  // tier field at bits 2..5
                    any = true;
                    head = head || s == h;
                    const unsigned long long k = (rank_of(C, tier - 1u) << 32) | rec.z;
                    kmin = k < kmin ? k : kmin;
                }
            }
        }
        lo = wmin32(lo);
        kmin = wmin64(kmin);
        const bool moved = ballot(any) != 0, unknown = ballot(late) != 0, hit = ballot(head) != 0;
        if (lane == 0) {
            wlb(C)[i] = unknown ? 0u : lo;
            if (moved) {
                C.frs[i] = 0;
                if (hit || h < 0 || kmin < C.holk[i]) C.hols[i] = kHolUnknown;
                else if (C.td) C.qn[i] = 0;
                qx_clear(C, i);
            }
        }
    }
    wave_sync();
}

// Adaptive headroom update of replica r: lane p < 10 handles tier p, with
// the headroom and the counter snapshots in HBM.  With a requests first
// admitted since the last update and their summed queue delay d, the
// headroom rises by a step when d > slo a, falls by a step when
// 256 d <= margin slo a, both tests in exact 128-bit arithmetic.
__device__ inline void adapt_headroom(const Ctx& C, const Params& P, uint32_t r, int lane)
{
    if (lane < kTiers) {
        const int p = lane;
        int32_t* hq = ext_hqr(P) + size_t(r) * kTiers;
        unsigned long long* snap = ext_hsnap(P) + size_t(r) * 2 * kTiers;
        const unsigned long long adm = C.stats[p * 8 + kAdmittedCnt], qd = C.stats[p * 8 + kQdelay];
        const unsigned long long a = adm - snap[p], d = qd - snap[kTiers + p];
        snap[p] = adm;
        snap[kTiers + p] = qd;
        if (p < int(C.K) && !(P.ext[kXZeroLowest] && p == int(C.K) - 1) && a != 0) {
            const unsigned long long slo = P.ext[kXSlo + p];
            const unsigned long long xl = slo * a, xh = __umul64hi(slo, a);
            const unsigned long long ms = slo * P.ext[kXAdaptMargin];  // < 2^29
            const unsigned long long yl = ms * a, yh = __umul64hi(ms, a);
            const unsigned long long dl = d << 8, dh = d >> 56;
            long long h = hq[p];
            if (xh == 0 && d > xl) {
                h += P.ext[kXAdaptUp];
                const long long mx = P.ext[kXAdaptMax];
                if (h > mx) h = mx;
            } else if (dh < yh || (dh == yh && dl <= yl)) {
                h -= P.ext[kXAdaptDown];
                if (h < 0) h = 0;
            }
            hq[p] = int32_t(h);
        }
    }
    wave_sync();
}

// ---------------------------------------------------------------------------
// k_step
// ---------------------------------------------------------------------------
// A barrier of the replica's waves (a wave-level one when a replica has one
// wave): every LDS and memory write before it is seen by every wave after it.
template <int NW>
__device__ __forceinline__ void block_sync()
{
    if (NW > 1) __syncthreads();
    else wave_sync();
}

// the wave's next entry of a work list, by its cursor; uniform
__device__ __forceinline__ int next_of(int* cursor, int lane)
{
    int k = 0;
    if (lane == 0) k = atomicAdd(cursor, 1);
    return rl(k, 0);
}

// Image of a replica's LDS between launches: a header {tick it stands at,
// kImgMagic, layout, LDS bytes} and the bytes.  The layout holds what the LDS
// and the memory it points into are laid out by and the host can change:
// queue-cache depth | waves << 4 | wheel capacity << 8 | extension depth << 20.
// Both are uniform over the block.
constexpr uint32_t kImgMagic = 0x4C445331u;
static_assert(kMaxSlots < 1u << 12, "a wheel capacity and an extension depth (both at most kMaxSlots) fit 12 bits");
template <uint32_t NT>
__device__ __forceinline__ uint32_t img_layout(const Params& P) { return P.qdepth | (NT / 64u) << 4 | P.wcap << 8 | P.qxd << 20; }
template <uint32_t NT>
__device__ inline bool image_read(const Params& P, uint32_t r, uint32_t t, char* lds, uint32_t tid)
{
    if (r >= P.img_r) return false;
    const uint4* m = P.img + size_t(r) * P.img_n;
    const uint4 h = *uniform_ptr(m);
    if (h.x != t || h.y != kImgMagic || h.z != (img_layout<NT>(P)) || h.w != P.img_lds) return false;
    uint4* l = reinterpret_cast<uint4*>(lds);
    const uint32_t n = P.img_lds / 16u;
    for (uint32_t j = tid; j < n; j += 4 * NT) {
        uint4 v[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) v[k] = j + k * NT < n ? m[1 + j + k * NT] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
            if (j + k * NT < n) l[j + k * NT] = v[k];
    }
    if (NT > 64) __syncthreads();
    else wave_sync();
    return true;
}
template <uint32_t NT>
__device__ inline void image_write(const Params& P, uint32_t r, uint32_t t, const char* lds, uint32_t tid)
{
    if (r >= P.img_r) return;
    uint4* m = P.img + size_t(r) * P.img_n;
    const uint4* l = reinterpret_cast<const uint4*>(lds);
    const uint32_t n = P.img_lds / 16u;
    for (uint32_t j = tid; j < n; j += NT) m[1 + j] = l[j];
    if (tid == 0) m[0] = make_uint4(t, kImgMagic, img_layout<NT>(P), P.img_lds);
}

// A staged copy's request: the running candidate of source i of largest tier,
// then fewest blocks, then newest, its slot in the key's low bits (tier rank 4
// bits, blocks 16, seq 32, slot 12); 0: nothing to move (an empty draining
// source).  Wave wid of NW reads chunks wid, wid + NW, ... and returns its own
// best.  (One wave scanning 2048 slots took 8K cycles of the wide workload's
// tick; the one-wave kernels scan a source as its pair is made.)
template <int NW>
__device__ inline unsigned long long staged_best(const Ctx& C, int i, uint32_t t, int lane, int wid)
{
    if (C.B[i] == 0) return 0ull;
    const size_t b = size_t(i) * C.S;
    const int nch = live_chunks(C, i, lane);
    unsigned long long bk = 0;
    for (int c0 = wid; c0 < nch; c0 += 4 * NW) {
        uint32_t v[4], m[4], q[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int c = c0 + g * NW;
            const uint4 rr = c < nch ? C.slot[b + c * 64 + lane] : make_uint4(0u, 0u, 0u, 0u);
            v[g] = rr.x; m[g] = rr.y; q[g] = rr.z;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if (wst(v[g]) == 2u && !(m[g] & kMigrating)) {
                const uint32_t fin = fin_of(v[g], t);
                const uint32_t nb = uint32_t(65535 - blocks_of(wlo(v[g]) - (fin - t), C.shift));
                const unsigned long long kk =
                    (((rank_of(C, (m[g] >> 2) & 15u) + 1ull) << 48 | static_cast<unsigned long long>(nb) << 32 | q[g]) << 12) |
                    uint32_t((c0 + g * NW) * 64 + lane);
                bk = kk > bk ? kk : bk;
            }
        }
    }
    return wmax64(bk);
}

// The staged copy of the request of key mx (staged_best) from instance src to
// slot ds of dst starts; one lane.
__device__ inline void staged_start(const Ctx& C, int src, int dst, int ds, unsigned long long mx)
{
    const int cs = int(mx & 0xFFFu);
    s_set_wm(C, size_t(dst) * C.S + ds, kInbW, kInbound);
    C.occ[dst * C.W + (ds >> 6)] |= 1ull << (ds & 63);
    C.live[dst] += 1;
    atomicOr(&s_meta(C, size_t(src) * C.S + cs), kMigrating);
    int* m = &C.mig[4 * src];
    m[0] = dst; m[1] = cs; m[2] = ds; m[3] = 0;
    stat(C, kMigStarted, 1);
}

// Bursts' rests kept for placement by all waves; more are placed as they come.
constexpr int kMaxRuns = 8;
// Places the m arrivals from index k1 on of this tick (records rec) that all go
// to one instance, behind its head of line, on its m lowest empty slots (run
// a = {instance, k1, m, sequence number of arrival 0}, b = {append to the kept
// queue order, ring entries, extension's head << 16 | count before}).  Waves
// take batches of 64 in turn.  One wave placed a burst at some 2K cycles a
// batch of 64: 18 of the 26K cycles that the dispatch of the wide workload's
// bursts took of a tick.  (This and the windows of admit_cached: 17.98 -> 15.70
// ms per call there.)
template <int NW>
__device__ inline void place_run(const Ctx& C, const unsigned long long* rec, uint32_t t, uint4 a, uint4 b, int lane, int wid)
{
    const int i = int(a.x), m = int(a.z);
    const unsigned long long* ra = rec + a.y;
    const int nq = int(b.y), xc = int(b.z & 0xFFFFu), xh = int(b.z >> 16);
    // empty slots up to and including each occupancy word, one word per lane
    const unsigned long long wd = lane < int(C.W) ? C.occ[i * C.W + lane] : kNone;
    const int fw = 64 - int(__popcll(wd));
    const int pre = wscan(fw, lane);
    const uint32_t wlo32 = uint32_t(~wd), whi32 = uint32_t(~wd >> 32);
    for (int k0 = wid * 64; k0 < m; k0 += 64 * NW) {
        const int k = k0 + lane;
        const bool in = k < m;
        const unsigned long long ar = in ? ra[k] : 0ull;
        // the word that holds the k-th empty slot: the first whose count exceeds k
        int w = 0;
#pragma unroll
        for (int step = 32; step; step >>= 1) {
            const int v = __shfl(pre, w + step - 1);
            w += v <= k ? step : 0;
        }
        const int before = __shfl(pre, w > 0 ? w - 1 : 0);
        const uint32_t f0 = uint32_t(__shfl(int(wlo32), w & 63)), f1 = uint32_t(__shfl(int(whi32), w & 63));
        const bool ok = in && w < int(C.W);
        const int s = w * 64 + kth_set_bit(static_cast<unsigned long long>(f1) << 32 | f0, k - (w > 0 ? before : 0));
        const int tier = int((ar >> 32) & 15u);
        const uint32_t seq = a.w + unsigned(ar >> 36);
        if (ok) {
            const uint32_t word = kWaitW | (uint32_t((ar >> 16) & 0xFFFFu) << 16) | uint32_t(ar & 0xFFFFu);
            C.slot[size_t(i) * C.S + s] = make_uint4(word, kWaiting | (uint32_t(tier) << 2), seq, t);
            if (b.x) {
                const uint4 en = make_uint4(seq, word, t, uint32_t(s) | (uint32_t(tier) << 12));
                const int at = xc > 0 ? C.td : nq + k;  // place behind the head while the ring has room
                const int e = xc > 0 ? xc + k : nq + k - C.td;
                if (at < C.td) C.qt[qc_at(C, i, at)] = en;
                else if (e < C.xd) *qx_at(C, i, xh, e) = en;
            }
            stat(C, tier * 8 + kArrived, 1);
            stat(C, tier * 8 + kDispatched, 1);
        } else if (in) {  // occupancy and live count disagree: flag, drop the arrival
            stat(C, kInvariant, 1);
            stat(C, tier * 8 + kArrived, 1);
            stat(C, tier * 8 + kRejected, 1);
        }
    }
    __syncthreads();
    if (wid == 0) {
        // the m lowest empty slots are taken
        const int take = min(fw, m - (pre - fw));
        if (lane < int(C.W) && take > 0) {
            const int p = kth_set_bit(~wd, take - 1);
            C.occ[i * C.W + lane] = wd | (p == 63 ? kNone : (2ull << p) - 1ull);
        }
        if (b.x && lane == 0) {
            const int r = xc > 0 ? 0 : min(m, C.td - nq);  // entered the ring
            C.qn[i] = nq + r;
            const int ne = min(C.xd, xc + m - r);
            C.xn[i] = ne > 0 ? (xh << 16) | ne : 0;
        }
    }
    __syncthreads();
}

// v, with the load that produces it complete
__device__ __forceinline__ unsigned long long landed(unsigned long long v)
{
    uint32_t lo = uint32_t(v), hi = uint32_t(v >> 32);
    asm volatile("" : "+v"(lo), "+v"(hi));
    return (static_cast<unsigned long long>(hi) << 32) | lo;
}

template <int IM, bool INF, bool EXT, bool QC, int NW>
__global__ __launch_bounds__(64 * NW, IM <= 64 ? 4 : 2) void k_step(Params P, unsigned long long t0, uint32_t nt)
{
    // IPL: instances per lane when one wave covers every instance (the serial
    // phases, run by wave 0); OPL: instances per lane of the instances a wave
    // owns in the per-instance phases, instance (64 j + lane) NW + wid
    constexpr bool WIDE = IM >= 128;
    constexpr int IPL = (IM + 63) / 64;
    constexpr int OPL = (IM + 64 * NW - 1) / (64 * NW);
    extern __shared__ __align__(16) char lds_raw[];
    Ctx C = carve<IM, INF, EXT, QC, NW>(lds_raw, P);
    const int lane = lane_id();
    const int wid = NW > 1 ? int(threadIdx.x >> 6) : 0;
    const uint32_t tid = threadIdx.x;
    constexpr uint32_t NT = 64u * NW;
    const uint32_t I = P.I, S = P.S, W = P.W;
    const uint32_t wsz = P.wsz;
    constexpr bool infaas = INF;  // the global policy: INFaaS cost, else Llumnix freeness

    for (uint32_t r = blockIdx.x; r < P.R; r += gridDim.x) {
        const uint32_t g = P.group_of[r];
        C.K = P.group_K32[g];
        const int32_t* hq = P.hq + g * kTiers;
        if (EXT) {
            // (the parameters are read from memory where they are used, so that
            // none of them stays in registers through the tick loop)
            const int32_t* hqr = ext_hqr(P);
            if (hqr) hq = hqr + size_t(r) * kTiers;
        }
        const size_t rb = size_t(r) * I * S;
        C.slot = P.slot + rb;
        if (C.xn) C.qx = P.qx + size_t(r) * I * P.qxd;
        C.wheel = P.wheel + size_t(r) * wsz * P.wcap;
        C.hist = P.hist + size_t(r) * kHistPerReplica;

        const uint32_t t0u = uint32_t(t0);
        // ---------------- prologue: derived per-instance state ----------------
        // The last launch left its LDS in the replica's image; it is taken up
        // again when nothing changed the state since (the image's tick is this
        // launch's first and its layout is the same; imports and clock moves
        // void it).  Reading every slot instead was 3.3K of the 19.4K cycles of
        // an enterprise tick in 50-tick steps (523 us a step, 459 with the
        // image) and 8.1K of 36K of the sweep's in 52-tick launches (2.75 ms per
        // 104 ticks, 2.01).
        const bool warm = image_read<NT>(P, r, t0u, lds_raw, tid);
        if (warm) {
            for (uint32_t i = tid; i < I; i += NT) C.drn[i] = P.drain[size_t(r) * I + i];
        } else {
        for (uint32_t j = tid; j < uint32_t(kNstat); j += NT) C.stats[j] = P.stats[size_t(r) * kNstat + j];
        for (uint32_t i = tid; i < I; i += NT) {
            C.freeb[i] = P.freeb[size_t(r) * I + i];
            C.drn[i] = P.drain[size_t(r) * I + i];
            for (int k = 0; k < 4; ++k) C.mig[4 * i + k] = P.mig[(size_t(r) * I + i) * 4 + k];
            C.inb[i] = 0;
            C.flags[i] = 0;
            C.tmask[i] = 0;
            C.frs[i] = 0;
            if (C.td) { C.qn[i] = 0; C.qh[i] = 0; }
            if (C.xn) C.xn[i] = 0;
            if (C.svc) C.svc[i] = P.svc[size_t(r) * I + i];
        }
        for (uint32_t b = tid; b < wsz / 2; b += NT) C.wc[b] = 0;
        if (tid == 0) { *C.lastn = 0; *C.nvic = 0; }
        for (uint32_t b = tid; b < (I * C.RB + 1) / 2; b += NT) C.res[b] = 0;
        for (uint32_t b = tid; b < (I * kTiers + 1) / 2; b += NT) C.tcnt[b] = 0;
        for (uint32_t b = tid; b < (wsz + 31) / 32; b += NT) C.wov[b] = 0;
        block_sync<NW>();
        for (uint32_t i = tid; i < I; i += NT) {
            const int d = C.mig[4 * i];
            if (d >= 0) C.inb[d] = C.mig[4 * i + 3];
        }
        block_sync<NW>();
        {
            // The slots are read as one flat run of I * W chunks of 64 (chunk c
            // of instance i is flat chunk i W + c), GP chunks per memory round
            // trip; an instance is summed up after its last chunk.  The arrival
            // ticks of the heads of line are read afterwards, lane-parallel.
            // (each wave reads the chunks of the instances it owns: wid, wid + NW, ...)
            constexpr int GP = IM >= 128 ? 16 : 8;
            const uint32_t nown = NW > 1 ? (I > uint32_t(wid) ? (I - uint32_t(wid) + NW - 1) / NW : 0u) : I;
            const uint32_t nfl = nown * W;
            int nB = 0, nlive = 0, nw = 0, held = 0;
            unsigned long long bk = kNone;
            int bs = 0;
            uint32_t bv = 0, bm = 0;
            for (uint32_t f0 = 0; f0 < nfl; f0 += GP) {
                uint32_t v[GP], m[GP], q[GP];
#pragma unroll
                for (int g = 0; g < GP; ++g) {
                    const bool in = f0 + g < nfl;
                    const uint32_t fo = (f0 + g) / W;
                    const size_t fs = (size_t(fo * NW + wid) * W + (f0 + g - fo * W)) * 64 + lane;
                    const uint4 rr = in ? C.slot[fs] : make_uint4(0u, 0u, 0u, 0u);
                    v[g] = rr.x; m[g] = rr.y; q[g] = rr.z;
                }
#pragma unroll
                for (int g = 0; g < GP; ++g) {
                    const uint32_t f = f0 + g;
                    if (f >= nfl) continue;
                    const uint32_t io = f / W, c = f - io * W, i = io * NW + uint32_t(wid);
                    const int s = int(c) * 64 + lane;
                    const uint32_t st = wst(v[g]);
                    const unsigned long long ow = ballot(v[g] != 0);
                    nlive += __popcll(ow);
                    nB += __popcll(ballot(st == 2u));
                    nw += __popcll(ballot(st == 1u));
                    if (lane == 0) C.occ[i * W + c] = ow;
                    if (st == 2u) {
                        const uint32_t lenf = wlo(v[g]), fin = fin_of(v[g], t0u);
                        held += blocks_of(lenf - (fin - t0u + 1u), C.shift);
                        c16_inc(C.res, res_idx(C, i, (lenf - fin - 1u) & C.bmask));
                        c16_inc(C.tcnt, i * kTiers + int((m[g] >> 2) & 15u));
                        const uint32_t place = wheel_put(C, fin, int(i), s);
                        if (C.td) s_meta(C, size_t(i) * S + s) = (m[g] & 0xFFu) | place;
                    } else if (st == 1u) {
                        const unsigned long long k = (rank_of(C, (m[g] >> 2) & 15u) << 32) | q[g];
                        if (k < bk) { bk = k; bs = s; bv = v[g]; bm = m[g]; }
                    }
                    if (c + 1 == W) {
                        held = wsum(held);
                        const unsigned long long mn = wmin64(bk);
                        int hs = kNoHol;
                        uint32_t hw = 0, hm = 0;
                        if (mn != kNone) {
                            const int wl = ffs64(ballot(bk == mn));
                            hs = rl(bs, wl);
                            hw = rlu(bv, wl);
                            hm = rlu(bm, wl);
                        }
                        if (lane == 0) {
                            C.B[i] = nB; C.live[i] = nlive; C.nwait[i] = nw;
                            C.held[i] = held;
                            if (hs >= 0) set_hol(C, int(i), hs, mn, hw, hm, 0u);
                            else clear_hol(C, int(i));
                            int tm = 0;
                            for (int p = 0; p < kTiers; ++p) tm |= c16_get(C.tcnt, i * kTiers + p) ? (1 << p) : 0;
                            C.tmask[i] = tm;
                        }
                        wave_sync();
                        nB = 0; nlive = 0; nw = 0; held = 0;
                        bk = kNone; bs = 0; bv = 0; bm = 0;
                    }
                }
            }
            block_sync<NW>();
            for (uint32_t i = tid; i < I; i += NT) {
                const int h = C.hols[i];
                if (h >= 0) C.hta[i] = s_tarr(C, size_t(i) * S + h);
            }
        }
        }
        if (EXT) {
            if (tid == 0) {
                const uint32_t per = P.ext[kXPromoPeriod], ep = P.ext[kXAdaptEpoch];
                xleft(C)[0] = per ? int(t0u % per) : 0;
                xleft(C)[1] = ep ? int(t0u % ep) : 0;
            }
            // (unknown: the first pass reads them)
            if (!warm)
                for (uint32_t i = tid; i < P.I; i += NT) wlb(C)[i] = 0u;
        }
        if (NW > 1 && tid == 0) { *C.gln = 0; *C.glnext = 0; }
        if (wid == 0) headroom_table(C, hq, lane);
        unsigned next_seq = P.next_seq[r];
        // slot-ticks per lane of a chunk of at most 1024 ticks: a tick adds at most
        // OPL x 2048 to run_acc, and to wait_acc as many after admission, IPL x 2048
        // placed by the dispatch and on lane 0 kMaxRuns bursts' rests: below 2^25
        static_assert(OPL == 1 && IPL <= 4 && kMaxRuns <= 8, "1024 ticks of slot counts fit 32 bits");
        uint32_t run_acc = 0, wait_acc = 0;
        const unsigned long long* recs = P.arr_rec + size_t(r) * P.chunk * P.arr_cap;
        const uint32_t* cnts = P.arr_cnt + size_t(r) * P.chunk;
        block_sync<NW>();

        // the arrivals of the next tick are loaded one tick ahead; records past
        // the tick's count are never used
        const uint32_t lim = P.arr_cap < 64u ? P.arr_cap : 64u;
        // arrival counts 64 ticks at a time, lane l holding tick (tl & ~63) + l:
        // a tick's count is a lane read of a register, so no tick waits for
        // a load (and for the stores before it) to make its count uniform
        uint32_t cnt64 = uint32_t(lane) < nt ? cnts[lane] : 0u;
        // The finish visits are loaded ahead in two stages, both right after a
        // tick's own visit: the entries of the bucket two ticks ahead (pf2_n of
        // them; kNoPf: none), and the slots' word, meta and arrival tick of the
        // entries loaded a tick earlier for the next tick's bucket (pf_n, pf_e,
        // pf_v, pf_m, pf_a).  A visit uses them when its bucket still holds
        // exactly pf_n entries (appends, such as a committed migration's new
        // entry, change the count) and no preemption touched a slot in between
        // (victims' entries are dropped, more victims than the list holds drop
        // the whole set); otherwise it loads again.  A running request's word,
        // tier and arrival tick never change while it runs, and whether it is
        // being copied out is read from the migration records at the visit.
        constexpr uint32_t kNoPf = 0xFFFFFFFFu;
        uint32_t pf_n = kNoPf, pf_e = 0, pf_v = 0, pf_m = 0, pf_a = 0;
        uint32_t pf2_n = kNoPf, pf2_e = 0;
        // (wave 0) ticks to the next pairing round, and whether a migration
        // record may be active (the staged-copy phase is skipped otherwise)
        uint32_t mig_left = (P.mig_interval - t0u % P.mig_interval) % P.mig_interval;
        bool migs = false;
        for (uint32_t i = lane; i < I; i += 64) migs = migs || C.mig[4 * i] >= 0;
        migs = ballot(migs) != 0;
        unsigned long long a_nx = uint32_t(lane) < lim ? recs[lane] : 0ull;
        for (uint32_t tl = 0; tl < nt; ++tl) {
            const uint32_t t = t0u + tl;
            const uint32_t n = rlu(cnt64, int(tl & 63u));
            const unsigned long long* rec = recs + size_t(tl) * P.arr_cap;
            // the records are waited for here, with the prefetched finish visit: at
            // their use the wait would take in the stores and histogram atomics
            // that the phases in between have just issued
            const unsigned long long a0 = landed(a_nx);

            // ============ Section 6.5: promotion, adaptive headroom ============
            // (the countdowns and parameters live in LDS: nothing of this stays
            // in registers across the tick)
            if (EXT) {
                const int pl = xleft(C)[0], al = xleft(C)[1];
                const int per = int(P.ext[kXPromoPeriod]), ep = int(P.ext[kXAdaptEpoch]);
                if (per && pl == 0) promote_waiting<NW>(C, P, t, lane, wid);
                if (wid == 0 && ep && al == 0) adapt_headroom(C, P, r, lane);
                block_sync<NW>();
                if (ep && al == 0) {
                    if (wid == 0) headroom_table(C, ext_hqr(P) + size_t(r) * kTiers, lane);
                    block_sync<NW>();
                }
                if (tid == 0) {
                    xleft(C)[0] = per && pl + 1 < per ? pl + 1 : 0;
                    xleft(C)[1] = ep && al + 1 < ep ? al + 1 : 0;
                }
            }

            // ===================== A: growth, preemption, finish =====================
            // an instance whose growth fits takes its blocks at once; the others
            // preempt first (and take them at the end of preempt)
            const uint32_t cres = (0u - t) & C.bmask;
            unsigned long long pre[OPL];
            bool preempting = false;
#pragma unroll
            for (int j = 0; j < OPL; ++j) {
                const uint32_t i = (uint32_t(lane) + 64u * j) * NW + uint32_t(wid);
                bool np = false;
                if (i < I) {
                    const int G = int(c16_get(C.res, res_idx(C, i, cres)));
                    const int fr = C.freeb[i], he = C.held[i];
                    np = G > fr;
                    if (np) {
                        C.gtmp[i] = G;
                    } else {
                        C.freeb[i] = fr - G;
                        C.held[i] = he + G;
                    }
                    if (INF) C.flags[i] &= ~kFlagIntf;
                    if (C.fsum) { C.fsum[i] = 0; C.fcnt[i] = 0; }
                }
                pre[j] = ballot(np);
                preempting = preempting || pre[j] != 0;
                if (NW > 1 && !WIDE && np) C.order[atomicAdd(C.gln, 1)] = int(i);
            }
            // migrations to abort: set by preemption and finish, kept in a register
            // (multi-wave kernels: another wave's preemption sets the block flag)
            bool abort_any = false;
            if constexpr (NW > 1 && !WIDE) {
                // Four waves: the preempting instances are listed and the waves take
                // them one at a time, as in admission below.  With each wave on the
                // instances it owns, the others waited for the one with most of
                // them: 15K of the overloaded study's 97K cycles a tick.
                if (tid == 0) {
                    *C.bsum = 0;  // the auto-scaling sum of this tick (phase C)
                    *C.wln = 0;   // the admission work list (phase B)
                    *C.wlnext = 0;
                }
                block_sync<NW>();
                const int ng = *C.gln;
                if (ng) {
                    for (int k = next_of(C.glnext, lane); k < ng; k = next_of(C.glnext, lane))
                        abort_any = preempt<4, 1, QC>(C, C.order[k], t, lane) || abort_any;
                    if (abort_any && lane == 0) *C.bflag = 1;
                    block_sync<NW>();
                }
                if (wid == 0) {
                    // (every wave has read the list's length where it is not 0)
                    if (lane == 0) { *C.gln = 0; *C.glnext = 0; }
                    preempting = *C.nvic != 0;
                    abort_any = *C.bflag != 0;
                }
            } else if (preempting) {
                wave_sync();
#pragma unroll
                for (int j = 0; j < OPL; ++j)
                    for (unsigned long long m = pre[j]; m; m &= m - 1)
                        abort_any = preempt<(IM >= 128 ? 16 : 4), (IM >= 128 ? 2 : 1), QC && IM < 128>(
                                        C, int((64u * j + ffs64(m)) * NW + uint32_t(wid)), t, lane) || abort_any;
            }
            // a bucket of more than 64 entries is visited by every wave (the count
            // and the overflow flag are read here, where no wave writes them:
            // all waves take the same branch)
            bool by_all = false;
            uint32_t nb_all = 0;
            if (WIDE) {
                const uint32_t bk = t & C.wmask;
                nb_all = (C.wc[bk >> 1] >> ((bk & 1u) * 16u)) & 0xFFFFu;
                by_all = nb_all > 64u && !((C.wov[bk >> 5] >> (bk & 31u)) & 1u);
            }
            if (WIDE) {
                if (abort_any && lane == 0) *C.bflag = 1;
                if (tid == 0) {
                    *C.bsum = 0;  // the auto-scaling sum of this tick (phase C)
                    *C.wln = 0;   // the admission work list (phase B)
                    *C.wlnext = 0;
                    *C.kcnt = 0;
                }
                block_sync<NW>();
                if (wid == 0) {
                    preempting = *C.nvic != 0;
                    abort_any = *C.bflag != 0;
                }
            }
            if constexpr (WIDE) {
                if (by_all) {
                    bool ab = false;
                    finish_wide<NW>(C, t, lane, wid, nb_all, ab);
                    if (ab && lane == 0) *C.bflag = 1;
                    block_sync<NW>();
                    if (wid == 0) {
                        wheel_set_count(C, t & C.wmask, uint32_t(*C.kcnt), lane);
                        abort_any = *C.bflag != 0;
                    }
                }
            }
            // a preempted request is waiting now: its prefetched entries (for this
            // tick's and the next tick's visit) are dropped (its wheel entry was
            // erased); more victims than the list holds make both visits load again
            bool pf_lost = false;
            if (preempting && wid == 0) {
                const int nv = *C.nvic;
                pf_lost = nv > kVic;
                for (int v = 0; v < nv && v < kVic; ++v) {
                    if (pf_e == C.vic[v]) pf_e = kTomb;
                    if (pf2_e == C.vic[v]) pf2_e = kTomb;
                }
            }
            wave_sync();
            // the finish visit and the release of aborted migrations: wave 0
            if (wid == 0) {
            if (lane == 0) *C.nvic = 0;
            {
                const uint32_t bk = t & C.wmask;
                const uint32_t nb = (C.wc[bk >> 1] >> ((bk & 1u) * 16u)) & 0xFFFFu;
                const bool ov = (C.wov[bk >> 5] >> (bk & 31u)) & 1u;
                if (WIDE && by_all) {  // (without WIDE here the others' code came out 5 % slower)
                    // (visited above)
                } else if (pf_n != kNoPf && !pf_lost && !ov && nb == pf_n) {
                    uint32_t* ent = C.wheel + size_t(bk) * C.wcap;
                    const uint32_t kept = finish_batch(C, t, lane, ent, 0, uint32_t(lane) < pf_n, pf_e, pf_v, pf_m, pf_a,
                                                       abort_any);
                    wheel_set_count(C, bk, kept, lane);
                } else {
                    finish_tick(C, t, lane, abort_any);
                }
                // slots of the next tick's bucket, from the entries loaded a tick ago
                pf_n = pf_lost ? kNoPf : pf2_n;
                pf_e = pf2_e;
                if (pf_n != kNoPf) {
                    const uint32_t pi = pf_e >> 16, ps = pf_e & 0xFFFFu;
                    const bool ok = uint32_t(lane) < pf_n && pi < I && ps < S;
                    const size_t idx = size_t(pi) * S + ps;
                    const uint4 rec = ok ? C.slot[idx] : make_uint4(0u, 0u, 0u, 0u);
                    pf_v = rec.x; pf_m = rec.y; pf_a = rec.w;
                }
                // entries of the bucket two ticks ahead (three distinct buckets needed)
                const uint32_t b2 = (t + 2u) & C.wmask;
                const uint32_t n2 = (C.wc[b2 >> 1] >> ((b2 & 1u) * 16u)) & 0xFFFFu;
                const bool ov2 = (C.wov[b2 >> 5] >> (b2 & 31u)) & 1u;
                pf2_n = !ov2 && n2 <= 64u && C.wmask >= 3u ? n2 : kNoPf;
                pf2_e = pf2_n != kNoPf && uint32_t(lane) < pf2_n ? C.wheel[size_t(b2) * C.wcap + lane] : 0u;
            }
            // ===================== A2: release reservations of aborted migrations =====================
            if (abort_any) {
                for (uint32_t i = lane; i < I; i += 64) {
                    if (!(C.flags[i] & kFlagAbort)) continue;
                    C.flags[i] &= ~kFlagAbort;
                    int* m = &C.mig[4 * i];
                    const int d = m[0];
                    if (d < 0) continue;
                    C.freeb[d] += m[3];
                    C.inb[d] = 0;
                    const size_t db = size_t(d) * S + m[2];
                    s_word(C, db) = 0;
                    C.occ[d * W + (m[2] >> 6)] &= ~(1ull << (m[2] & 63));
                    C.live[d] -= 1;
                    m[0] = -1; m[1] = 0; m[2] = 0; m[3] = 0;
                    stat(C, kMigAborted, 1);
                }
                wave_sync();
            }
            if (NW > 1 && lane == 0) *C.bflag = 0;
            }  // wave 0
            block_sync<NW>();

            // ===================== B: admission (lane-parallel rounds); C: freeness =====================
            // Eight-wave kernels: the instances with admission work (an unknown
            // head of line, or a known one that fits) are listed, and the waves
            // take them one at a time from the list, each admitting on its
            // instance to the end: a few long queues no longer load one wave.
            // Admissions on different instances touch only their own state and
            // shared counters, so the order does not matter.
            if (WIDE) {
#pragma unroll
                for (int j = 0; j < OPL; ++j) {
                    const uint32_t i = (uint32_t(lane) + 64u * j) * NW + uint32_t(wid);
                    const bool need = i < I && (C.hols[i] == kHolUnknown || (C.hols[i] >= 0 && C.hold[i] <= C.freeb[i]));
                    if (need) C.order[atomicAdd(C.wln, 1)] = int(i);
                }
                block_sync<NW>();
                const int nl = *C.wln;
                for (int k = next_of(C.wlnext, lane); k < nl; k = next_of(C.wlnext, lane))
                    admit_all<16, 3, true>(C, C.order[k], t, lane);
                // phase C reads the instances each wave owns, which any wave
                // may have admitted on
                block_sync<NW>();
            } else if constexpr (NW > 1) {
                // Four waves: each lane admits the known heads of line of its
                // instance that fit one by one; what takes a whole wave -- a
                // rescan, the previous tick's arrivals, a gather -- is listed and
                // taken as above.  (Each wave on its own instances left the others
                // waiting for 16K of the overloaded study's 97K cycles a tick;
                // this and the preemptions' list: 23.33 -> 21.08 ms per 500 ticks.
                // Eight chunks of slots a round trip instead of four: 22.65, for
                // 77 spilled registers instead of 48.)
                const int i = lane * NW + wid;
                if (uint32_t(i) < I) {
                    const int h = C.hols[i], hd = C.hold[i], fr = C.freeb[i], nw = C.nwait[i], fs = C.frs[i], qn = C.qn[i];
                    bool need = h == kHolUnknown;
                    if (h >= 0 && hd <= fr) {
                        need = fs || (nw >= 2 && nw <= 64 && qn == 0);
                        if (!need) {
                            do {
                                admit_head(C, i, t);
                            } while (C.hols[i] >= 0 && C.hold[i] <= C.freeb[i]);
                            need = C.hols[i] == kHolUnknown;
                        }
                    }
                    if (need) C.order[atomicAdd(C.wln, 1)] = i;
                }
                block_sync<NW>();
                const int nl = *C.wln;
                if (nl) {
                    for (int k = next_of(C.wlnext, lane); k < nl; k = next_of(C.wlnext, lane))
                        admit_all<4, 2, false>(C, C.order[k], t, lane);
                    block_sync<NW>();
                }
            } else {
                // lane l holds instance l; its summary is read once per round
                const int i = lane;
                const bool own = uint32_t(i) < I;
                for (;;) {
                    int h = kNoHol, hd = 0, fr = 0, nw = 0, fs = 0, qn = 0;
                    auto look = [&] {
                        if (own) {
                            h = C.hols[i]; hd = C.hold[i]; fr = C.freeb[i]; nw = C.nwait[i]; fs = C.frs[i];
                            if (C.td) qn = C.qn[i];
                        }
                    };
                    look();
                    // heads of line left unknown: found by a rescan, which admits at once
                    bool any = false;
                    const unsigned long long um = ballot(h == kHolUnknown);
                    if (um) {
                        for (unsigned long long m = um; m; m &= m - 1)
                            any = rescan_admit<4, 2>(C, ffs64(m), t, lane) || any;
                        look();
                    }
                    const bool fits = h >= 0 && hd <= fr;
                    // queues that hold the previous tick's arrivals only
                    const unsigned long long fm = ballot(fits && fs);
                    if (fm) admit_fresh_all(C, t, lane);
                    const bool rest = fits && !fs;
                    if (ballot(rest)) {
                        const bool batch = rest && nw >= 2 && nw <= 64 && !(C.td && qn > 0);
                        if (rest && !batch) {
                            // the only waiting request, a queue longer than a wave or one
                            // whose next requests are cached: admit heads of line one at a
                            // time while they fit and are known
                            do {
                                admit_head(C, i, t);
                            } while (C.hols[i] >= 0 && C.hold[i] <= C.freeb[i]);
                            // an unknown head of line is found by the next round's rescan
                            any = any || C.hols[i] == kHolUnknown;
                        }
                        wave_sync();
                        for (unsigned long long m = ballot(batch); m; m &= m - 1) admit_batch<4>(C, ffs64(m), t, lane);
                    }
                    if (!ballot(any)) break;
                }
            }
            // auto-scaling signal (Section 3.6): the cluster average of the
            // normal-priority freeness F_normal = (free - head-of-line demand) /
            // max(B, 1) -- no headroom, no draining sentinel -- in fixed point,
            // floor(F_normal * 2^20) per instance, against -1/2 and 3/2
            double fsum = 0.0;
            // (the one-wave kernels hand each lane's instance on to the dispatch)
            int c_num = 0, c_hold = 0, c_nw = 0;
            double c_den = 1.0, c_rd = 1.0, c_fd = 0.0;
#pragma unroll
            for (int j = 0; j < OPL; ++j) {
                const uint32_t i = (uint32_t(lane) + 64u * j) * NW + uint32_t(wid);
                if (i >= I) continue;
                // every field first: one LDS round trip
                const int fr = C.freeb[i], hd = C.hold[i], tm = C.tmask[i], b = C.B[i], nw = C.nwait[i], he = C.held[i],
                          ib = C.inb[i];
                // Eq. 1-4 and the normal-priority freeness share the divisor
                const double den = double(b > 0 ? b : 1), rd = 1.0 / den;
                const int num = 256 * (fr - hd) - headroom_sum(C, tm);
                const double f = quot(double(num), den, rd);
                C.num[i] = num;
                C.fd[i] = f;
                c_num = num; c_hold = hd; c_nw = nw; c_den = den; c_rd = rd; c_fd = f;
                // slot-ticks: running and waiting requests at the end of the tick.
                // Later phases move running and waiting requests between
                // instances (commits, queued moves) and add only the arrivals
                // the dispatch places, counted there
                run_acc += unsigned(b);
                wait_acc += unsigned(nw);
                if (fr < 0 || fr + he + ib != int(C.M)) stat(C, kInvariant, 1);
                // floor(x 2^20 / den): x 2^20 is exact in a double (|x| < 2^22) and
                // the correctly rounded quotient never crosses an integer (the
                // quotient, below 2^42, sits at least 1/den >= 2^-11 from one, more
                // than half an ulp).  Sums of 256 such integers are exact.
                fsum += floor(quot(double(fr - hd) * 1048576.0, den, rd));
            }
            fsum = wsum_f64<(IM < 64 ? IM : 64)>(fsum);
            if (C.svc) {
                // INFaaS: service-time estimate from this tick's finishes, then
                // the state penalty (OVERLOADED before INTERFERED before ACTIVE)
#pragma unroll
                for (int j = 0; j < OPL; ++j) {
                    const uint32_t i = (uint32_t(lane) + 64u * j) * NW + uint32_t(wid);
                    if (i >= I) continue;
                    const int c = C.fcnt[i];
                    if (c > 0) {
                        // floor(256 sum / c): sum < 2^43, so 256 sum is exact in a
                        // double; the residual corrects the rounded quotient
                        const long long num = static_cast<long long>(C.fsum[i] * 256ull);
                        long long mean = static_cast<long long>(floor(double(num) / double(c)));
                        const long long rr = num - mean * c;
                        if (rr < 0) mean -= 1;
                        else if (rr >= c) mean += 1;
                        C.svc[i] += (mean - C.svc[i]) >> P.ewma_shift;  // arithmetic shift: floor
                    }
                    C.pen[i] = C.hols[i] >= 0 && C.hold[i] > C.freeb[i] ? int(P.pen_over)
                             : (C.flags[i] & kFlagIntf) ? int(P.pen_intf) : 0;
                }
            }
            if (NW > 1) {
                if (lane == 0)
                    atomicAdd(reinterpret_cast<unsigned long long*>(C.bsum),
                              static_cast<unsigned long long>(static_cast<long long>(fsum)));
                block_sync<NW>();
                fsum = double(*C.bsum);
            }
            if (tid == 0) {
                const double half = double(I) * 524288.0;
                if (fsum < -half) stat(C, kScaleOut, 1);
                else if (fsum > 3.0 * half) stat(C, kScaleIn, 1);
            }
            wave_sync();

            // the dispatch and the migrations (phases D and E): wave 0 (pairing:
            // whether it runs this tick and how many instances can pair)
            bool e2 = false;
            int nruns = 0;  // bursts' rests to place
            uint4* runs = reinterpret_cast<uint4*>(WIDE ? C.rsel - 64 * wid : nullptr);
            int n2 = 0, npairs = 0;
            if (wid == 0) {
            // the next tick's records: a read of 2K cycles on the sweep, whose
            // records fit no cache, waited for at the top of the tick (issued after
            // the dispatch: 1.5K of 16.8K cycles there, sweep 8.87 ms per 1000
            // ticks, here 8.64; ahead of the freeness phase, across which they cost
            // registers, 8.93).  Four waves, whose tick is longer, load them after it
            // (gauss10 with extensions 4.26 ms per 250 ticks, before it 4.34)
            auto load_next = [&] {
                if (tl + 1 >= nt) return;
                if (((tl + 1u) & 63u) == 0) {
                    const uint32_t* cn = uniform_ptr(cnts + tl + 1u);
                    cnt64 = tl + 1u + lane < nt ? cn[lane] : 0u;
                }
                const unsigned long long* rn = uniform_ptr(rec + P.arr_cap);
                a_nx = uint32_t(lane) < lim ? rn[lane] : 0ull;
            };
            if (NW == 1 || WIDE) load_next();

            // ===================== D: tier-ordered dispatch =====================
            // an instance with an empty queue now holds, after this dispatch, only
            // this tick's arrivals; they are recorded in LDS when they fit one wave
            // (frs is written with the dispatch's write-back, from the queue length before it)
            if (lane == 0) *C.lastn = 0;
            if (n == 0)
                for (uint32_t i = lane; i < I; i += 64) C.frs[i] = C.nwait[i] == 0;
            if (n > 0) {
                const unsigned seq0 = next_seq;
                next_seq += n;
                // per-instance dispatch state in registers: lane l, register j <-> instance 64 j + l
                // key: F of the instances that can take an arrival (minus infinity
                // for a full instance and, in the first mode, for a draining one)
                double key[IPL], fnew[IPL], den[IPL], rd[IPL];
                int live_r[IPL], nw_r[IPL], nadd[IPL], num_r[IPL], hold_r[IPL];
                bool head_r[IPL];  // its head of line is an arrival of this batch
                unsigned long long hk_r[IPL];
#pragma unroll
                for (int j = 0; j < IPL; ++j) {
                    const uint32_t i = lane + 64 * j;
                    nadd[j] = 0;
                    head_r[j] = false;
                    num_r[j] = 0;
                    hold_r[j] = 0;
                    nw_r[j] = 0;
                    fnew[j] = 0.0;
                    den[j] = 1.0;
                    rd[j] = 1.0;
                    live_r[j] = int(S); hk_r[j] = 0;
                    key[j] = -__builtin_inf();
                    if (i < I) {
                        const int h = C.hols[i], dr = C.drn[i];
                        live_r[j] = C.live[i];
                        hk_r[j] = C.holk[i];
                        double f;
                        if (NW == 1) {
                            num_r[j] = c_num; hold_r[j] = c_hold; nw_r[j] = c_nw; den[j] = c_den; rd[j] = c_rd; f = c_fd;
                        } else {
                            num_r[j] = C.num[i]; hold_r[j] = C.hold[i]; nw_r[j] = C.nwait[i];
                            const int b = C.B[i];
                            den[j] = double(b > 0 ? b : 1);
                            rd[j] = 1.0 / den[j];
                            f = C.fd[i];
                        }
                        if (h == kNoHol) hk_r[j] = kNone;
                        if (infaas) f = -infaas_cost(C, P, int(i), 0);
                        if (live_r[j] < int(S) && !dr) key[j] = f;
                    }
                }
                int cur = -1;
                bool full = false;
                bool drain_mode = false;  // every instance with room is draining (Section 3.4 fallback)
                int nfall = 0;
                // (a burst's records are loaded one batch of 64 ahead)
                unsigned long long a_bt = a0;
                for (uint32_t k0 = 0; k0 < n; k0 += 64) {
                    const uint32_t cn = n - k0 < 64 ? n - k0 : 64;
                    const unsigned long long a = a_bt;
                    if (n - k0 > 64) a_bt = k0 + 64 + lane < n ? rec[k0 + 64 + lane] : 0ull;
                    int tgt = -1, rank = 0;  // rank: among this batch's arrivals bound for tgt
                    unsigned long long heads = 0;  // arrivals of this batch that became a head of line
                    uint32_t k = 0;
                    while (k < cn && !full) {
                        if (cur < 0) {
                            // One arrival: what it would change on every instance is computed
                            // beside the argmax's chain -- whether it becomes the head of
                            // line there, and F then (Eq. 1-2: F moves by the change of
                            // head-of-line demand).  The step is straight-line code: a
                            // division after the argmax and the branches of a step shared
                            // with the runs below made it 1150 cycles of a lone wave.
                            const unsigned long long ak = rl64(a, int(k));
                            const unsigned long long hk = rank_of(C, uint32_t(ak >> 32) & 15u) << 32 | (seq0 + unsigned(ak >> 36));
                            const int dem = blocks_of(uint32_t(ak & 0xFFFFu), C.shift);
                            unsigned long long lower[IPL];
                            int nn[IPL];
                            double fn[IPL];
#pragma unroll
                            for (int j = 0; j < IPL; ++j) {
                                lower[j] = ballot(hk < hk_r[j]);
                                nn[j] = num_r[j] - 256 * (dem - hold_r[j]);
                                fn[j] = infaas ? 0.0 : quot(double(nn[j]), den[j], rd[j]);
                            }
                            double lb = key[0];
#pragma unroll
                            for (int j = 1; j < IPL; ++j) lb = fmax(lb, key[j]);
                            double mv = wave_max_f64<(IM < 64 ? IM : 64)>(lb);
                            if (__builtin_expect(mv == -__builtin_inf(), 0)) {
                                if (drain_mode) { full = true; break; }
                                // no non-draining instance has a free slot: the least
                                // loaded draining one (largest F without the sentinel);
                                // slots only fill up, so the mode holds for the tick
                                drain_mode = true;
#pragma unroll
                                for (int j = 0; j < IPL; ++j) {
                                    const uint32_t i = lane + 64 * j;
                                    key[j] = i < I && live_r[j] < int(S) && C.drn[i]
                                                 ? (infaas ? -infaas_cost(C, P, int(i), nadd[j]) : C.fd[i])
                                                 : -__builtin_inf();
                                }
                                lb = key[0];
#pragma unroll
                                for (int j = 1; j < IPL; ++j) lb = fmax(lb, key[j]);
                                mv = wave_max_f64<(IM < 64 ? IM : 64)>(lb);
                                if (mv == -__builtin_inf()) { full = true; break; }
                            }
                            if (INF && IPL == 1 && P.alpha256 > 0) {
                                // INFaaS: a placement raises its instance's cost by alpha
                                // whatever the arrival, so the instances less than alpha
                                // above the cheapest are all taken once, in (cost, index)
                                // order, before any is taken again: one round places as
                                // many arrivals as there are such instances.  (An argmax per
                                // arrival was 12.3K of the INFaaS sweep's 41K cycles a tick.)
                                const unsigned long long win = ballot(key[0] > mv - double(P.alpha256));
                                int rk = 0;
                                for (unsigned long long w = win; w; w &= w - 1) {
                                    const int l = ffs64(w);
                                    const double fl = __hiloint2double(rl(__double2hiint(key[0]), l), rl(__double2loint(key[0]), l));
                                    rk += (fl > key[0]) | ((fl == key[0]) & (l < lane)) ? 1 : 0;
                                }
                                const int m = min(int(cn - k), __popcll(win));
                                const bool pick = ((win >> lane) & 1ull) && rk < m;
                                const unsigned long long pm = ballot(pick);
                                // the instance of rank r goes to lane k + r, the others elsewhere
                                int dest = __popcll(~pm & lanemask_lt());
                                dest += dest < int(k) ? 0 : m;
                                dest = pick ? int(k) + rk : dest;
                                const int ti = __builtin_amdgcn_ds_permute(dest * 4, lane);
                                const int tn = __builtin_amdgcn_ds_permute(dest * 4, nadd[0]);
                                // and its arrival to the instance
                                const uint32_t alo = uint32_t(__builtin_amdgcn_ds_bpermute(dest * 4, int(uint32_t(a))));
                                const uint32_t ahi = uint32_t(__builtin_amdgcn_ds_bpermute(dest * 4, int(uint32_t(a >> 32))));
                                const unsigned long long hi = rank_of(C, ahi & 15u) << 32 | (seq0 + (ahi >> 4));
                                const bool hd = pick && hi < hk_r[0];
                                const unsigned long long hm = ballot(hd);
                                live_r[0] += pick ? 1 : 0;
                                nadd[0] += pick ? 1 : 0;
                                head_r[0] = head_r[0] || hd;
                                hk_r[0] = hd ? hi : hk_r[0];
                                hold_r[0] = hd ? blocks_of(alo & 0xFFFFu, C.shift) : hold_r[0];
                                key[0] = pick ? key[0] - double(P.alpha256) : key[0];
                                key[0] = pick && live_r[0] >= int(S) ? -__builtin_inf() : key[0];
                                const bool mine = lane >= int(k) && lane < int(k) + m;
                                if (mine) { tgt = ti; rank = tn; }
                                heads |= ballot(mine && ((hm >> (ti & 63)) & 1ull));
                                nfall += drain_mode ? m : 0;
                                k += uint32_t(m);
                                continue;
                            }
                            int jc = 0, lc = 0;
                            bool becomes = false;
#pragma unroll
                            for (int j = IPL - 1; j >= 0; --j) {
                                const unsigned long long bm = ballot(key[j] == mv);
                                if (IPL == 1 || bm) {
                                    jc = j;
                                    lc = ffs64(bm);
                                    becomes = (lower[j] >> lc) & 1ull;
                                }
                            }
                            // Arrival k goes to instance 64 jc + lc.  If it becomes its head of
                            // line, F changes and the argmax is taken again.  Otherwise F
                            // stays, and so does the argmax for the following arrivals, none
                            // of which can become the head of line (keys increase along the
                            // arrival order): they all go there until its slots run out.
                            // (under INFaaS every placement raises the cost by alpha)
                            if (becomes || (infaas && P.alpha256 > 0)) {
                                int na0 = 0;
#pragma unroll
                                for (int j = 0; j < IPL; ++j) {
                                    if (j != jc) continue;
                                    // (a new head of line is the instance's first arrival of the tick)
                                    if (infaas) na0 = rl(nadd[j], lc);
                                    const bool me = lane == lc, hd = me && becomes;
                                    live_r[j] += me ? 1 : 0;
                                    nadd[j] += me ? 1 : 0;
                                    head_r[j] = head_r[j] || hd;
                                    hk_r[j] = hd ? hk : hk_r[j];
                                    num_r[j] = hd ? nn[j] : num_r[j];
                                    hold_r[j] = hd ? dem : hold_r[j];
                                    if (infaas) {
                                        key[j] = me ? key[j] - double(P.alpha256) : key[j];
                                    } else {
                                        fnew[j] = hd ? fn[j] : fnew[j];
                                        key[j] = hd ? fn[j] : key[j];
                                    }
                                    key[j] = me && live_r[j] >= int(S) ? -__builtin_inf() : key[j];
                                }
                                heads |= static_cast<unsigned long long>(becomes) << k;
                                if (lane == int(k)) { tgt = 64 * jc + lc; rank = na0; }
                                nfall += drain_mode ? 1 : 0;
                                ++k;
                                continue;
                            }
                            cur = 64 * jc + lc;
                        }
                        // a run of arrivals that change nothing goes to cur
                        const int jc = IPL == 1 ? 0 : cur >> 6, lc = IPL == 1 ? cur : cur & 63;
                        int lv = 0, na0 = 0;
#pragma unroll
                        for (int j = 0; j < IPL; ++j)
                            if (j == jc) { lv = rl(live_r[j], lc); na0 = rl(nadd[j], lc); }
                        const int m = min(int(cn - k), int(S) - lv);
#pragma unroll
                        for (int j = 0; j < IPL; ++j) {
                            if (j != jc) continue;
                            const bool me = lane == lc;
                            live_r[j] += me ? m : 0;
                            nadd[j] += me ? m : 0;
                            key[j] = me && lv + m >= int(S) ? -__builtin_inf() : key[j];
                        }
                        if (lane >= int(k) && lane < int(k) + m) { tgt = cur; rank = na0 + lane - int(k); }
                        if (lv + m >= int(S)) cur = -1;
                        nfall += drain_mode ? m : 0;
                        k += uint32_t(m);
                    }
                    // write the dispatch state back for the slot assignment and later phases
                    bool qc_any = false;
#pragma unroll
                    for (int j = 0; j < IPL; ++j) {
                        const uint32_t i = lane + 64 * j;
                        if (i >= I) continue;
                        C.live[i] = live_r[j];
                        const int nw0 = nw_r[j];
                        if (k0 == 0) C.frs[i] = nw0 == 0 && n <= uint32_t(kLast);
                        nw_r[j] = nw0 + nadd[j];
                        C.nwait[i] = nw_r[j];
                        wait_acc += unsigned(nadd[j]);
                        if (head_r[j]) {
                            C.num[i] = num_r[j];
                            C.hold[i] = hold_r[j];
                            C.fd[i] = fnew[j];
                        }
                        if (C.ext && nadd[j] > 0) wlb(C)[i] = t < wlb(C)[i] ? t : wlb(C)[i];
                        if (C.td && nadd[j] > 0) {
                            // queue cache: an arrival that became the head of line pushes
                            // the old head to the front of the cache; the others enter it
                            // once their slots are known (an empty queue's arrivals are
                            // served by the list of this tick's placements)
                            const bool known = C.hols[i] >= 0, push = known && head_r[j];
                            if (push)
                                qc_insert_at(C, int(i), 0, qc_pack(C.holk[i], C.hols[i], C.hwd[i], C.hmt[i], C.hta[i]));
                            // (what is listed, after the push: it may drop the ring's last
                            // entry, or a full extension as a whole)
                            const bool all = nw0 + (push ? 1 : 0) == (known ? 1 + C.qn[i] + qx_count(C, int(i)) : 0);
                            const bool skip = !known && n <= uint32_t(kLast);
                            C.order[i] = skip ? kQcSkip : (all ? kQcAll : kQcPart) | (head_r[j] ? kQcHead : 0);
                            qc_any = qc_any || !skip;
                        }
                        nadd[j] = 0;
                        if (head_r[j]) C.holk[i] = hk_r[j];
                        head_r[j] = false;
                    }
                    wave_sync();
                    // slot assignment: the arrivals bound for one instance take its
                    // lowest empty slots in arrival order
                    const int tier = int((a >> 32) & 15u);
                    int s = -1;
                    bool searched = false;
                    const unsigned long long tgm = ballot(tgt >= 0);
                    if (W > 8 && W <= uint32_t(IM) && tgm) {
                        const int ft = rl(tgt, ffs64(tgm));
                        if (!ballot(tgt >= 0 && tgt != ft)) {
                            // the whole batch goes to one instance (a burst): the
                            // inclusive prefix of its free slots per occupancy word
                            // (gtmp, free during the dispatch), and each arrival's
                            // word by binary search
                            const unsigned long long wdl = uint32_t(lane) < W ? C.occ[ft * W + lane] : kNone;
                            const int pre = wscan(64 - __popcll(wdl), lane);
                            if (uint32_t(lane) < W) C.gtmp[lane] = pre;
                            wave_sync();
                            if (tgt >= 0) {
                                int lo = 0, hi = int(W) - 1;
                                while (lo < hi) {
                                    const int mid = (lo + hi) >> 1;
                                    if (C.gtmp[mid] > rank) hi = mid;
                                    else lo = mid + 1;
                                }
                                if (C.gtmp[lo] > rank) {
                                    const int before = lo ? C.gtmp[lo - 1] : 0;
                                    s = lo * 64 + kth_set_bit(~C.occ[ft * W + lo], rank - before);
                                }
                            }
                            searched = true;
                        }
                    }
                    if (tgt >= 0 && !searched) {
                        // the rank-th empty slot: its occupancy word, four words per
                        // step, then its place in that word (once for all lanes,
                        // wherever their words lie)
                        int rk = rank, wi = -1;
                        unsigned long long fw = 0;
                        for (uint32_t w0 = 0; w0 < W; w0 += 4) {
                            unsigned long long wd[4];
#pragma unroll
                            for (int k = 0; k < 4; ++k) wd[k] = w0 + k < W ? C.occ[tgt * W + w0 + k] : kNone;
                            // empty slots of the first one, two, three and four words
                            const int c0 = 64 - __popcll(wd[0]), c1 = c0 + 64 - __popcll(wd[1]),
                                      c2 = c1 + 64 - __popcll(wd[2]), c3 = c2 + 64 - __popcll(wd[3]);
                            if (rk >= c3) { rk -= c3; continue; }
                            const bool h = rk >= c1, q = rk >= (h ? c2 : c0);
                            const unsigned long long lo = h ? wd[2] : wd[0], hi = h ? wd[3] : wd[1];
                            fw = ~(q ? hi : lo);
                            rk -= h ? (q ? c2 : c1) : (q ? c0 : 0);
                            wi = int(w0) + (h ? 2 : 0) + (q ? 1 : 0);
                            break;
                        }
                        if (wi >= 0) s = wi * 64 + kth_set_bit(fw, rk);
                    }
                    if (tgt >= 0 && s < 0) {  // occupancy and live count disagree: flag, drop the arrival
                        stat(C, kInvariant, 1);
                        stat(C, tier * 8 + kRejected, 1);
                        if ((heads >> lane) & 1ull) C.hols[tgt] = kHolUnknown;
                        tgt = -2;
                    }
                    wave_sync();
                    if (n <= uint32_t(kLast)) {
                        const unsigned long long pm = ballot(tgt >= 0);
                        if (tgt >= 0) {
                            const int q = __popcll(pm & lanemask_lt());
                            C.lw[q] = kWaitW | (uint32_t((a >> 16) & 0xFFFFu) << 16) | uint32_t(a & 0xFFFFu);
                            C.lsl[q] = (uint32_t(tgt) << 16) | (uint32_t(tier) << 12) | uint32_t(s);
                            C.lsq[q] = seq0 + unsigned(a >> 36);
                        }
                        if (lane == 0) *C.lastn = __popcll(pm);
                    }
                    if (tgt >= 0) {
                        atomicOr(&C.occ[tgt * W + (s >> 6)], 1ull << (s & 63));
                        const size_t sb = size_t(tgt) * S + s;
                        const uint32_t word = kWaitW | (uint32_t((a >> 16) & 0xFFFFu) << 16) | uint32_t(a & 0xFFFFu);
                        const uint32_t meta = kWaiting | (unsigned(tier) << 2);
                        C.slot[sb] = make_uint4(word, meta, seq0 + unsigned(a >> 36), t);
                        if ((heads >> lane) & 1ull) {
                            C.hols[tgt] = s;
                            C.hwd[tgt] = word;
                            C.hmt[tgt] = meta;
                            C.hta[tgt] = t;
                        }
                    }
                    bool beyond = true;  // this lane's arrival is larger than every cached entry
                    if (C.td && ballot(qc_any)) {
                        // the arrivals behind a head of line enter its queue cache
                        wave_sync();
                        const uint32_t seq = seq0 + unsigned(a >> 36);
                        const int mode = tgt >= 0 ? C.order[tgt] : kQcSkip;
                        const int r = rank - ((mode & kQcHead) ? 1 : 0);  // among them; -1: the head of line
                        const unsigned long long key = arr_key(C, tier, seq);
                        const uint4 en = make_uint4(seq, kWaitW | (uint32_t((a >> 16) & 0xFFFFu) << 16) | uint32_t(a & 0xFFFFu),
                                                    t, uint32_t(s) | (uint32_t(tier) << 12));
                        const bool can = (mode & 3) != kQcSkip && r >= 0;
                        int nq = 0, xc = 0, xh = 0;
                        bool behind = true;  // larger than every cached entry
                        if (can) {
                            nq = C.qn[tgt];
                            if (C.xn) { const int xv = C.xn[tgt]; xc = xv & 0xFFFF; xh = xv >> 16; }
                            if (nq + xc > 0) {
                                const uint4 le = xc > 0 ? *qx_at(C, tgt, xh, xc - 1) : C.qt[qc_at(C, tgt, nq - 1)];
                                behind = key > qc_key(C, le);
                            }
                            // the first one behind a cache that lists the whole queue: all are
                            if (r == 0 && behind && (mode & 3) == kQcAll) C.order[tgt] = mode | kQcRun;
                        }
                        wave_sync();
                        const bool run = can && (C.order[tgt] & kQcRun);
                        if (run) {
                            // a run behind the cached entries, all at once (the ring fills
                            // before the extension starts)
                            if (xc == 0 && nq + r < C.td) {
                                C.qt[qc_at(C, tgt, nq + r)] = en;
                                atomicAdd(&C.qn[tgt], 1);
                            } else if (C.xn) {
                                const int k = xc > 0 ? xc + r : nq + r - C.td;
                                if (k < C.xd) {
                                    *qx_at(C, tgt, xh, k) = en;
                                    atomicAdd(&C.xn[tgt], 1);
                                }
                            }
                        }
                        beyond = behind;
                        // the others by a merge per instance
                        const unsigned long long inside = ballot(can && !run && !behind);
                        const bool enter = can && !run && (!behind || (xc == 0 && nq < C.td && (mode & 3) == kQcAll));
                        for (unsigned long long em = ballot(enter); em;) {
                            const int l = ffs64(em), ii = rl(tgt, l);
                            const unsigned long long mine = em & ballot(tgt == ii);
                            qc_merge(C, ii, mine, key, en, (rl(mode, l) & 3) == kQcAll, inside, lane);
                            em &= ~mine;
                        }
                    }
                    // every arrival is dispatched (tgt >= 0) or rejected: no free slot
                    // anywhere (-1), or dropped by the occupancy check (-2, counted
                    // above)
                    if (lane < int(cn)) stat(C, tier * 8 + kArrived, 1);
                    if (tgt >= 0) stat(C, tier * 8 + kDispatched, 1);
                    else if (tgt == -1 && lane < int(cn)) stat(C, tier * 8 + kRejected, 1);
                    wave_sync();
                    // The rest of a burst that goes on to the same instance is placed by
                    // all waves after this loop (place_run); here only the counts move
                    // on.  Its arrivals follow the kept queue order (append) or lie
                    // beyond it; else they take the batches above one by one.
                    if (WIDE && cur >= 0 && k0 + 64 < n && nruns < kMaxRuns) {
                        const int jc = cur >> 6, lc = cur & 63;
                        const bool append = C.td && (C.order[cur] & kQcRun);
                        if (!C.td || append || (ballot(beyond) >> 63)) {
                            int lv = 0;
#pragma unroll
                            for (int j = 0; j < IPL; ++j)
                                if (j == jc) lv = rl(live_r[j], lc);
                            const int m = min(int(n - k0 - 64), int(S) - lv);
                            if (lane == 0) {
                                runs[2 * nruns] = make_uint4(uint32_t(cur), k0 + 64u, uint32_t(m), seq0);
                                runs[2 * nruns + 1] = make_uint4(append ? 1u : 0u, append ? uint32_t(C.qn[cur]) : 0u, append ? uint32_t(C.xn[cur]) : 0u, 0u);
                                C.live[cur] += m;
                                C.nwait[cur] += m;
                            }
#pragma unroll
                            for (int j = 0; j < IPL; ++j) {
                                const bool me = j == jc && lane == lc;
                                live_r[j] += me ? m : 0;
                                nw_r[j] += me ? m : 0;
                                key[j] = me && live_r[j] >= int(S) ? -__builtin_inf() : key[j];
                            }
                            wait_acc += lane == 0 ? unsigned(m) : 0u;
                            nfall += drain_mode ? m : 0;
                            cur = -1;
                            ++nruns;
                            k0 += uint32_t(m);
                            if (k0 + 64 < n) a_bt = k0 + 64 + lane < n ? rec[k0 + 64 + lane] : 0ull;
                            wave_sync();
                        }
                    }
                }
                if (lane == 0 && nfall) stat(C, kDrainFallback, unsigned(nfall));
            }
            if (NW > 1 && !WIDE) load_next();
            if (WIDE && lane == 0) *C.kcnt = nruns;
            if (WIDE) wave_sync();
            }  // wave 0
            if constexpr (WIDE) {
                block_sync<NW>();
                nruns = *C.kcnt;
                for (int x = 0; x < nruns; ++x) place_run<NW>(C, rec, t, runs[2 * x], runs[2 * x + 1], lane, wid);
            }
            if (wid == 0) {
            // ===================== E1: staged copies =====================
            // a commit leaves the source slot and its wheel entry (without places,
            // source slot in gtmp and finish tick in order, searched after the loop)
            if (migs) {
            if (!C.td)
                for (uint32_t i = lane; i < I; i += 64) C.gtmp[i] = -1;
            for (uint32_t i = lane; i < I; i += 64) {
                int* m = &C.mig[4 * i];
                const int d = m[0];
                if (d < 0) continue;
                const size_t sb = size_t(i) * S + m[1], db = size_t(d) * S + m[2];
                const uint4 srec = C.slot[sb];
                const uint32_t v = srec.x;
                const uint32_t fin = fin_of(v, t);
                const int bl = blocks_of(wlo(v) - (fin - t), C.shift);
                int w = bl - m[3];
                if (w > int(P.mig_stage)) w = int(P.mig_stage);
                if (w > C.freeb[d]) {
                    C.freeb[d] += m[3];
                    C.inb[d] = 0;
                    s_word(C, db) = 0;
                    C.occ[d * W + (m[2] >> 6)] &= ~(1ull << (m[2] & 63));
                    C.live[d] -= 1;
                    s_meta(C, sb) = srec.y & ~kMigrating;
                    m[0] = -1; m[1] = 0; m[2] = 0; m[3] = 0;
                    stat(C, kMigAborted, 1);
                    set_f(C, d);
                    continue;
                }
                C.freeb[d] -= w;
                m[3] += w;
                C.inb[d] += w;
                if (m[3] == bl) {
                    const uint32_t mm = srec.y;
                    const int tier = int((mm >> 2) & 15u);
                    const int rr = int((wlo(v) - fin - 1u) & C.bmask);
                    const uint32_t place = wheel_put(C, fin, d, m[2]);
                    C.slot[db] = make_uint4(v, (mm & 0xFFu & ~(3u | kMigrating)) | kRunning | place, srec.z, srec.w);
                    if (C.td) {
                        wheel_erase(C, fin, mm);
                    } else {
                        C.gtmp[i] = m[1];
                        C.order[i] = int(fin);
                    }
                    s_word(C, sb) = 0;
                    C.occ[i * W + (m[1] >> 6)] &= ~(1ull << (m[1] & 63));
                    C.live[i] -= 1;
                    C.freeb[i] += bl;
                    C.held[i] -= bl;
                    C.held[d] += bl;
                    C.inb[d] = 0;
                    C.B[i] -= 1;
                    C.B[d] += 1;
                    c16_dec(C.res, res_idx(C, i, rr));
                    c16_inc(C.res, res_idx(C, d, rr));
                    tier_dec(C, int(i), tier);
                    tier_inc(C, d, tier);
                    m[0] = -1; m[1] = 0; m[2] = 0; m[3] = 0;
                    stat(C, kMigCommitted, 1);
                    set_f(C, int(i));
                }
                set_f(C, d);
            }
            wave_sync();
            if (!C.td) {
#pragma unroll
                for (int j = 0; j < IPL; ++j) {
                    const uint32_t i0 = lane + 64 * j;
                    for (unsigned long long m = ballot(i0 < I && C.gtmp[i0] >= 0); m; m &= m - 1) {
                        const int ii = 64 * j + ffs64(m);
                        wheel_erase_search(C, uint32_t(C.order[ii]), ii, C.gtmp[ii], lane);
                    }
                }
                wave_sync();
            }
            bool live = false;
            for (uint32_t i = lane; i < I; i += 64) live = live || C.mig[4 * i] >= 0;
            migs = ballot(live) != 0;
            }

            // ===================== E2: pairing on interval ticks =====================
            const bool mig_tick = mig_left == 0;
            mig_left = mig_tick ? P.mig_interval - 1u : mig_left - 1u;
            // pairing in three parts: which instances can pair and their keys
            // (wave 0), their order (wave 0 by counting ranks; in the kernels for
            // more than 64 instances only as many of the lowest and highest as can pair,
            // or the whole order by every thread), the pairs (wave 0, the staged
            // copies' candidates by all waves)
            npairs = 0;
            bool sort = false;
            if (!infaas && mig_tick) {
                // F and the draining flag of each lane's instances
                // A round moves something only if an instance with F < 0 (or a
                // draining one) holds a request and one that isn't draining has a
                // free slot.  (Drained clusters wait empty for their removal, and
                // an overloaded cluster's slots are full after most dispatches:
                // ordering and testing the pairs all the same took 7.6K of the
                // draining sweep's 21.9K cycles a tick.)
                double ef[IPL];
                bool ng[IPL];
                bool neg = false, room = false;
#pragma unroll
                for (int j = 0; j < IPL; ++j) {
                    const uint32_t i = lane + 64 * j;
                    ef[j] = 0.0;
                    ng[j] = false;
                    if (i < I) {
                        const double f = C.fd[i];
                        const int dr = C.drn[i], held = C.B[i] + C.nwait[i], lv = C.live[i];
                        ef[j] = dr ? -__builtin_inf() : f;
                        ng[j] = dr || f < 0.0;
                        neg = neg || (ng[j] && held > 0);
                        room = room || (!dr && lv < int(S));
                    }
                }
                if (ballot(neg) && ballot(room)) {
                    e2 = true;
                    // the instances not in a migration (no record is active: all)
                    unsigned long long avm[IPL];
                    if (migs) {
                        for (uint32_t i = lane; i < I; i += 64) C.flags[i] &= ~kFlagBusy;
                        wave_sync();
                        for (uint32_t i = lane; i < I; i += 64) {
                            const int d = C.mig[4 * i];
                            if (d >= 0) { atomicOr(&C.flags[i], kFlagBusy); atomicOr(&C.flags[d], kFlagBusy); }
                        }
                        wave_sync();
                    }
#pragma unroll
                    for (int j = 0; j < IPL; ++j) {
                        const uint32_t i = lane + 64 * j;
                        avm[j] = ballot(i < I && !(migs && (C.flags[i] & kFlagBusy)));
                        n2 += __popcll(avm[j]);
                        npairs += __popcll(avm[j] & ballot(ng[j]));
                    }
                    // a source past those with F < 0 (or draining) ends the round
                    npairs = min(min(int(P.mig_max_pairs), n2 / 2), npairs);
                    if (WIDE && npairs <= kPickPairs) {
                        // L's first and last npairs entries: the smallest and the
                        // largest (F, index) left, one pair after the other
                        double lo[IPL], hi[IPL];
#pragma unroll
                        for (int j = 0; j < IPL; ++j) {
                            const bool av = (avm[j] >> lane) & 1ull;
                            lo[j] = av ? -ef[j] : -__builtin_inf();
                            hi[j] = av ? ef[j] : -__builtin_inf();
                            // a draining instance comes first: -ef is plus infinity
                        }
                        for (int k = 0; k < npairs; ++k) {
                            double a = lo[0], b = hi[0];
#pragma unroll
                            for (int j = 1; j < IPL; ++j) { a = fmax(a, lo[j]); b = fmax(b, hi[j]); }
                            a = wave_max_f64<64>(a);
                            b = wave_max_f64<64>(b);
                            // only draining instances are left as destinations: the round ends
                            if (b == -__builtin_inf()) { npairs = k; break; }
                            int is = 0, id = 0;
#pragma unroll
                            for (int j = IPL - 1; j >= 0; --j) {
                                const unsigned long long m = ballot(lo[j] == a);
                                if (m) is = 64 * j + ffs64(m);
                            }
#pragma unroll
                            for (int j = 0; j < IPL; ++j) {
                                const unsigned long long m = ballot(hi[j] == b);
                                if (m) id = 64 * j + 63 - __clzll(static_cast<long long>(m));
                            }
#pragma unroll
                            for (int j = 0; j < IPL; ++j) {
                                const int i = lane + 64 * j;
                                lo[j] = i == is ? -__builtin_inf() : lo[j];
                                hi[j] = i == id ? -__builtin_inf() : hi[j];
                            }
                            if (lane == 0) { C.order[k] = is; C.order[n2 - 1 - k] = id; }
                        }
                    } else if (WIDE) {
                        sort = true;
                        // the keys for the workgroup's count, in the freeness array
                        // (set again in phase C before its next use): F as an
                        // order-preserving 64-bit key; an instance in a migration
                        // carries the largest one
#pragma unroll
                        for (int j = 0; j < IPL; ++j) {
                            const uint32_t i = lane + 64 * j;
                            const unsigned long long bits = static_cast<unsigned long long>(__double_as_longlong(ef[j]));
                            const unsigned long long fk = (bits >> 63) ? ~bits : bits | (1ull << 63);
                            if (i < I)
                                reinterpret_cast<unsigned long long*>(C.fd)[i] = (avm[j] >> lane) & 1ull ? fk : kNone;
                        }
                    } else {
                        // L: every instance's rank by (F, index), from every other
                        // lane's F (the lanes above it also count an equal one)
                        int rk = 0;
                        for (unsigned long long mm = avm[0]; mm; mm &= mm - 1) {
                            const int l = ffs64(mm);
                            const double fl = __hiloint2double(rl(__double2hiint(ef[0]), l), rl(__double2loint(ef[0]), l));
                            rk += (fl < ef[0]) | ((fl == ef[0]) & (l < lane)) ? 1 : 0;
                        }
                        if ((avm[0] >> lane) & 1ull) C.order[rk] = lane;
                    }
                }
            }
            if (WIDE && lane == 0) *C.e2go = sort ? 1 : 0;
            wave_sync();
            }  // wave 0
            if (WIDE) block_sync<NW>();
            if (WIDE && *C.e2go) {
                // L in the eight-wave kernels: each instance's rank in (F, index)
                // order, in two steps: waves 0..3 each sort a block of 64
                // instances by counting (into the rescans' selection buffers,
                // free at this point of the tick), then every instance adds its
                // place in each block, found by bisection, summed in gtmp[]
                const unsigned long long* key = reinterpret_cast<const unsigned long long*>(C.fd);
                constexpr uint32_t kParts = NT / uint32_t(IM);
                const uint32_t nblk = (I + 63u) / 64u;
                ulonglong2* sblk = reinterpret_cast<ulonglong2*>(C.rsel - 64 * wid);
                for (uint32_t i = tid; i < I; i += NT) C.gtmp[i] = 0;
                if (uint32_t(wid) < nblk) {
                    // (entries past I and unavailable instances carry the largest key)
                    const uint32_t i = 64u * uint32_t(wid) + uint32_t(lane);
                    const unsigned long long kb = i < I ? key[i] : kNone;
                    int r0 = 0, r1 = 0, r2 = 0, r3 = 0;
                    for (int j = 0; j < 64; j += 4) {
                        const unsigned long long k0 = rl64(kb, j), k1 = rl64(kb, j + 1), k2 = rl64(kb, j + 2),
                                                 k3 = rl64(kb, j + 3);
                        r0 += int((k0 < kb) | ((k0 == kb) & (j < lane)));
                        r1 += int((k1 < kb) | ((k1 == kb) & (j + 1 < lane)));
                        r2 += int((k2 < kb) | ((k2 == kb) & (j + 2 < lane)));
                        r3 += int((k3 < kb) | ((k3 == kb) & (j + 3 < lane)));
                    }
                    sblk[64 * wid + r0 + r1 + r2 + r3] = make_ulonglong2(kb, i);
                }
                block_sync<NW>();
                {
                    const uint32_t i = tid % uint32_t(IM);
                    const uint32_t part = uint32_t(__builtin_amdgcn_readfirstlane(int(tid / uint32_t(IM))));
                    const unsigned long long ki = i < I ? key[i] : kNone;
                    if (ki != kNone) {
                        int rk = 0;
                        for (uint32_t bk = part; bk < nblk; bk += kParts) {
                            // entries of block bk below (ki, i)
                            int lo = 0, hi = 64;
                            while (lo < hi) {
                                const int mid = (lo + hi) >> 1;
                                const ulonglong2 e = sblk[64 * bk + mid];
                                if (e.x < ki || (e.x == ki && e.y < i)) lo = mid + 1;
                                else hi = mid;
                            }
                            rk += lo;
                        }
                        if (rk) atomicAdd(&C.gtmp[i], rk);
                    }
                }
                block_sync<NW>();
                for (uint32_t i = tid; i < I; i += NT)
                    if (key[i] != kNone) C.order[C.gtmp[i]] = int(i);
                block_sync<NW>();
            }
            if (wid == 0) {
                int nst = 0;  // staged copies to start
                if (e2) {
                    // Pairs (L[k], L[n2 - 1 - k]) use disjoint instances and one
                    // snapshot of F, so the stopping pair is found for all pairs at
                    // once (lane k tests pair k), the queued moves of the pairs
                    // before it run in parallel, and so do the staged copies once
                    // every wave has scanned its part of the sources' slots.
                    for (int k0 = 0; k0 < npairs; k0 += 64) {
                        const int k = k0 + lane;
                        const bool in = k < npairs;
                        const int src = in ? C.order[k] : 0, dst = in ? C.order[n2 - 1 - k] : 0;
                        bool stop = false;
                        if (in) {
                            if (C.drn[dst]) {
                                // a draining destination: every instance left is draining
                                stop = true;
                            } else if (!C.drn[src]) {
                                // (a draining source is overloaded and any destination is
                                // more than theta freer)
                                const int bs = C.B[src], bd = C.B[dst], ns = C.num[src], nd = C.num[dst];
                                const long long es = bs > 0 ? bs : 1, ed = bd > 0 ? bd : 1;
                                const long long lhs = (long long)P.theta_den * (nd * es - ns * ed);
                                const long long rhs = (long long)P.theta_num * 256 * es * ed;
                                stop = ns >= 0 || lhs < rhs;
                            }
                        }
                        const unsigned long long sm = ballot(stop);
                        const int kstop = sm ? ffs64(sm) : 64;
                        // the destination's lowest empty slot; a full one skips its pair
                        int ds = -1;
                        if (in && lane < kstop && C.live[dst] < int(S)) {
                            for (uint32_t w = 0; w < W; ++w) {
                                const unsigned long long word = C.occ[dst * W + w];
                                if (word != kNone) { ds = int(w) * 64 + ffs64(~word); break; }
                            }
                        }
                        const bool act = ds >= 0;
                        const int h = act ? C.hols[src] : kNoHol;
                        bool deep = false;
                        uint4 dq = make_uint4(0u, 0u, 0u, 0u);
                        if (act && h >= 0) {
                            // queued move of the source's head of line (fields cached in LDS)
                            const size_t dsb = size_t(dst) * S + ds, hb = size_t(src) * S + h;
                            const uint32_t hw = C.hwd[src], hm = C.hmt[src], ht = C.hta[src];
                            const unsigned long long key = C.holk[src];
                            C.slot[dsb] = make_uint4(hw, hm, uint32_t(key), ht);
                            s_word(C, hb) = 0;
                            C.occ[src * W + (h >> 6)] &= ~(1ull << (h & 63));
                            C.occ[dst * W + (ds >> 6)] |= 1ull << (ds & 63);
                            C.live[src] -= 1; C.nwait[src] -= 1;
                            C.live[dst] += 1; C.nwait[dst] += 1;
                            C.frs[src] = 0; C.frs[dst] = 0;
                            deep = hol_insert(C, dst, key, ds, hw, hm, ht);
                            if (C.xn) dq = qc_pack(key, ds, hw, hm, ht);
                            hol_pop(C, src);
                            stat(C, kMigQueued, 1);
                            if (C.ext) wlb(C)[dst] = ht < wlb(C)[dst] ? ht : wlb(C)[dst];
                        }
                        wave_sync();
                        if (C.xn) {
                            for (unsigned long long dm = ballot(deep); dm; dm &= dm - 1) {
                                const int l = ffs64(dm);
                                qx_insert(C, rl(dst, l), make_uint4(rlu(dq.x, l), rlu(dq.y, l), rlu(dq.z, l), rlu(dq.w, l)), lane);
                            }
                        }
                        const unsigned long long pm = ballot(act && h < 0);
                        if constexpr (NW > 1) {
                            // staged copies are listed: source, destination, its slot
                            if (act && h < 0) {
                                const int x = nst + __popcll(pm & lanemask_lt());
                                C.gtmp[x] = src | (dst << 8) | (ds << 16);
                                reinterpret_cast<unsigned long long*>(C.fd)[x] = 0ull;
                            }
                            nst += __popcll(pm);
                        } else {
                            for (unsigned long long w = pm; w; w &= w - 1) {
                                const int l = ffs64(w);
                                const int psrc = rl(src, l);
                                const unsigned long long mx = staged_best<1>(C, psrc, t, lane, 0);
                                if (mx == 0) continue;
                                const int pdst = rl(dst, l), pds = rl(ds, l);
                                if (lane == 0) staged_start(C, psrc, pdst, pds, mx);
                                migs = true;
                                wave_sync();
                            }
                        }
                        if (sm) break;
                    }
                }
                if (NW > 1) {
                    if (lane == 0) *C.e2n2 = nst;
                    migs = migs || nst > 0;
                }
                wave_sync();
            }
            if constexpr (NW > 1) {
                block_sync<NW>();
                const int nstaged = *C.e2n2;
                if (nstaged) {
                    unsigned long long* best = reinterpret_cast<unsigned long long*>(C.fd);
                    for (int x = 0; x < nstaged; ++x) {
                        const unsigned long long mx = staged_best<NW>(C, C.gtmp[x] & 0xFF, t, lane, wid);
                        if (lane == 0 && mx) atomicMax(&best[x], mx);
                    }
                    block_sync<NW>();
                    if (wid == 0) {
                        for (int x = lane; x < nstaged; x += 64) {
                            const int e = C.gtmp[x];
                            if (best[x]) staged_start(C, e & 0xFF, (e >> 8) & 0xFF, e >> 16, best[x]);
                        }
                        wave_sync();
                    }
                }
            }
            block_sync<NW>();
        }

        // ---------------- epilogue ----------------
        const unsigned long long run_sum = wsum64(run_acc), wait_sum = wsum64(wait_acc);
        if (lane == 0) {
            stat(C, kRunSlotTicks, run_sum);
            stat(C, kWaitSlotTicks, wait_sum);
            if (wid == 0) stat(C, kTicks, nt);
        }
        block_sync<NW>();
        for (uint32_t j = tid; j < uint32_t(kNstat); j += NT) P.stats[size_t(r) * kNstat + j] = C.stats[j];
        for (uint32_t i = tid; i < I; i += NT) {
            P.freeb[size_t(r) * I + i] = C.freeb[i];
            if (C.svc) P.svc[size_t(r) * I + i] = C.svc[i];
            for (int k = 0; k < 4; ++k) P.mig[(size_t(r) * I + i) * 4 + k] = C.mig[4 * i + k];
        }
        if (tid == 0) P.next_seq[r] = next_seq;
        image_write<NT>(P, r, t0u + nt, lds_raw, tid);
        block_sync<NW>();
    }
}

}  // namespace

// The instantiations of the step kernel are compiled in twelve translation
// units (this file with MTS_STEP_PART = 0..11): bit 0 the INFaaS policy, bit 1
// the Section 6.5 extensions; 0..3 the one-wave kernels, 4..7 those for more
// than 64 instances, 8..11 the four-wave kernels (always with a queue cache).
// Each gives the kernel for IM instances with (qc) or without a queue cache.
#ifdef MTS_STEP_PART
#define MTS_STEP_FN2(p) step_part_##p
#define MTS_STEP_FN(p) MTS_STEP_FN2(p)
namespace {
template <bool QC>
const void* step_of(uint32_t IM)
{
    constexpr bool INF = (MTS_STEP_PART & 1) != 0, EXT = (MTS_STEP_PART & 2) != 0;
#if MTS_STEP_PART & 4
    return IM == 128 ? reinterpret_cast<const void*>(&k_step<128, INF, EXT, QC, 8>)
                     : reinterpret_cast<const void*>(&k_step<256, INF, EXT, QC, 8>);
#else
    constexpr int NW = MTS_STEP_PART & 8 ? 4 : 1;
    return IM == 16   ? reinterpret_cast<const void*>(&k_step<16, INF, EXT, QC, NW>)
           : IM == 32 ? reinterpret_cast<const void*>(&k_step<32, INF, EXT, QC, NW>)
                      : reinterpret_cast<const void*>(&k_step<64, INF, EXT, QC, NW>);
#endif
}
}  // namespace
#if MTS_STEP_PART & 8
const void* MTS_STEP_FN(MTS_STEP_PART)(uint32_t IM, bool) { return step_of<true>(IM); }
#else
const void* MTS_STEP_FN(MTS_STEP_PART)(uint32_t IM, bool qc) { return qc ? step_of<true>(IM) : step_of<false>(IM); }
#endif

#else

const void* step_part_0(uint32_t, bool);
const void* step_part_1(uint32_t, bool);
const void* step_part_2(uint32_t, bool);
const void* step_part_3(uint32_t, bool);
const void* step_part_4(uint32_t, bool);
const void* step_part_5(uint32_t, bool);
const void* step_part_6(uint32_t, bool);
const void* step_part_7(uint32_t, bool);
const void* step_part_8(uint32_t, bool);
const void* step_part_9(uint32_t, bool);
const void* step_part_10(uint32_t, bool);
const void* step_part_11(uint32_t, bool);

namespace {

// ---------------------------------------------------------------------------
// initial state: every slot empty, free = M, no migrations, zero counters
// ---------------------------------------------------------------------------
__global__ void k_init(Params P)
{
    const size_t nslots = size_t(P.R) * P.I * P.S;
    const size_t stride = size_t(gridDim.x) * blockDim.x;
    const size_t t0 = size_t(blockIdx.x) * blockDim.x + threadIdx.x;
    for (size_t s = t0; s < nslots; s += stride) P.slot[s] = make_uint4(0u, 0u, 0u, 0u);
    for (size_t j = t0; j < size_t(P.R) * P.I; j += stride) {
        P.freeb[j] = int32_t(P.M);
        P.mig[4 * j] = -1; P.mig[4 * j + 1] = 0; P.mig[4 * j + 2] = 0; P.mig[4 * j + 3] = 0;
        P.drain[j] = 0;
    }
    for (size_t j = t0; j < size_t(P.R) * kHistPerReplica; j += stride) P.hist[j] = 0;
    for (size_t j = t0; j < size_t(P.R) * P.I; j += stride) P.svc[j] = 0;
    for (size_t j = t0; j < size_t(P.R) * kNstat; j += stride) P.stats[j] = 0;
    for (size_t j = t0; j < P.R; j += stride) {
        P.next_seq[j] = 0;
        P.digest[j] = 0;
        if (j < P.img_r) P.img[j * P.img_n] = make_uint4(0u, 0u, 0u, 0u);
    }
    if (P.hsnap)
        for (size_t j = t0; j < size_t(P.R) * 2 * kTiers; j += stride) P.hsnap[j] = 0;
}

// ---------------------------------------------------------------------------
// moving the clock by delta ticks keeps every running request's remaining
// output: its finish tick moves by the same delta
// ---------------------------------------------------------------------------
__global__ void k_shift_clock(Params P, uint32_t delta)
{
    for (size_t j = size_t(blockIdx.x) * blockDim.x + threadIdx.x; j < P.img_r; j += size_t(gridDim.x) * blockDim.x)
        P.img[j * P.img_n] = make_uint4(0u, 0u, 0u, 0u);
    const size_t nslots = size_t(P.R) * P.I * P.S;
    const size_t stride = size_t(gridDim.x) * blockDim.x;
    for (size_t s = size_t(blockIdx.x) * blockDim.x + threadIdx.x; s < nslots; s += stride) {
        uint32_t* w = reinterpret_cast<uint32_t*>(P.slot + s);
        const uint32_t v = *w;
        if (wst(v) == 2u) *w = (v & ~(kFin << 16)) | (((wmid(v) + delta) & kFin) << 16);
    }
}

// ---------------------------------------------------------------------------
// per-replica digest of the canonical state at tick `tick` (the next tick to
// run): wrapping sum of SplitMix64-finalised slot and instance records
// (Steele, Lea, Flood, OOPSLA 2014); one block per replica
// ---------------------------------------------------------------------------
__device__ inline unsigned long long mix64(unsigned long long z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ __launch_bounds__(256) void k_digest(Params P, uint32_t r0, uint32_t tick)
{
    __shared__ unsigned long long part[4];
    const uint32_t r = r0 + blockIdx.x;
    const size_t IS = size_t(P.I) * P.S;
    const size_t rb = size_t(r) * IS;
    const unsigned long long gm = mix64(P.id_base + r);
    unsigned long long d = 0;
    for (size_t s = threadIdx.x; s < IS; s += blockDim.x) {
        // an empty slot has a zero word; an inbound reservation's seq and
        // arrival tick are zero in the canonical state (the device leaves them)
        const uint4 rec = P.slot[rb + s];
        const uint32_t hw = rec.x;
        if (hw == 0u) continue;
        const bool inb = wst(hw) == kInbound;
        const unsigned m = rec.y & 0xFFu;
        const unsigned long long a = static_cast<unsigned long long>(slot_lr(hw, tick)) |
                                     (static_cast<unsigned long long>(inb ? 0u : rec.z) << 32);
        const unsigned long long b = static_cast<unsigned long long>(inb ? 0u : rec.w) |
                                     (static_cast<unsigned long long>(m) << 32);
        const unsigned long long p = mix64(gm + 2ull * s + 1ull);
        d += mix64(p ^ a) + mix64(p ^ b);
    }
    for (uint32_t i = threadIdx.x; i < P.I; i += blockDim.x) {
        const int32_t* m = P.mig + (size_t(r) * P.I + i) * 4;
        const unsigned long long p = mix64(gm + 2ull * (IS + i) + 1ull);
        const unsigned long long c = static_cast<unsigned long long>(uint32_t(P.freeb[size_t(r) * P.I + i])) |
                                     (static_cast<unsigned long long>(uint32_t(m[0])) << 32);
        const unsigned long long e = static_cast<unsigned long long>(uint32_t(m[1])) |
                                     (static_cast<unsigned long long>(uint32_t(m[2])) << 32);
        const unsigned long long f = static_cast<unsigned long long>(uint32_t(m[3])) |
                                     (static_cast<unsigned long long>(P.drain[size_t(r) * P.I + i]) << 32);
        d += mix64(p ^ c) + mix64(p ^ e) + mix64(p ^ f);
    }
    for (int o = 32; o > 0; o >>= 1) d += __shfl_xor(d, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = d;
    __syncthreads();
    if (threadIdx.x == 0) P.digest[r] = part[0] + part[1] + part[2] + part[3];
}

}  // namespace

size_t lds_bytes(uint32_t I, uint32_t S, uint32_t RB, uint32_t wsz, uint32_t policy, uint32_t qdepth, bool ext, uint32_t nw)
{
    return lds_layout(imax_for(I), I, S / 64, RB, wsz, policy, qdepth, ext, nw).total;
}

int launch_init(const Params& p, hipStream_t stream)
{
    hipLaunchKernelGGL(k_init, dim3(1024), dim3(256), 0, stream, p);
    return int(hipGetLastError());
}


namespace {

// the kernels with the adaptive-headroom / promotion code are separate
// instantiations, so that the others carry none of its registers
bool ext_on(const Params& p) { return p.adapt_epoch != 0 || p.promo_period != 0; }

const void* step_fn(const Params& p)
{
    using Part = const void* (*)(uint32_t, bool);
    static constexpr Part parts[12] = {step_part_0, step_part_1, step_part_2,  step_part_3,
                                       step_part_4, step_part_5, step_part_6,  step_part_7,
                                       step_part_8, step_part_9, step_part_10, step_part_11};
    const uint32_t IM = imax_for(p.I);
    const int k = (p.policy == MTS_POLICY_INFAAS ? 1 : 0) | (ext_on(p) ? 2 : 0) | (IM >= 128 ? 4 : p.nw > 1 ? 8 : 0);
    return parts[k](IM, p.qdepth != 0);
}

size_t step_lds(const Params& p)
{
    const size_t lds = lds_bytes(p.I, p.S, p.RB, p.wsz, p.policy, p.qdepth, ext_on(p), p.nw);
    if (lds > 64 * 1024) {
        // raise the dynamic LDS limit; a real failure shows up at the launch
        (void)hipFuncSetAttribute(step_fn(p), hipFuncAttributeMaxDynamicSharedMemorySize, int(lds));
        (void)hipGetLastError();
    }
    return lds;
}

}  // namespace

int step_threads(const Params& p) { return int(64 * p.nw); }

int step_blocks_per_cu(const Params& p)
{
    const size_t lds = step_lds(p);
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, step_fn(p), step_threads(p), lds) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    return nb;
}

int launch_step(const Params& p, unsigned long long t0, uint32_t nt, uint32_t blocks, hipStream_t stream)
{
    const size_t lds = step_lds(p);
    Params q = p;
    q.img_lds = uint32_t(lds);
    if (lds + 16 > size_t(p.img_n) * 16) q.img_r = 0;  // a depth the image has no room for
    void* args[] = {&q, &t0, &nt};
    const hipError_t rc = hipLaunchKernel(step_fn(p), dim3(blocks), dim3(uint32_t(step_threads(p))), args, lds, stream);
    if (rc != hipSuccess) { (void)hipGetLastError(); return int(rc); }
    return int(hipGetLastError());
}

int launch_shift_clock(const Params& p, uint32_t delta, hipStream_t stream)
{
    hipLaunchKernelGGL(k_shift_clock, dim3(1024), dim3(256), 0, stream, p, delta);
    return int(hipGetLastError());
}

// ---------------------------------------------------------------------------
// slot records to the canonical arrays of mts_export_state and back: f0 and
// f the handle's flat slot index.  Streaming passes of 16 + 13 bytes per slot;
// the host's loops over the same slots took most of a checkpoint's time.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_pack(Params P, size_t f0, uint32_t n, uint32_t tick, uint8_t* meta, uint32_t* lr,
                                              uint32_t* seq, uint32_t* tarr)
{
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += stride) {
        const uint4 rec = P.slot[f0 + j];
        const uint32_t w = rec.x;
        const bool gone = slot_gone(w);
        if (lr) lr[j] = slot_lr(w, tick);
        if (meta) meta[j] = w == 0 ? 0 : uint8_t(rec.y);
        if (seq) seq[j] = gone ? 0 : rec.z;
        if (tarr) tarr[j] = gone ? 0 : rec.w;
    }
}

// sets *bad when a slot is not acceptable (slot_ok)
__global__ __launch_bounds__(256) void k_check_slots(Params P, size_t f0, uint32_t n, const uint8_t* meta, const uint32_t* lr,
                                                     uint32_t* bad)
{
    const uint32_t IS = P.I * P.S, stride = gridDim.x * blockDim.x;
    bool b = false;
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += stride) {
        const uint32_t m = meta[j];
        const uint32_t K = m ? P.group_K32[P.group_of[(f0 + j) / IS]] : 0u;
        b = b || !slot_ok(m, lr[j], K);
    }
    if (b) atomicOr(bad, 1u);
}

// running requests are re-encoded relative to tick
__global__ __launch_bounds__(256) void k_unpack(Params P, size_t f0, uint32_t n, uint32_t tick, const uint8_t* meta,
                                                const uint32_t* lr, const uint32_t* seq, const uint32_t* tarr)
{
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t j = blockIdx.x * blockDim.x + threadIdx.x; j < n; j += stride) {
        const uint32_t m = meta[j];
        P.slot[f0 + j] = make_uint4(slot_word(m, lr[j], tick), m, seq[j], tarr[j]);
    }
}

namespace {
dim3 slot_grid(uint32_t n) { return dim3((n + 1023) / 1024 < 2048 ? (n + 1023) / 1024 : 2048); }
}  // namespace

int launch_pack(const Params& p, size_t f0, uint32_t n, uint32_t tick, uint8_t* meta, uint32_t* lr, uint32_t* seq,
                uint32_t* tarr, hipStream_t stream)
{
    if (n == 0) return 0;
    hipLaunchKernelGGL(k_pack, slot_grid(n), dim3(256), 0, stream, p, f0, n, tick, meta, lr, seq, tarr);
    return int(hipGetLastError());
}
int launch_check_slots(const Params& p, size_t f0, uint32_t n, const uint8_t* meta, const uint32_t* lr, uint32_t* bad,
                       hipStream_t stream)
{
    if (n == 0) return 0;
    hipLaunchKernelGGL(k_check_slots, slot_grid(n), dim3(256), 0, stream, p, f0, n, meta, lr, bad);
    return int(hipGetLastError());
}
int launch_unpack(const Params& p, size_t f0, uint32_t n, uint32_t tick, const uint8_t* meta, const uint32_t* lr,
                  const uint32_t* seq, const uint32_t* tarr, hipStream_t stream)
{
    if (n == 0) return 0;
    hipLaunchKernelGGL(k_unpack, slot_grid(n), dim3(256), 0, stream, p, f0, n, tick, meta, lr, seq, tarr);
    return int(hipGetLastError());
}

// voids the images of replicas [r0, r0 + nr)
__global__ void k_void_images(Params P, uint32_t r0, uint32_t nr)
{
    const uint32_t j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < nr && r0 + j < P.img_r) P.img[size_t(r0 + j) * P.img_n] = make_uint4(0u, 0u, 0u, 0u);
}

int launch_void_images(const Params& p, uint32_t r0, uint32_t nr, hipStream_t stream)
{
    if (r0 >= p.img_r || nr == 0) return 0;
    hipLaunchKernelGGL(k_void_images, dim3((nr + 255) / 256), dim3(256), 0, stream, p, r0, nr);
    return int(hipGetLastError());
}

int launch_digest(const Params& p, uint32_t r0, uint32_t nr, uint32_t tick, hipStream_t stream)
{
    if (nr == 0) return 0;
    hipLaunchKernelGGL(k_digest, dim3(nr), dim3(256), 0, stream, p, r0, tick);
    return int(hipGetLastError());
}

#endif  // MTS_STEP_PART

}  // namespace mts
