// The channel kernel: one or more workgroups decode an utterance, frame after frame, on the device.
// Included by wfst_decoder.hip inside its anonymous namespace.
//
// A "cluster" of G workgroups (1, 2, 4 or 8) owns a channel.  The token keys are shared out among
// them by the top bits of the key's hash: the owner of a key recombines everything that arrives
// there, keeps the token, and expands it.  Per frame:
//
//   expand     every workgroup expands its tokens and appends candidates {next, cost, source, arc} to
//              one segment per owner (simple states are not touched: their candidate is implied by
//              the token, and the best of them is known from the smallest token cost)
//   exchange 1 segment sizes and best costs
//   recombine  the owner's candidates go through an open-addressing table in LDS; the implied self-loop
//              candidates of its tokens look their own key up there; both are histogrammed
//   exchange 2 histograms: every workgroup finds the same cutoff, and where its tokens go in the set
//   tokens     survivors become tokens; those an epsilon arc can enter go into a table in LDS
//   closure    rounds of: expand the worklist over epsilon arcs into segments per owner, exchange of the
//              segment sizes, candidates meet the tokens in the table
//
// What bounds it: a frame of 10 k tokens is about 20 k arcs and 350 KB of memory traffic, a few
// microseconds for the chip, but a chain of some thirty dependent steps (loads, LDS round trips,
// barriers).  One workgroup takes 60-90 us for it, most of that because each step's work goes over
// 16 waves several times; spread over 8 compute units the steps are down to one round each.
//
// Workgroups talk through words {tag, value} of 64 bits, written and polled with relaxed
// atomics, the tag being the number of the exchange; the candidates travel the same way (two 8-byte
// stores; the writer waits for them before it posts the sizes).  A cluster's workgroups run on one
// XCD, so all of this stays in its L2.  Between compute units of different XCDs an exchange takes 1.1 us,
// 0.75 us more with 2 KB of data; one made with device-scope fences takes 9 us on an idle chip and
// over 100 us on a full one, since a fence writes back and invalidates whole L2 caches.
//
// The times in this file's comments are pairs, measured in turn on one card when the step was made, and later
// steps have moved both; the same code differs by a few percent between cards.

constexpr int kMaxG = 8;                      // workgroups of a cluster
constexpr int kKR = 3;                        // candidate records a lane keeps in registers from fill to token
constexpr int kNotes = kTabSlots + kKR * 1024; // candidates of a pass whose slots are noted
constexpr int kMapMax = kTabSlots * 3 / 4;    // most destinations in a table
constexpr unsigned kRefTok = 0x80000000u;     // low word of a table value: a token of the set, by local number
constexpr unsigned kRefStay = 0xFFFFFFFFu;    // ... or: a self-loop candidate won here
constexpr int kBoxWords = 512;                // mailbox words of one workgroup and exchange parity
constexpr int kBoxAux = 8, kBoxSel = 12, kBoxHist = 16;   // (three words of selection)
static_assert(kRegions == 4 && kMaxG == 2 * kRegions, "a region of keys is at most two workgroups'");
constexpr int kPolls = 1 << 23;               // most polls of a wait (seconds)
constexpr int kStartTicks = 5000;             // how long the first workgroup of a cluster waits for the others (50 us)
constexpr int kXcds = 8;                      // XCDs of the chip
constexpr int kHwXccId = 20 | (4 - 1) << 11;   // hardware register XCC_ID, bits 0-3: the XCD a wave runs on
constexpr int kListInts = 2 + kXcds + 2;       // counters in a launch's lists (an even number: 64-bit entries before them)
constexpr int kResetTid = 2 * 64, kStoredTid = 3 * 64, kPublishTid = 4 * 64;   // single threads' work between two frames, a wave each
constexpr int kAux = 4;                       // best cost, status, tokens made by the closure, smallest cost in a simple state

struct ClusterArgs {                          // device memory of the workgroups, by ticket of the cluster and number in it
  int G;                                      // workgroups per cluster
  int n_clusters;                             // clusters that decode (a launch can have some more, which end at once)
  unsigned seq;                               // number of the launch: tags the words of the formation
  int seg_cap;                                // records per segment
  int qcap;
  unsigned ticks;                             // how long the first workgroup of a cluster waits for the others (10 ns)
  int polls;                                  // how often a workgroup looks for another's word before it gives up
  int4 *cand;                                 // [workgroup][2][G][seg_cap]
  int2 *tok;                                  // [workgroup][2][qcap] the workgroup's own tokens {key + flags, cost}
  int *gi;                                    // [workgroup][2][qcap] their numbers in the set
  int4 *wl;                                   // [workgroup][2][qcap]
  unsigned long long *box;                    // [workgroup][2][kBoxWords] by XCD and order of arrival there
  unsigned long long *hello;                  // [workgroup][2] arrived / decided, likewise
};

constexpr int kHubDeg2 = 128;                 // arcs beyond which a state's arcs are shared by all waves
// The arcs of up to 64 work items of a wave, flattened over its lanes.  Arc f is the arc of the item whose
// number is the count of items that end before f: a bit per arc says where an item ends, and a lane counts the bits
// below its own.  (One LDS read and a count.  A binary search over prefix sums takes six dependent LDS reads, 1.5k
// cycles per 128 arcs: with it, and with runs of 64 tokens however small the set, one utterance of 10.8 k tokens per
// frame took 11.2 instead of 10.6 ms, one of 900 tokens 2.06 instead of 2.02 ms.)
struct alignas(16) WaveItem { int abase; float tcost; int src; int pad; };   // unit address of the first arc minus the arcs of the items before;
                                              // src: number of the token in its set | its state in the boosting acceptor << 16
struct alignas(16) WaveLds2 {
  unsigned long long last[kWaveTok * kHubDeg2 / 64];   // bit f: arc f is the last of its item
  WaveItem item[kWaveTok + 1];                // items with arcs, in order (lanes behind the last arc may read one more)
};
// The closure does the same over epsilon arcs, with smaller lists (the table lies in the memory of the others).  A
// state with more than kEpsDeg of them is listed in segments that all waves share.
constexpr int kWlLds = 96;                     // first entries of a worklist, kept in LDS
constexpr int kEpsTok = 32, kEpsDeg = 64, kEpsSeg = 64 * kU, kEpsSegs = 224;
struct alignas(16) WaveEps {
  unsigned long long last[kEpsTok * kEpsDeg / 64];
  WaveItem item[kEpsTok + 1];
};
struct alignas(16) Smem2 {
  union {
    struct { float ac[kMaxV]; WaveLds2 w[kWaves]; HubLds hub; } e;
    TableLds t;
  } u;
  union {
    struct { WaveEps w[kWaves]; WaveItem seg[kEpsSegs]; } ek;   // closure (of a segment `pad` is the number of arcs)
    struct {
      unsigned hasstay[kQueueMax / 32];       // bit i: local token i's first arc is the usual self-loop (other arcs follow)
      unsigned all[256], before[256];         // sums of the cluster's histograms: of all workgroups, of those before this one
    } s;
    int4 mk[kWaves][64];                      // survivors on their way to become tokens
  } v;
  int4 wl[2][kWlLds];                         // the closure's worklists, this round's and the next one's
  unsigned short tokof[kTabSlots];            // closure table: local token of a slot, 0xFFFF: none yet, or the last of a full set
  alignas(16) unsigned hist[256]; unsigned hist2[256], hist3[256];
  unsigned wave_tot[kWaves];
  int n_seg[kMaxG];                           // candidates pushed per segment
  alignas(16) int seg_lo[kMaxG]; unsigned seg_rel[kMaxG];   // own candidates, flattened: number of a segment's first one (none: INT_MAX),
                                              // and what turns a candidate's number into its place in the work memory
  int2 told[2];                               // by the parity of the exchange: how many they are; is the closure over (1), does some
                                              // candidate's state have epsilon arcs (2)
  unsigned x_best, x_minsimple;
  int x_status, x_made;
  int x_before;                               // overflows of the frame before
  int more, status_before, n_eseg;
  unsigned best_ord, min_simple;
  float stay_ac;
  int n_hub, next_run, done_waves;
  int made[4];                                // tokens made so far: outside simple states, in simple states; worklist entries; table entries
  int n_loc, n_win;
  int n_in;                                   // candidates of the workgroup that shares a region of keys with this one (0: none does);
                                              // where a region may hold too many, those inside the beam in the fullest one
  int map_bad, status, overfull;
  int polls, dead;                            // most polls of a wait; one has ended without its word
  int k_sel, n_sel, n_sel_c, k_keep, redo, n_emit, n_emit_all, gbase;
  unsigned ratio;
  int path_frames, trace_from, trace_words, sel_idx, job;
  unsigned long long red64, red64b;
  long long ctr[8], earc_before;               // (earc_before: ctr[kCtEarc] when the frame began)
  int bk[kBoostSlots]; float bv[kBoostSlots]; unsigned bft[kBoostSlots];
  long long prof[16];
  long long prof_t0;
};
static_assert(sizeof(Smem2) <= 160 * 1024, "LDS of a compute unit");
static_assert(offsetof(Smem2, u) % 16 == 0 && sizeof(TableLds) % 16 == 0 && offsetof(Smem2, v.s.all) % 16 == 0 && offsetof(Smem2, hist) % 16 == 0, "16 bytes at a time");
static_assert(kNotes == kTabSlots + kKR * kBlock, "a register each");
static_assert(kKR * kBlock <= kMapMax, "one register-held round fits the table");

struct Cx {                   // block-uniform view of one channel
  const DevGraph &g; const DevChannels &c; const ClusterArgs &w; Smem2 &sm;
  int4 *cand;                 // solo: the channel's four regions; cluster: slot 0's first segment
  int4 *win; int win_cap;     // recombined tokens when they do not fit registers
  int2 *tq; int *gi; int4 *wl0;      // two buffers of qcap each: tokens, their numbers (cluster), worklists
  int2 *q0;                   // the channel's dense token queue, two buffers
  int2 *lat; unsigned *frame_off;
  unsigned long long *dig_sum; int *dig_cnt;
  ChanState s;
  unsigned lat_cap;
  // cluster
  int G, lg, me, seg_cap;     // (a cluster that came out smaller than planned has larger segments)
  size_t seg_stride;          // records of one workgroup's segments, all owners
  unsigned xc, hc;            // exchanges, and histogram exchanges, so far
  unsigned long long *box0;   // slot 0's mailbox
  // own tokens
  int n, n_front, n_emit;     // [0, n_front): not in simple states; [n_front, n_emit): simple; the rest: made by the closure
};
// The lane's number, opaque to the compiler: what is computed from it is computed again in every phase
// instead of being kept (and spilled) through the frame loop.
__device__ __forceinline__ int lane_id() { int t = threadIdx.x; asm volatile("" : "+v"(t)); return t; }
// (one LDS instruction that nobody waits for)
__device__ __forceinline__ void count2(Smem2 &sm, int which, int n) { atomicAdd((unsigned long long *)&sm.ctr[which], (unsigned long long)(long long)n); }
template <bool kProf> __device__ __forceinline__ void mark(Cx &x, int phase) {
  if (kProf && threadIdx.x == 0) {
    const long long now = (long long)wall_clock64();
    x.sm.prof[phase] += now - x.sm.prof_t0;
    x.sm.prof_t0 = now;
  }
}

// ------------------------------------------------------------------ memory other workgroups read or wrote
// The workgroups of a cluster run on one XCD, and the compute units of an XCD share one L2.  A store of
// workgroup scope goes through to that L2 (the vector cache writes through) and is acknowledged there, a
// load of device scope passes the compute unit's vector cache by and is served by the L2, and a
// read-modify-write is done in it: enough for workgroups of one XCD, and nothing waits for the memory
// behind the L2.  (A load of workgroup scope may hit a stale line of the vector cache.)  With stores of device
// scope, which are acknowledged behind the L2: one utterance of 11 k tokens per frame 12.0 instead of 11.2 ms, 32 at
// once 44.7 instead of 40.8 ms, 256 at once 73.0 instead of 67.2 ms; with the workgroups of a cluster on any
// XCDs 12.6, 45.9 and 73.3 ms.
constexpr auto kLoadScope = __HIP_MEMORY_SCOPE_AGENT, kStoreScope = __HIP_MEMORY_SCOPE_WORKGROUP;
__device__ __forceinline__ unsigned long long aload(const unsigned long long *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, kLoadScope);
}
__device__ __forceinline__ void astore(unsigned long long *p, unsigned long long v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, kStoreScope);
}
__device__ __forceinline__ unsigned long long u64_of(int lo, int hi) { return ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo; }
template <bool kCl> __device__ __forceinline__ void put4(int4 *p, int4 v) {
  if (kCl) {
    unsigned long long *q = reinterpret_cast<unsigned long long *>(p);
    astore(q, u64_of(v.x, v.y)); astore(q + 1, u64_of(v.z, v.w));
  } else *p = v;
}
template <bool kCl> __device__ __forceinline__ int4 get4(const int4 *p) {
  if (!kCl) return *p;
  const unsigned long long *q = reinterpret_cast<const unsigned long long *>(p);
  const unsigned long long a = aload(q), b = aload(q + 1);
  return make_int4((int)(unsigned)a, (int)(a >> 32), (int)(unsigned)b, (int)(b >> 32));
}
template <bool kCl> __device__ __forceinline__ void put_lat(int2 *p, int prev, int arc) {
  if (kCl) astore(reinterpret_cast<unsigned long long *>(p), u64_of(prev, arc));
  else *p = make_int2(prev, arc);
}
template <bool kCl> __device__ __forceinline__ int2 get_lat(const int2 *p) {
  if (!kCl) return *p;
  const unsigned long long a = aload(reinterpret_cast<const unsigned long long *>(p));
  return make_int2((int)(unsigned)a, (int)(a >> 32));
}

// Every wait is bounded (seconds): a partner that never posts ends the channel with an error instead of hanging the
// launch.  Is it time to give up, after n looks in vain?  sm.dead is then set.
__device__ __forceinline__ bool give_up_wait(Smem2 &sm, int n, int polls) {
  const bool over = n >= polls || ((n & 1023) == 1023 && __hip_atomic_load(&sm.dead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
  if (over) sm.dead = 1;
  return over;
}
// Wait until the word carries the tag (its upper half); returns the word, or 0 (no tag is) for a wait that was given up.
__device__ __forceinline__ unsigned long long poll_word(Smem2 &sm, const unsigned long long *p, unsigned tag, int polls) {
  for (int n = 0;; ++n) {
    const unsigned long long v = aload(p);
    if ((unsigned)(v >> 32) == tag) return v;
    if (give_up_wait(sm, n, polls)) return 0;
  }
}
__device__ __forceinline__ unsigned poll(Smem2 &sm, const unsigned long long *p, unsigned tag) {
  return (unsigned)poll_word(sm, p, tag, sm.polls);
}
__device__ __forceinline__ unsigned long long *box_of(const Cx &x, int r) {
  return x.box0 + (unsigned)((r * 2 + (int)(x.xc & 1u)) * kBoxWords);
}
// The set of segments (of two) that the last exchange of sizes was about; candidates on their way go to the other one.
__device__ __forceinline__ int seg_set(const Cx &x) { return (int)((x.xc - x.hc) & 1u); }
__device__ __forceinline__ unsigned long long *hist_of(const Cx &x, int r) {
  return x.box0 + (unsigned)((r * 2 + (int)(x.hc & 1u)) * kBoxWords + kBoxHist);
}
__device__ __forceinline__ void post(const Cx &x, int word, unsigned v) {
  astore(box_of(x, x.me) + word, ((unsigned long long)x.xc << 32) | v);
}
// The cluster's counter of tokens in the set under construction (the closure takes numbers from it).
__device__ __forceinline__ unsigned *set_size_of(const Cx &x) { return reinterpret_cast<unsigned *>(x.box0 + kBoxWords - 1); }
__device__ __forceinline__ void set_counter(const Cx &x, int n) { __hip_atomic_store(set_size_of(x), (unsigned)n, __ATOMIC_RELAXED, kStoreScope); }
// Entry f of a per-frame table of n entries (a ring if the stream outlives it).
__device__ __forceinline__ int ring_at(int f, int n) { return f < n ? f : f % n; }
// Every store of this thread has reached the L2.
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Owner of a key among 2^lg parts: the top bits of its hash.
__device__ __forceinline__ int part_of(int key, int lg) { return (int)((hash_state(key) >> 1) >> (31 - lg)); }

// Post the sizes of the segments this workgroup has filled, its best cost and its status.  All threads call it, when
// what the others go on to read or add to is in the L2: the candidates of all waves, by stores_done() and then a barrier, and the
// set's counter, which thread 0 of the first workgroup stores before a frame's first closure round, by stores_done() of
// its wave, which posts.
template <bool kCl>
__device__ __forceinline__ void post_sizes(Cx &x) {
  Smem2 &sm = x.sm;
  const int tid = lane_id();
  if (!kCl) return;
  ++x.xc;
  static_assert(((kStLattice | kStCapacity) & ~0xff) == 0, "the word of the status has 8 bits for it");
  static_assert(kBoxAux == kMaxG, "a lane per word");
  if (tid < kBoxAux + kAux) {
    const int q = tid - kBoxAux;
    unsigned v = 0;
    if (tid < x.G) { v = (unsigned)sm.n_seg[tid]; sm.n_seg[tid] = 0; }
    const bool any = __ballot(v != 0) != 0ull;
    if (q == 0) v = sm.best_ord;
    if (q == 1) { v = (unsigned)(sm.status | sm.status_before << 8 | sm.more << 16 | (int)any << 17); sm.more = 0; }
    if (q == 2) v = (unsigned)(sm.n_loc - x.n_emit);
    if (q == 3) v = sm.min_simple;
    if (tid < x.G || q >= 0) post(x, tid, v);
  }
}
// Take the cluster's sizes: own candidates are [0, n_own) afterwards.  Ends with a barrier.  Three waves share the
// work, and sums go by lane reads: the sizes through LDS, one wave for all of the rest and butterflies for minima made an exchange
// 0.3 us longer (four or five exchanges a frame: one utterance of 10.8 k tokens 9.93 instead of 9.70 ms, with the other trips
// through LDS that are now not waited for).  A workgroup looks only at its own sizes and at those of the one it shares a
// region with.
// A workgroup of the closure that gets no candidates and has none to expand goes from here straight into the next exchange, while
// some of its waves may still be reading what this one told.  So the closure goes by sm.told alone: an exchange overwrites what
// the one two before it left there, and no wave still reads that, since all of them have come to the barrier of the one between.
// (One set of words and a barrier on that way: one utterance 9.48 instead of 9.40 ms, 32 32.89 instead of 32.66; with this
// 9.41 and 32.33 against 9.38 and 32.27 with nothing.)
template <bool kCl>
__device__ __forceinline__ void take_sizes(Cx &x) {
  Smem2 &sm = x.sm;
  const int tid = lane_id(), lane = tid & 63;
  const int region_cap = x.c.region_cap;
  if (tid < 64) {
    if (kCl) {
      // lane r: writer r's segment for this workgroup; of a cluster of 8, lane 8 + r: for the one it shares a region with
      unsigned v = 0;
      const int r = lane & (kMaxG - 1);
      if (lane < (x.G == kMaxG ? 2 * kMaxG : x.G)) v = min((unsigned)poll_word(sm, box_of(x, r) + (x.me ^ (lane >> 3)), x.xc, sm.polls), (unsigned)x.seg_cap);
      const unsigned inc = wave_scan_add(v);
      const unsigned own = (unsigned)__builtin_amdgcn_readlane((int)inc, kMaxG - 1);
      if (lane < kMaxG) {
        const int lo = (int)(inc - v);
        sm.seg_lo[lane] = lane < x.G ? lo : INT_MAX;
        sm.seg_rel[lane] = (unsigned)(lane * 2 + seg_set(x)) * (unsigned)x.seg_stride + (unsigned)(x.me * x.seg_cap - lo);
      }
      if (lane == 0) sm.told[x.xc & 1u].x = (int)own;
      if (lane == 2 * kMaxG - 1) sm.n_in = (int)(inc - own);         // (0 unless there are eight)
    } else {
      const int n = lane < kRegions ? min(sm.n_seg[lane], region_cap) : 0;
      const int inc = (int)wave_scan_add((unsigned)n);
      if (lane < kRegions) { sm.seg_lo[lane] = inc - n; sm.seg_rel[lane] = (unsigned)(lane * region_cap - (inc - n)); sm.n_seg[lane] = 0; }
      const int status = sm.status, more = sm.more;
      if (lane == 0) { sm.x_best = sm.best_ord; sm.x_status = status; sm.more = 0; }
      if (lane == kRegions - 1) sm.told[0] = make_int2(inc, (int)(inc == 0 || status != 0) | more << 1);
    }
  } else if (kCl && tid < 192) {                 // best costs and status, and (the next wave) tokens made and costs in simple states
    unsigned long long w = 0;
    const bool second = tid >= 128;
    const int which = lane & 1;
    const bool mine = lane < kAux / 2 * x.G;
    if (mine) w = poll_word(sm, box_of(x, lane >> 1) + kBoxAux + which + (second ? 2 : 0), x.xc, sm.polls);
    const unsigned v = (unsigned)w;
    if (second) {
      const unsigned made = wave_sum(mine && which == 0 ? v : 0u), ms = wave_min(mine && which == 1 ? v : kOrdNone);
      if (lane == 0) { sm.x_made = (int)made; sm.x_minsimple = ms; }
    } else {
      const unsigned best = wave_min(mine && which == 0 ? v : kOrdNone), st = mine && which == 1 ? v : 0u;
      auto any = [&](unsigned bits) { return __ballot((st & bits) != 0) != 0ull; };
      const int now = (any(kStLattice) ? kStLattice : 0) | (any(kStCapacity) || __ballot(mine && w == 0ull) != 0ull ? kStCapacity : 0);
      const int before = (any(kStLattice << 8) ? kStLattice : 0) | (any(kStCapacity << 8) ? kStCapacity : 0);
      const int more = any(1u << 16), some = any(1u << 17);
      if (lane == 0) { sm.x_best = best; sm.x_status = now; sm.x_before = before; sm.told[x.xc & 1u].y = (int)(!some || now != 0) | more << 1; }
    }
  }
  __syncthreads();
}

// Address of own candidate i (flattened over the segments of the last exchange): four LDS reads, a comparison and a
// select per segment.  (With the segment's number, its first candidate and 64-bit products instead of one 32-bit offset it was
// twice as many instructions: 256 utterances 62.0 instead of 61.5 ms, 32 32.35 instead of 32.13, one 8.86 instead of 8.80.)
template <bool kCl>
__device__ __forceinline__ const int4 *cand_at(const Cx &x, int i) {
  const Smem2 &sm = x.sm;
  const int4 lo0 = *reinterpret_cast<const int4 *>(&sm.seg_lo[0]);
  const uint4 re0 = *reinterpret_cast<const uint4 *>(&sm.seg_rel[0]);
  unsigned rel = re0.x;
  rel = i >= lo0.y ? re0.y : rel; rel = i >= lo0.z ? re0.z : rel; rel = i >= lo0.w ? re0.w : rel;
  if (!kCl) return x.cand + (rel + (unsigned)i);
  const int4 lo1 = *reinterpret_cast<const int4 *>(&sm.seg_lo[4]);
  const uint4 re1 = *reinterpret_cast<const uint4 *>(&sm.seg_rel[4]);
  rel = i >= lo1.x ? re1.x : rel; rel = i >= lo1.y ? re1.y : rel; rel = i >= lo1.z ? re1.z : rel; rel = i >= lo1.w ? re1.w : rel;
  return x.cand + (rel + (unsigned)i);
}

// Append a batch of N candidates per lane to their owners' segments.  The lanes of a segment get
// consecutive slots from one LDS atomic instruction, so their stores coalesce.
template <bool kCl, int N>
__device__ __forceinline__ void push_cands2(Cx &x, const int (&ok)[N], const int (&next)[N], const float (&nc)[N],
                                            const int (&src)[N], const int (&arc)[N], int buf) {
  const int lg = kCl ? x.lg : kRegionBits;
  const int cap = kCl ? x.seg_cap : x.c.region_cap;
  int4 *out = kCl ? x.cand + (size_t)(x.me * 2 + buf) * x.seg_stride : x.cand;
  int p[N], slot[N];                             // (all places are asked for before the first is waited for)
#pragma unroll
  for (int u = 0; u < N; ++u) {
    p[u] = part_of(key_of(next[u]), lg); slot[u] = 0;
    if (ok[u]) slot[u] = atomicAdd(&x.sm.n_seg[p[u]], 1);
  }
#pragma unroll
  for (int u = 0; u < N; ++u)
    if (ok[u]) {
      if (slot[u] < cap) put4<kCl>(out + (size_t)p[u] * cap + slot[u], make_int4(next[u], __float_as_int(nc[u]), src[u], arc[u]));
      else atomicOr(&x.sm.status, kStCapacity);
    }
}

__device__ __forceinline__ float boost_step2(const Smem2 &sm, int b, int word, int &nb) {
  unsigned h = boost_slot(word);
  float root_score = 0.0f; int root_to = 0;
  for (;;) {
    const int k = sm.bk[h];
    if (k == 0) break;                       // the table is never full (kBoostMax < kBoostSlots)
    if (k == word) {
      const unsigned ft = sm.bft[h];
      const int from = (int)(ft & 0xffffu);
      if (from == b) { nb = (int)(ft >> 16); return sm.bv[h]; }
      if (from == 0) { root_to = (int)(ft >> 16); root_score = sm.bv[h]; }
    }
    h = (h + 1) & (kBoostSlots - 1);
  }
  nb = root_to;
  return root_score;
}

__device__ __forceinline__ float stay_cost2(const Cx &x, float c) { return canon((c + x.g.simple_w) + x.sm.stay_ac); }

// ------------------------------------------------------------------ ExpandArcs (emitting)
template <bool kCl, int N>
__device__ __forceinline__ void emit_arcs2(Cx &x, int (&ok)[N], const int4 (&a)[N], const float (&tc)[N],
                                           const int (&src)[N], const int (&arc)[N], float beam, bool boosted) {
  Smem2 &sm = x.sm;
  const unsigned bo = __hip_atomic_load(&sm.best_ord, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  const float rb = bo == kOrdNone ? INFINITY : ord2f(bo);
  unsigned o = kOrdNone;
  float nc[N]; int next[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    nc[u] = canon((tc[u] + __int_as_float(a[u].y)) + sm.u.e.ac[a[u].z - 1]);
    next[u] = a[u].x;
    if (boosted) {                             // the destination's key carries the token's state in B
      const int b = (int)((unsigned)src[u] >> 16);
      int nb = b;
      if (a[u].w != 0 && ok[u]) nc[u] = canon(nc[u] + boost_step2(sm, b, a[u].w, nb));   // + B's score
      next[u] |= nb << x.g.blk_bits;
    }
    ok[u] &= (int)(nc[u] < INFINITY) & (int)!((nc[u] - rb) > beam);
    o = min(o, ok[u] ? f2ord(nc[u]) : kOrdNone);
  }
  if (__ballot(o < bo) != 0ull) {
    const unsigned m = wave_min(o);
    if ((threadIdx.x & 63) == 0) atomicMin(&sm.best_ord, m);
  }
  push_cands2<kCl, N>(x, ok, next, nc, src, arc, kCl ? seg_set(x) ^ 1 : 0);
}
__device__ __forceinline__ int next_run2(Smem2 &sm) {
  int r = 0;
  if ((threadIdx.x & 63) == 0) r = atomicAdd(&sm.next_run, 1);
  return uni(r);
}
// Lists the items of a wave, one per lane (deg arcs from unit address `first`, at most kHubDeg2 (kEpsDeg) of them; 0: no
// item); returns the number of arcs.
template <class L>
__device__ __forceinline__ int list_items(L &wl, unsigned deg, int first, float cost, int src) {
  const int lane = lane_id() & 63;
  constexpr int kWords = sizeof(wl.last) / 8;
  static_assert(kWords == 128 || kWords <= 64, "cleared by one store per lane");
  const unsigned inc = wave_scan_add(deg);
  const unsigned long long has = __ballot(deg != 0);
  if (kWords == 128) { wl.last[2 * lane & (kWords - 1)] = 0ull; wl.last[(2 * lane + 1) & (kWords - 1)] = 0ull; }
  else if (lane < kWords) wl.last[lane] = 0ull;
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (deg) {
    const unsigned e = inc - 1;
    atomicOr(&wl.last[e >> 6], 1ull << (e & 63));
    wl.item[__builtin_amdgcn_mbcnt_hi((unsigned)(has >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)has, 0u))] = WaveItem{first - (int)(inc - deg), cost, src, 0};
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  return __builtin_amdgcn_readlane((int)inc, 63);
}
// The item of the lane's arc in the w-th run of 64 arcs; `before`: items that end in earlier runs (kept by the caller).
template <class L>
__device__ __forceinline__ WaveItem item_of(const L &wl, int w, int &before) {
  const unsigned long long m = wl.last[w & (int)(sizeof(wl.last) / 8 - 1)];    // (a run behind the last arc: anything)
  const unsigned lo = uni((unsigned)m), hi = uni((unsigned)(m >> 32));
  const int j = before + (int)__builtin_amdgcn_mbcnt_hi(hi, __builtin_amdgcn_mbcnt_lo(lo, 0u));
  before += __popc(lo) + __popc(hi);
  return wl.item[min(j, (int)(sizeof(wl.item) / sizeof(WaveItem)) - 1)];
}
// The tokens of a wave, one per lane (`valid`; id: local number | number in the set << 16): a lane reads the
// 16 bytes at the end of its token's header (degrees and the first arc); the other arcs are flattened over the 64
// lanes, and states with more than kHubDeg2 arcs are listed for all waves.  Returns the emitting arcs expanded
// (wave-uniform).
template <bool kCl>
__device__ __forceinline__ unsigned run2(Cx &x, WaveLds2 &wl, int2 tk, int id, bool valid, float beam, bool boosted) {
  Smem2 &sm = x.sm;
  HubLds &hb = sm.u.e.hub;
  const int lane = lane_id() & 63;
  const unsigned bm = x.g.blk_mask; const int bbits = x.g.blk_bits;
  const int blk = (int)((unsigned)tk.x & bm);
  int4 hd = make_int4(0, 0, 0, 1);                       // no arcs; ilabel 1 keeps the acoustic lookup in range
  if (valid) hd = load_block_head(x.g.unit, blk);
  // number in the set, and the token's state in the boosting acceptor (0 without one)
  const int srct = (int)((unsigned)id >> 16) | (int)((((unsigned)tk.x & kKeyMask) >> bbits) << 16);
  int ne = (int)((unsigned)hd.x & kPackE); const int nx = (int)((unsigned)hd.x >> kPackXShift);
  if (ne == (int)kPackE) ne = x.g.unit[2 * (size_t)(unsigned)blk].z;        // a very large state: exact degree
  int has = (int)(ne > 0) & (int)(nx == 0);           // the unit after the header is an emitting arc
  unsigned deg = (unsigned)(ne - has);
  int first = 2 * blk + 1 + nx + has;                 // unit address of the first arc left
  const float cost = __int_as_float(tk.y);
  int4 a0 = make_int4(hd.y, hd.z, has ? (hd.w & kLabelMask) : 1, 0);
  unsigned n_arcs = (unsigned)__popcll(__ballot(has));
  {
    // The first arc is the usual self-loop: its candidate is implied, like that of a token in a
    // simple state; the bit set says for which tokens.  Here it only lowers the running best.
    const int loop = has & (int)((unsigned)hd.w >> 31);
    const float nc = stay_cost2(x, cost);
    const unsigned bo = __hip_atomic_load(&sm.best_ord, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    const unsigned o = (loop && nc < INFINITY) ? f2ord(nc) : kOrdNone;
    if (__ballot(o < bo) != 0ull) {
      const unsigned mo = wave_min(o);
      if (lane == 0) atomicMin(&sm.best_ord, mo);
    }
    const int tok = id & 0xffff;
    if (loop) atomicOr(&sm.v.s.hasstay[tok >> 5], 1u << (tok & 31));
    has &= (int)!loop;
  }
  if (boosted && has) a0.w = x.g.unit[2 * (size_t)(unsigned)blk + 1].w;    // the first arc's olabel
  if (deg > (unsigned)kHubDeg2) {                     // to the shared list, if it has room
    const int h = atomicAdd(&sm.n_hub, 1);
    if (h < kHubCap) {
      hb.first[h] = first; hb.deg[h] = (int)deg; hb.tcost[h] = cost; hb.ttok[h] = srct;
      __hip_atomic_store(&hb.ready[h], 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
      deg = 0;
    }
  }
  // two arcs per lane and step; the first step takes the batch's first arcs and 64 of the others.  (A state that found
  // the shared list full comes back with its next kHubDeg2 arcs: an item has no more.)
  for (int f0 = -64;; f0 = 0) {
    const unsigned take = min(deg, (unsigned)kHubDeg2);
    const unsigned M = (unsigned)list_items(wl, take, first, cost, srct);
    n_arcs += M;
    int w = 0, before = 0;
    do {
      int ok[2], src[2], arc[2]; int4 a[2]; float tc[2];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int f = f0 + u * 64 + lane;
        if (u == 0 && f0 < 0) { ok[0] = has; src[0] = srct; arc[0] = 2 * blk + 1; tc[0] = cost; a[0] = a0; continue; }
        ok[u] = f < (int)M;
        const WaveItem it = item_of(wl, w++, before);
        src[u] = it.src; tc[u] = it.tcost;
        arc[u] = it.abase + f;
        a[u] = make_int4(0, 0, 1, 0);
        if (ok[u]) a[u] = load_emitting_arc<false>(x.g, arc[u], boosted);
      }
      emit_arcs2<kCl, 2>(x, ok, a, tc, src, arc, beam, boosted);
      f0 += 128;
    } while (f0 < (int)M);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    deg -= take; first += (int)take;
    if (__ballot(deg != 0) == 0ull) break;
  }
  return n_arcs;
}
// A wave's tokens to expand.  The tokens outside simple states come first, then (among simple ones, which are skipped)
// those the closure made; a run is `size` of them, so that all waves have one where the set is small.
struct Run { int2 tk; int i, gi; bool valid; };   // (nothing is made of its numbers before they are needed: that would wait for them)
__device__ __forceinline__ int run_size(const Cx &x) {
  return min(kWaveTok, max(16, (x.n_front + x.n - x.n_emit + kWaves - 1) / kWaves));
}
template <bool kCl>
__device__ __forceinline__ Run load_run(const Cx &x, const int2 *Q, const int *GI, int r, int size) {
  const int lane = lane_id() & 63, j = r * size + lane;
  // (all lanes load, those without a token the first record: behind a branch the record would be copied, and so waited for)
  Run run{};
  run.valid = lane < size && j < x.n_front + x.n - x.n_emit;
  run.i = !run.valid ? 0 : j < x.n_front ? j : j - x.n_front + x.n_emit;
  run.tk = Q[run.i];
  if (kCl) run.gi = GI[run.i];
  return run;
}
// On entry sm.next_run == kWaves, sm.done_waves == 0, sm.n_hub == 0 and the hub list's ready
// and seg_next words are zero (the caller sets them before its barrier); `run`: the wave's first run.
template <bool kCl, bool kBoost>
__device__ __forceinline__ void expand2(Cx &x, const int2 *Q, const int *GI, Run run) {
  Smem2 &sm = x.sm;
  HubLds &hb = sm.u.e.hub;
  const int tid = lane_id(), lane = tid & 63, wave = tid >> 6;
  const float beam = x.s.beam;
  const bool boosted = kBoost && x.s.boost_n > 0;
  WaveLds2 &wl = sm.u.e.w[uni(wave)];
  const int size = run_size(x), total = x.n_front + x.n - x.n_emit;
  // the simple tokens of the emitting step have one arc each
  unsigned long long n_arcs = tid < 64 ? (unsigned long long)(x.n_emit - x.n_front) : 0ull;
  for (int r = uni(wave); r * size < total;) {
    r = size * kWaves >= total ? kWaves : next_run2(sm);
    const bool more = r * size < total;
    Run nxt{};
    if (more) nxt = load_run<kCl>(x, Q, GI, r, size);
    const bool other = run.valid && ((unsigned)run.tk.x & kFlagSimple) == 0;
    n_arcs += (unsigned)__popcll(__ballot(run.valid && !other));
    n_arcs += run2<kCl>(x, wl, run.tk, run.i | ((kCl ? run.gi : run.i) << 16), other, beam, boosted);
    if (more) run = nxt;
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  if (lane == 0) atomicAdd(&sm.done_waves, 1);
  // ---- listed states, a segment at a time, until every wave is done listing and none is left
  {
    int h = 0, spins = 0;
    while (h < kHubCap) {
      int ready = uni(__hip_atomic_load(&hb.ready[h], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
      if (!ready) {
        const int done = uni(__hip_atomic_load(&sm.done_waves, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
        if (done == kWaves) {                           // nobody lists any more: is the entry really absent?
          ready = uni(__hip_atomic_load(&hb.ready[h], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
          if (!ready) break;
        } else {
          if (++spins > (1 << 22)) { if (lane == 0) atomicOr(&sm.status, kStCapacity); break; }   // never expected
          __builtin_amdgcn_s_sleep(2);
          continue;
        }
      }
      int seg = 0;
      if (lane == 0) seg = atomicAdd(&hb.seg_next[h], 1);
      seg = uni(seg);
      const int deg = uni(hb.deg[h]);
      const int f0 = seg * kHubSeg;
      if (f0 >= deg) { ++h; continue; }
      const int first = uni(hb.first[h]), tok = uni(hb.ttok[h]); const float cost = uni(hb.tcost[h]);
      {
        int ok[kUE], src[kUE], arc[kUE]; int4 a[kUE]; float tc[kUE];
#pragma unroll
        for (int u = 0; u < kUE; ++u) {
          const int f = f0 + u * 64 + lane;
          ok[u] = f < deg;
          arc[u] = first + (ok[u] ? f : deg - 1);      // lanes past the end repeat the last arc (no branch)
          src[u] = tok; tc[u] = cost;
          a[u] = load_emitting_arc<false>(x.g, arc[u], boosted);
        }
        emit_arcs2<kCl, kUE>(x, ok, a, tc, src, arc, beam, boosted);
      }
      n_arcs += (unsigned)min(kHubSeg, deg - f0);
    }
  }
  if (lane == 0 && n_arcs) atomicAdd((unsigned long long *)&sm.ctr[kCtEarc], n_arcs);
}

// ------------------------------------------------------------------ recombination in LDS
__device__ __forceinline__ void clear_table(Smem2 &sm) {
  static_assert(sizeof(TableLds) % (16 * kBlock) == 0 && kKeyEmpty == -1 && kValEmpty == ~0ull, "cleared 16 bytes at a time");
  int4 *p = reinterpret_cast<int4 *>(&sm.u.t);
#pragma unroll
  for (int i = 0; i < (int)(sizeof(TableLds) / (16 * kBlock)); ++i) p[i * kBlock + threadIdx.x] = make_int4(-1, -1, -1, -1);
}
// Which of P equal parts of its owner's keys a key belongs to.
__device__ __forceinline__ int group2(int key, int lg, int P) {
  return (int)((((hash_state(key) << lg) >> 21) * (unsigned)P) >> 11);
}

// Lower the destination's table entry to this candidate if (cost, arc id, source's B state) is
// smaller.  In the closure (kClosure) the entry may be a token of the set, and a claimed slot is marked as
// having none.  Returns the slot, or -1 and sm.overfull if kProbeLimit probes have found none: the table is (nearly) full, or
// the keys lie at regular distances, as those of states one behind the other do, and their probe sequences are alike.  Every
// caller goes on from there with more passes.
template <bool kCl, bool kClosure>
__device__ __forceinline__ int insert2(Cx &x, int dst, float cost, int arc, int src, int idx,
                                       const int *NGI, unsigned lat_base) {
  TableLds &t = x.sm.u.t;
  unsigned s = probe_start(dst);
  const unsigned step = probe_step(dst);
  int old;
  for (int probes = 0;; ++probes) {
    old = atomicCAS(&t.keys[s], kKeyEmpty, dst);
    if (old == kKeyEmpty || old == dst) break;
    s = (s + step) & kTabMask;
    if (probes >= kProbeLimit) { old = kKeyNone; break; }
  }
  if (old == kKeyNone) { atomicOr(&x.sm.overfull, 1); return -1; }
  if (kClosure && old == kKeyEmpty) x.sm.tokof[s] = 0xFFFFu;
  const unsigned oc = f2ord(cost);
  const unsigned long long mine = ((unsigned long long)oc << 32) | (unsigned)idx;
  unsigned long long cur = kValEmpty;
  if (old != kKeyEmpty) cur = t.vals[s];
  for (;;) {
    const unsigned cc = (unsigned)(cur >> 32);
    bool better = oc < cc;
    if (oc == cc && cur != kValEmpty) {            // exact tie: lower arc id, then lower B state of the source
      int oarc, osrc;
      const unsigned low = (unsigned)cur;
      if (kClosure && (low & kRefTok)) {
        const int li = (int)(low & ~kRefTok);
        // (a token that found no room was never written; its channel stops after this frame)
        const unsigned at = (unsigned)(kCl ? NGI[li] : li);
        const int2 bp = at < (unsigned)x.c.qcap && lat_base + at < x.lat_cap ? get_lat<kCl>(x.lat + lat_base + at) : make_int2(0, 0);
        osrc = bp.x; oarc = bp.y;
      } else {
        const int4 o = get4<kCl>(cand_at<kCl>(x, (int)low));
        osrc = o.z; oarc = o.w;
      }
      better = (unsigned)arc < (unsigned)oarc;
      if (arc == oarc) better = ((unsigned)src >> 16) < ((unsigned)osrc >> 16);
    }
    if (!better) break;
    const unsigned long long prev = atomicCAS(&t.vals[s], cur, mine);
    if (prev == cur) break;
    cur = prev;
  }
  return (int)s;
}
// Slot of a key, or -1.
__device__ __forceinline__ int find2(const Smem2 &sm, int key) {
  const TableLds &t = sm.u.t;
  unsigned s = probe_start(key);
  const unsigned step = probe_step(key);
  int k = t.keys[s];
  for (int probes = 0; k != key && k != kKeyEmpty && probes <= kProbeLimit; ++probes) { s = (s + step) & kTabMask; k = t.keys[s]; }
  return k == key ? (int)s : -1;
}

// The implied self-loop candidates of the tokens (of sub-group g of G): a candidate inside the beam and the
// selected bins looks its key up; it is its state's recombined token unless the table holds a
// better one (cost, then arc id).  `nxt`: the lane's first token.  Returns the lane's winners as bits (bit k: token k * kBlock + tid).
template <bool kCl>
__device__ __forceinline__ unsigned long long stays2(Cx &x, const int2 *Q, int2 nxt, const Cutoff &cut, int k_sel, int g, int P) {
  Smem2 &sm = x.sm;
  TableLds &t = sm.u.t;
  const int tid = lane_id(), n = x.n;
  const int lg = kCl ? x.lg : 0;
  unsigned long long won = 0;
  for (int k = 0; k * kBlock < n; ++k) {
    const int i = k * kBlock + tid;
    const int2 q = nxt;
    if (i + kBlock < n) nxt = Q[i + kBlock];
    const int key = key_of(q.x);
    const float nc = stay_cost2(x, __int_as_float(q.y));
    const int b = cut.bin(nc);
    int in = (int)(i < n) & (int)(((unsigned)q.x & kFlagSimple) != 0);
    // (most of the set is a block of tokens in simple states)
    if (k * kBlock < x.n_front || (k + 1) * kBlock > x.n_emit) in |= (int)(i < n) & (int)((sm.v.s.hasstay[(i & (kQueueMax - 1)) >> 5] >> (i & 31)) & 1u);
    in &= (int)(nc < INFINITY) & (int)cut.in_beam(nc) & (int)(b < k_sel);
    if (P > 1) in &= (int)(group2(key, lg, P) == g);
    if (in) {
      const int sl = find2(sm, key);
      int win = 1;
      if (sl >= 0) {
        const unsigned long long v = t.vals[sl];
        const unsigned oc = f2ord(nc), cc = (unsigned)(v >> 32);
        win = (int)(oc < cc);
        if (oc == cc) win = (int)(2u * ((unsigned)q.x & x.g.blk_mask) + 1u < (unsigned)get4<kCl>(cand_at<kCl>(x, (int)(unsigned)v)).w);
        if (win) t.vals[sl] = ((unsigned long long)oc << 32) | kRefStay;
      }
      if (win) atomicAdd(&sm.hist[b], 1u);
      won |= (unsigned long long)win << k;
    }
  }
  return won;
}

// ------------------------------------------------------------------ token creation
// An entry of a worklist of the closure {number in the set, key, cost, new}: a short list is read out of LDS.
__device__ __forceinline__ void list_eps(Cx &x, int sel, int wi, int4 e) {
  if (wi < kWlLds) x.sm.wl[sel][wi] = e;
  else if (wi < x.c.qcap) (x.wl0 + sel * x.c.qcap)[wi] = e;
}
// New tokens of the emitting step, one per lane: own record, number in the set, backpointer, an entry in the
// worklist if the state has epsilon arcs, and one in the closure's table if an epsilon arc enters it.
// Tokens outside simple states are numbered from the front, the others from the back.
template <bool kCl, bool kOpt>
__device__ __forceinline__ void make2(Cx &x, int ok, int next, int costbits, int src, int arc, const Cutoff &cut,
                                      int2 *NQ, int *NGI, unsigned lat_base, int n_emit, int gbase) {
  Smem2 &sm = x.sm;
  TableLds &t = sm.u.t;
  const int lane = lane_id() & 63;
  const int simple = (int)(((unsigned)next & kFlagSimple) != 0);
  int cb = costbits;
  if (kOpt && x.c.cost_offset) cb = __float_as_int(canon(__int_as_float(costbits) - cut.best));
  // places from the four counters with one LDS instruction: lane q takes counter q's
  const unsigned long long lt = (1ull << lane) - 1ull;
  const unsigned long long m0 = __ballot(ok & (int)!simple), m1 = __ballot(ok & simple);
  const unsigned long long m2 = __ballot(ok & (int)((unsigned)next >> 31)), m3 = __ballot(ok & (int)(((unsigned)next >> 30) & 1u));
  static_assert(kFlagHasEps == 1u << 31 && kFlagEpsIn == 1u << 30, "flag bits");
  int at = 0;
  if (lane < 4) at = atomicAdd(&sm.made[lane], __popcll(lane == 0 ? m0 : lane == 1 ? m1 : lane == 2 ? m2 : m3));
  const int li = simple ? n_emit - 1 - (__builtin_amdgcn_readlane(at, 1) + __popcll(m1 & lt)) : __builtin_amdgcn_readlane(at, 0) + __popcll(m0 & lt);
  const int wi = __builtin_amdgcn_readlane(at, 2) + __popcll(m2 & lt);
  const int gidx = gbase + li;
  unsigned ms = kOrdNone;
  if (ok) {
    if (gidx >= x.c.qcap) atomicOr(&sm.status, kStCapacity);
    else {
      const int key = key_of(next);
      NQ[li] = make_int2(next, cb);
      if (kCl) NGI[li] = gidx;
      if (simple) ms = f2ord(__int_as_float(cb));
      if (lat_base + (unsigned)gidx >= x.lat_cap) atomicOr(&sm.status, kStLattice);
      else put_lat<kCl>(x.lat + lat_base + (unsigned)gidx, src, arc);
      if ((unsigned)next & kFlagEpsIn) {
        if (kCl ? __builtin_amdgcn_readlane(at, 3) + __popcll(m3 & lt) >= kMapMax : n_emit > kMapMax) sm.map_bad = 1;   // they (might) not fit
        else {
          unsigned s = probe_start(key);
          const unsigned step = probe_step(key);
          int probes = 0;
          while (atomicCAS(&t.keys[s], kKeyEmpty, key) != kKeyEmpty && probes < kProbeLimit) { s = (s + step) & kTabMask; ++probes; }
          if (probes >= kProbeLimit) sm.map_bad = 1;
          else { t.vals[s] = ((unsigned long long)f2ord(__int_as_float(cb)) << 32) | kRefTok | (unsigned)li; sm.tokof[s] = (unsigned short)li; }
        }
      }
    }
    // (for a token without room the entry is one that comes to nothing: infinite cost)
    if ((unsigned)next & kFlagHasEps) list_eps(x, 0, wi, gidx < x.c.qcap ? make_int4(gidx, key_of(next), cb, 1) : make_int4(0, 0, __float_as_int(INFINITY), 0));
  }
  // smallest cost in a simple state: one lane's business, and only if it gets smaller
  const unsigned cur = __hip_atomic_load(&sm.min_simple, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if (__ballot(ms < cur) != 0ull) {
    const unsigned m = wave_min(ms);
    if (lane == 0) atomicMin(&sm.min_simple, m);
  }
}

// ------------------------------------------------------------------ Prune
// Recombination of the candidates and the tokens' own self-loops, cutoff, new tokens.
//
// Usually a workgroup has at most kKR * kBlock candidates: a lane then keeps its records in registers
// from the table insert to the new token, and every candidate inside the beam is recombined.
// With more, a sample tells which bins can survive max-active (k_sel), only those are recombined, in
// as many table passes as they need, and the records are read again; a selection that turns out too
// small to decide the cutoff, or a pass that meets too many destinations, is done again (all workgroups
// of a cluster decide that from the same numbers).
// A cluster that has broken up gets no tokens: what it knows of the others' candidates and
// histograms is not complete, and places in the set come from them.
template <bool kCl, bool kProf, bool kOpt>
__device__ __forceinline__ void prune2(Cx &x, const int2 *Q, const int *GI, int2 *NQ, int *NGI, unsigned lat_base, Cutoff &cut, bool init) {
  Smem2 &sm = x.sm;
  TableLds &t = sm.u.t;
  const int tid = lane_id(), lane = tid & 63;
  const unsigned bo = uni(sm.x_best);
  cut.best = init ? 0.0f : bo == kOrdNone ? INFINITY : ord2f(bo);
  cut.beam = x.s.beam; cut.scale = x.s.scale; cut.k_keep = 256;
  const unsigned ma = (unsigned)x.s.max_active;
  const int lg = kCl ? x.lg : 0;
  // (the start token of an initialisation comes as its owner's only candidate and winner)
  const int start_mine = init && (!kCl || part_of(key_of((int)x.g.start), x.lg) == x.me);
  const int n_own = init ? start_mine : uni(sm.told[kCl ? x.xc & 1u : 0].x);
  const int n_tok = x.n;
  bool small = n_own <= kKR * kBlock;
  int k_sel = 256, n_sel = n_own + n_tok, n_sel_c = n_own;
  if (kCl && !init && n_own + uni(sm.n_in) > x.c.region_cap) {
    // One workgroup's buffer has four regions, by the top bits of the key's hash, and a channel whose
    // candidates inside the beam do not fit theirs stops.  The segments of a cluster hold more, so they
    // are counted here, all of them, but only where a region can have that many.
    unsigned *const n_reg = sm.wave_tot;
    __syncthreads();
    if (tid < kRegions) n_reg[tid] = 0;
    __syncthreads();
    for (int i0 = 0; i0 < n_own; i0 += kBlock) {
      int r = -1;
      if (i0 + tid < n_own) {
        const int4 cd = get4<kCl>(cand_at<kCl>(x, i0 + tid));
        if (cut.in_beam(__int_as_float(cd.y))) r = part_of(key_of(cd.x), kRegionBits);
      }
#pragma unroll
      for (int q = 0; q < kRegions; ++q) {
        const unsigned long long m = __ballot(r == q);
        if (lane == 0 && m) atomicAdd(&n_reg[q], (unsigned)__popcll(m));
      }
    }
    __syncthreads();
    if (tid == 0) sm.n_in = (int)max(max(n_reg[0], n_reg[1]), max(n_reg[2], n_reg[3]));
  }
  unsigned long long won = 0;
  // With more candidates than registers hold, a candidate's slot is noted: in LDS (the closure's map is free) of as many as the
  // table has slots, in registers of the next kKR * kBlock, and a bit says which of a lane's candidates have won: the records are read only
  // where they go into the table and where they become tokens.  (Without the registers two workgroups with 10,000 tokens between
  // them miss the limit in some frames: 256 utterances 61.4 instead of 60.4 ms.)
  bool noted = false;
  unsigned long long won_c = 0;
  // A pass reads the candidates of a part of the keys: one workgroup's four regions are parts of their own (or two and two),
  // the segments of a cluster are one.
  int parts = 1;
  auto part_at = [&](int j) { return j == parts ? n_own : kCl ? 0 : uni(sm.seg_lo[j * (kRegions / parts)]); };
  // Where the lane's candidate number k lies (a bit of won_c each, part by part).
  auto place_of = [&](int k) {
    if (kCl) return k * kBlock + tid;
    int at = 0;
    for (int j = 0; j < parts; ++j) {
      const int r0 = part_at(j), n_it = (part_at(j + 1) - r0 + kBlock - 1) / kBlock;
      at = r0 + k * kBlock + tid;
      if (k < n_it) break;
      k -= n_it;
    }
    return at;
  };
  int k_noted = 0;                                 // bits used
  // the lane's records, one per kBlock candidates: picked by a rolled loop (its body is large)
  static_assert(kKR == 3, "three named records");
  int4 rec0 = make_int4(0, 0, 0, 0), rec1 = rec0, rec2 = rec0; int slot0 = -1, slot1 = -1, slot2 = -1;
  auto rec_at = [&](int k) { return k == 0 ? rec0 : k == 1 ? rec1 : rec2; };
  auto slot_at = [&](int k) { return k == 0 ? slot0 : k == 1 ? slot1 : slot2; };
  auto set_slot = [&](int k, int v) { if (k == 0) slot0 = v; else if (k == 1) slot1 = v; else slot2 = v; };
  if (init) {
    rec0 = make_int4((int)x.g.start, 0, -1, -1); slot0 = tid == 0 ? 0 : -1;
    if (tid == 0) { sm.n_emit = start_mine; sm.gbase = 0; sm.n_emit_all = 1; sm.k_keep = 256; }
    __syncthreads();
  } else if (small) {
    if (tid < n_own) rec0 = get4<kCl>(cand_at<kCl>(x, tid));
    if (kBlock + tid < n_own) rec1 = get4<kCl>(cand_at<kCl>(x, kBlock + tid));
    if (2 * kBlock + tid < n_own) rec2 = get4<kCl>(cand_at<kCl>(x, 2 * kBlock + tid));
  } else if (n_own > kGroupTarget) {
    // ---- select: bins of the implied candidates, and of a sample of the others (one run of 64 in 2^sel_shift)
    if (tid < 256) { sm.hist2[tid] = 0; sm.hist3[tid] = 0; }
    __syncthreads();
    for (int i = tid; i < n_tok; i += kBlock) {
      const int2 q = Q[i];
      const float nc = stay_cost2(x, __int_as_float(q.y));
      const int in = (int)(((unsigned)q.x & kFlagSimple) != 0) | (int)((sm.v.s.hasstay[i >> 5] >> (i & 31)) & 1u);
      if (in & (int)(nc < INFINITY) & (int)cut.in_beam(nc)) atomicAdd(&sm.hist3[cut.bin(nc)], 1u);
    }
    const int sh = x.c.sel_shift;
    int n_sampled = 0;
    for (int i0 = (tid >> 6) << 6; (i0 << sh) < n_own; i0 += kBlock) {
      const int i = (i0 << sh) + lane;
      if (i < n_own) {
        const float c = __int_as_float(get4<kCl>(cand_at<kCl>(x, i)).y);
        if (cut.in_beam(c)) atomicAdd(&sm.hist2[cut.bin(c)], 1u);
      }
    }
    n_sampled = ((n_own >> (6 + sh)) << 6) + min(n_own & ((64 << sh) - 1), 64);
    __syncthreads();
    if (tid < 64) {
      const float up = (float)max(1, n_own) / (float)max(1, n_sampled);
      float hb[4]; unsigned hs[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) { hs[j] = sm.hist3[4 * tid + j]; hb[j] = (float)sm.hist2[4 * tid + j] * up; }
      const unsigned s = hs[0] + hs[1] + hs[2] + hs[3] + (unsigned)(hb[0] + hb[1] + hb[2] + hb[3]);
      const unsigned inc = wave_scan_add(s);
      const unsigned n_in = (unsigned)__builtin_amdgcn_readlane((int)inc, 63);
      // keys are shared out by hash: a workgroup's part of max_active, and some room for chance
      const float want = (float)ma * x.s.sel_ratio / (float)(kCl ? x.G : 1) + 256.0f;
      const unsigned target = want < 2.0e9f ? (unsigned)want : 2000000000u;
      int ks = 256; unsigned nsel = (unsigned)(n_own + n_tok), nsel_c = (unsigned)n_own;
      if (n_in > target) {
        float run = (float)(inc - s), run_c = 0.0f;
        int first = 256; float at = 0.0f, at_c = 0.0f;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          run += (float)hs[j] + hb[j]; run_c += hb[j];
          if (run >= (float)target && first == 256) { first = 4 * tid + j; at = run; at_c = run_c; }
        }
        const int fm = (int)wave_min((unsigned)first);
        const int owner = __ffsll((long long)__ballot(first == fm && fm != 256)) - 1;
        if (owner >= 0) {
          const float lane_c = hb[0] + hb[1] + hb[2] + hb[3];
          const float before_c = (float)wave_sum((tid & 63) < owner ? (unsigned)lane_c : 0u);
          nsel = (unsigned)__shfl(at, owner, 64);
          nsel_c = min((unsigned)n_own, (unsigned)(before_c + __shfl(at_c, owner, 64)));
          ks = fm + 1;                                   // bins [0, ks) are selected
        }
      }
      if (tid == 0) { sm.k_sel = ks; sm.n_sel = (int)nsel; sm.n_sel_c = (int)nsel_c; }
    }
    __syncthreads();
    k_sel = uni(sm.k_sel); n_sel = uni(sm.n_sel); n_sel_c = uni(sm.n_sel_c);
  }
  mark<kProf>(x, kPhSelect);

  int mult = 1;
  for (int attempt = 0; !init; ++attempt) {
    // ---- table passes over sub-groups of the keys; with the records in registers there is one, of everything in the beam
    // (One pass up to 6,144 candidates, a load of 0.75 if no two go to one state: with up to 5,120 and 4,096 a batch of 256 took 61.7
    // and 61.5 instead of 60.5 ms; with up to 7,168 and 8,192 it was the same, but six batches in flight 300.8 and 313.6 instead of 297.9.)
    int P = small || (n_sel_c <= kGroupTarget && mult == 1) ? 1 : min(2048, (int)((float)n_sel_c * 1.15f / (float)kGroupTarget + 1.0f) * mult);
    // (one workgroup: whole regions, two at a time if two passes will do, so that a pass reads only its own; with four
    // passes where two do, and the winners copied, six batches of 256 in flight took 309 instead of 302 ms)
    if (!kCl && P > 2) P = (P + kRegions - 1) / kRegions * kRegions;
    parts = kCl ? 1 : min(P, kRegions);
    won = 0; won_c = 0; k_noted = 0;
    noted = !small;
    for (int j = 0; j < parts && noted; ++j) {
      const int n_part = part_at(j + 1) - part_at(j);
      noted = n_part <= kNotes;
      k_noted += (n_part + kBlock - 1) / kBlock;
    }
    static_assert(kNotes * kRegions <= 64 * kBlock, "a bit per candidate of a lane");
    for (int g = 0; g < P; ++g) {
      if (g > 0) { clear_table(sm); __syncthreads(); }       // (before the first it is clear)
      mark<kProf>(x, kPhTabClear);
      const int part = g / (P / parts), r0 = part_at(part), r1 = part_at(part + 1);
      int4 nxt = make_int4(0, 0, 0, 0);
      if (!small && r0 + tid < r1) nxt = get4<kCl>(cand_at<kCl>(x, r0 + tid));
      int2 tok0 = make_int2(0, 0);                 // (on its way while the table is filled)
      if (tid < n_tok) tok0 = Q[tid];
#pragma unroll 1
      for (int k = 0, i0 = r0; i0 < r1; ++k, i0 += kBlock) {
        const int i = i0 + tid;
        const int4 cd = small ? rec_at(k) : nxt;
        if (!small && i + kBlock < r1) nxt = get4<kCl>(cand_at<kCl>(x, i + kBlock));
        const float c = __int_as_float(cd.y);
        const int key = key_of(cd.x);
        int take = (int)(i < r1) & (int)cut.in_beam(c) & (int)(cut.bin(c) < k_sel) & (int)((P == 1) | (group2(key, lg, P) == g));
        int sl = -1;
        if (take) sl = insert2<kCl, false>(x, key, c, cd.w, cd.z, i, nullptr, 0u);
        if (small) set_slot(k, sl);
        else if (noted) {
          if (k * kBlock < kTabSlots) { if (i < r1) sm.tokof[i - r0] = (unsigned short)sl; }
          else if (k == kTabSlots / kBlock) slot0 = sl;
          else if (k == kTabSlots / kBlock + 1) slot1 = sl;
          else slot2 = sl;
        }
      }
      __syncthreads();
      mark<kProf>(x, kPhTabFill);
      won |= stays2<kCl>(x, Q, tok0, cut, k_sel, g, P);
      __syncthreads();
      mark<kProf>(x, kPhSelect);
      // every candidate that was inserted looks at its slot again: the one still there has won
      if (noted) {
        int k = 0;
        for (int q = 0; q < part; ++q) k += (part_at(q + 1) - part_at(q) + kBlock - 1) / kBlock;
#pragma unroll 1
        for (int i0 = r0; i0 < r1; ++k, i0 += kBlock) {
          const int i = i0 + tid;
          unsigned sl = 0xFFFFu;
          if (i0 - r0 < kTabSlots) { if (i < r1) sl = sm.tokof[i - r0]; }
          else sl = (unsigned)slot_at((i0 - r0 - kTabSlots) / kBlock) & 0xFFFFu;
          if (sl != 0xFFFFu) {
            const unsigned long long v = t.vals[sl];
            if ((unsigned)v == (unsigned)i) { won_c |= 1ull << k; atomicAdd(&sm.hist[cut.bin(ord2f((unsigned)(v >> 32)))], 1u); }
          }
        }
        if (P > 1) __syncthreads();
        mark<kProf>(x, kPhTabScan);
        continue;
      }
      if (!small && r0 + tid < r1) nxt = get4<kCl>(cand_at<kCl>(x, r0 + tid));
#pragma unroll 1
      for (int k = 0, i0 = r0; i0 < r1; ++k, i0 += kBlock) {
        const int i = i0 + tid;
        const int4 cd = small ? rec_at(k) : nxt;
        if (!small && i + kBlock < r1) nxt = get4<kCl>(cand_at<kCl>(x, i + kBlock));
        const float c = __int_as_float(cd.y);
        int sl = -1;
        if (small) sl = slot_at(k);
        else {
          const int key = key_of(cd.x);
          if ((int)(i < r1) & (int)cut.in_beam(c) & (int)(cut.bin(c) < k_sel) & (int)((P == 1) | (group2(key, lg, P) == g))) sl = find2(sm, key);
        }
        int win[1] = {0}, wi[1];
        if (sl >= 0) win[0] = (int)((unsigned)t.vals[sl] == (unsigned)i);
        if (win[0]) atomicAdd(&sm.hist[cut.bin(c)], 1u);
        if (small) { if (!win[0]) set_slot(k, -1); }
        else {
          wave_alloc_n<1>(&sm.n_win, win, wi);
          if (win[0]) { if (wi[0] < x.win_cap) x.win[wi[0]] = cd; else atomicOr(&sm.status, kStCapacity); }
        }
      }
      if (P > 1) __syncthreads();
      mark<kProf>(x, kPhTabScan);
    }
    __syncthreads();                               // the histogram is complete, the table is free
    // ---- cutoff from the histogram of recombined tokens of the whole cluster
    if (kCl) {
      ++x.xc;
      // two bins per word, 24 bits each, and a tag of 16 bits: histogram exchanges have a number and a parity of
      // their own, so that a word always replaces the one of two such exchanges ago and a short tag is enough
      ++x.hc;
      if (tid < 128) astore(hist_of(x, x.me) + tid, ((unsigned long long)(x.hc & 0xffffu) << 48) | ((unsigned long long)sm.hist[2 * tid + 1] << 24) | sm.hist[2 * tid]);
      if (tid >= 128 && tid < 131) post(x, kBoxSel + tid - 128, tid == 128 ? (unsigned)(k_sel | (sm.overfull << 16)) : (unsigned)(tid == 129 ? n_sel : sm.n_in));
    }
    clear_table(sm);
    if (kCl) {
      // (the first wave waits for the words of selection at the same time)
      const int which = lane & 3;
      const bool mine = tid < 4 * x.G && which < 3;
      unsigned v = 0;
      if (tid < x.G * 128) {
        const unsigned long long *p = hist_of(x, tid >> 7) + (tid & 127);
        const unsigned long long *ps = box_of(x, mine ? lane >> 2 : 0) + kBoxSel + which;
        unsigned long long h = 0;
        for (int n = 0;; ++n) {
          h = aload(p);
          bool there = (unsigned)(h >> 48) == (x.hc & 0xffffu);
          if (mine) { const unsigned long long w = aload(ps); v = (unsigned)w; there &= (unsigned)(w >> 32) == x.xc; }
          if (there) break;
          if (give_up_wait(sm, n, sm.polls)) { h = 0; v = 0; break; }
        }
        // (two bins with one add; the lanes of a wave have different ones)
        const unsigned long long two = (h & 0xffffffull) | ((h >> 24) & 0xffffffull) << 32;
        atomicAdd(reinterpret_cast<unsigned long long *>(&sm.v.s.all[2 * (tid & 127)]), two);
        if ((tid >> 7) < x.me) atomicAdd(reinterpret_cast<unsigned long long *>(&sm.v.s.before[2 * (tid & 127)]), two);
      }
      if (tid < 64) {
        const unsigned ks = wave_min(mine && which == 0 ? v & 0xffffu : 256u);
        const unsigned over = __ballot(mine && which == 0 && (v >> 16) != 0) != 0ull;
        const unsigned ns = wave_sum(mine && which == 1 ? v : 0u);
        if (x.G == kMaxG) v += (unsigned)__shfl_xor((int)v, 4, 64);    // two workgroups to a region
        const unsigned long long crowded = __ballot(mine && which == 2 && v > (unsigned)x.c.region_cap);
        if (lane == 0 && crowded) atomicOr(&sm.status, kStCapacity);
        if (lane == 0) { sm.k_sel = (int)ks; sm.overfull = (int)over; sm.n_sel = (int)ns; }
      }
      __syncthreads();
    }
    if (tid < 64) {
      const int ks = kCl ? sm.k_sel : k_sel, ns = kCl ? sm.n_sel : n_sel;
      // (sums that the lanes have made as the histograms came; read histogram by histogram, one wave took 1.5 us for this)
      auto bins4 = [&](const unsigned (&b)[256]) { return *reinterpret_cast<const uint4 *>(&b[4 * tid]); };
      const uint4 own4 = bins4(sm.hist);
      uint4 all4 = own4, before4 = make_uint4(0, 0, 0, 0);
      if (kCl) { all4 = bins4(sm.v.s.all); before4 = bins4(sm.v.s.before); }
      unsigned h[4] = {all4.x, all4.y, all4.z, all4.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) if (4 * tid + j >= ks) h[j] = 0;
      const unsigned s = h[0] + h[1] + h[2] + h[3];
      const unsigned inc = wave_scan_add(s);
      const unsigned n_u = (unsigned)__builtin_amdgcn_readlane((int)inc, 63);
      int kk = 256, redo = 0;
      if (sm.overfull) redo = 2;                     // the histogram is worth nothing: more passes
      else if (n_u > ma) {
        unsigned run = inc - s;
        int first = 256;
#pragma unroll
        for (int j = 0; j < 4; ++j) { run += h[j]; if (run > ma && first == 256) first = 4 * tid + j; }
        kk = (int)wave_min((unsigned)first);
        if (tid == 0 && (!kCl || x.me == 0)) { sm.ctr[kCtMaxAct]++; if (kk < 1) sm.ctr[kCtBin0]++; }
        if (kk < 1) kk = 1;
      } else if (ks < 256) redo = 1;                 // too many duplicates among the selected
      // the survivors of every workgroup: where its tokens start in the set, and how many
      const int lim = min(kk, ks) - 4 * tid;
      auto kept = [&](const uint4 &q) { return wave_sum((lim > 0 ? q.x : 0u) + (lim > 1 ? q.y : 0u) + (lim > 2 ? q.z : 0u) + (lim > 3 ? q.w : 0u)); };
      unsigned mine = kept(own4), before = 0, all = mine;
      if (kCl) { before = kept(before4); all = kept(all4); }
      if (kCl && sm.dead) { kk = 0; redo = 0; mine = before = all = 0; }
      if (tid == 0) {
        sm.k_keep = kk; sm.redo = redo; sm.n_emit = (int)mine; sm.gbase = (int)before; sm.n_emit_all = (int)min(all, 0x7fffffffu);
        // next frame's selection: enough candidates for max_active distinct destinations
        const float r = redo ? x.s.sel_ratio * 2.0f : ks < 256 ? 1.2f * (float)ns / (float)max(1u, n_u) : x.s.sel_ratio;
        sm.ratio = __float_as_uint(fminf(fmaxf(r, 1.2f), 16.0f));
      }
    }
    __syncthreads();
    const int redo = uni(sm.redo);
    if (redo != 2) x.s.sel_ratio = uni(__uint_as_float(sm.ratio));
    if (!redo) break;
    if (attempt >= 12) { if (tid == 0) atomicOr(&sm.status, kStCapacity); break; }   // never expected: 2048 passes
    if (tid == 0 && (!kCl || x.me == 0)) sm.prof[15]++;   // counted, not timed: re-recombinations
    if (tid < 256) { sm.hist[tid] = 0; if (kCl) { sm.v.s.all[tid] = 0; sm.v.s.before[tid] = 0; } }
    if (tid == 0) { sm.n_win = 0; sm.overfull = 0; }
    // (a table has room for what registers hold, but room is not enough: of 3,000 keys at regular distances one can have 1,000 others
    // ahead of it.  The records are then read again, and the passes are more.)
    if (redo == 2) { mult *= 2; small = false; }
    else { k_sel = 256; n_sel = n_own + n_tok; n_sel_c = n_own; }
    __syncthreads();
  }
  cut.k_keep = uni(sm.k_keep);
  mark<kProf>(x, kPhOther);

  // ---- survivors become tokens
  const int n_emit = uni(sm.n_emit), gbase = uni(sm.gbase);
  // First the candidates that won, then the tokens that stay where they are, made from the records of
  // the current set.  A third of the lanes have one at a time, and making a token is long (LDS counters, the closure's
  // table), so every wave collects 64 of them before it makes any: 32 utterances of 8.1 k tokens per frame 36.7 -> 36.0 ms,
  // 64 of 11.7 k on a graph that branches everywhere 27.9 -> 27.2 ms; where a wave has fewer than 64 in all (900 tokens per
  // frame and workgroup) it makes no difference.
  const int n_c = small ? n_own : uni(min(sm.n_win, x.win_cap));
  const int k_c = noted ? k_noted : (n_c + kBlock - 1) / kBlock, k_all = k_c + (n_tok + kBlock - 1) / kBlock;
  int4 nxt = make_int4(0, 0, 0, 0);
  auto is_winner = [&](int k) { return noted ? (int)((won_c >> k) & 1ull) : (int)(k * kBlock + tid < n_c); };
  auto fetch = [&](int k) {
    if (k < k_c) { if (!small && is_winner(k)) nxt = noted ? get4<kCl>(cand_at<kCl>(x, place_of(k))) : x.win[k * kBlock + tid]; }
    else if ((k - k_c) * kBlock + tid < n_tok) { const int i = (k - k_c) * kBlock + tid; const int2 q = Q[i]; nxt.x = q.x; nxt.y = q.y; nxt.z = kCl ? GI[i] : i; }
  };
  fetch(0);
  int4 *mk = sm.v.mk[uni(tid >> 6)];
  int n_mk = 0;
#pragma unroll 1
  for (int k = 0; k <= k_all; ++k) {
    int4 cr = k < k_c && small ? rec_at(k) : nxt;
    int ok = 0;
    if (k < k_all) {
      fetch(k + 1);
      if (k < k_c) ok = small ? (int)(slot_at(k) >= 0) : is_winner(k);
      else {
        ok = (int)((won >> (k - k_c)) & 1ull);
        cr.y = __float_as_int(stay_cost2(x, __int_as_float(cr.y)));
        cr.z |= (int)((((unsigned)cr.x & kKeyMask) >> x.g.blk_bits) << 16);
        cr.w = 2 * (int)((unsigned)cr.x & x.g.blk_mask) + 1;     // the self-loop: the unit after the header
      }
      ok &= (int)(cut.bin(__int_as_float(cr.y)) < cut.k_keep);
    }
    const unsigned long long m = __ballot(ok);
    const int at = n_mk + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    if (ok && at < 64) mk[at] = cr;
    n_mk += __popcll(m);
    if (n_mk < (k < k_all ? 64 : 1)) continue;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int4 r = mk[lane];
    make2<kCl, kOpt>(x, (int)(lane < n_mk), r.x, r.y, r.z, r.w, cut, NQ, NGI, lat_base, n_emit, gbase);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    if (ok && at >= 64) mk[at - 64] = cr;
    n_mk -= 64;
  }
  if (kOpt && x.c.frame_best && tid == 0 && (!kCl || x.me == 0) && x.s.frame + 1 <= x.c.max_frames) {
    // the lattice kernel needs it for links across this frame's boundary
    const size_t chan = (size_t)(x.frame_off - x.c.frame_off) / (size_t)(x.c.max_frames + 2);
    x.c.frame_best[chan * (size_t)(x.c.max_frames + 1) + (size_t)x.s.frame + 1] = uni(sm.n_emit_all) > 0 ? cut.best : 0.0f;
  }
  if (kOpt && x.c.cost_offset && uni(sm.n_emit_all) > 0) {   // the stored costs are relative to this frame's best from here on
    x.s.offset = uni(x.s.offset + (double)cut.best);
    cut.best = 0.0f;
  }
  __syncthreads();
  x.n_front = uni(sm.made[0]); x.n_emit = n_emit;
  if (tid == 0) {
    sm.n_loc = n_emit; if (!init) count2(sm, kCtKept, min(n_emit, x.c.qcap));
    if (kCl && x.me == 0) set_counter(x, sm.n_emit_all);
  }
  if (tid < 256) sm.hist[tid] = 0;
  mark<kProf>(x, kPhCutoff);
}

// ------------------------------------------------------------------ epsilon closure
// One candidate that is its destination's best (win[u]): a token the set has takes its cost and
// backpointer, a destination without one gets a token; either way it is expanded in the next round.
// `full`: the workgroup had as many tokens as a set holds when the round began.
// All lanes of the wave call it.
template <bool kCl>
__device__ __forceinline__ void apply2(Cx &x, int win, const int4 &rec, int slot, int2 *NQ, int *NGI, unsigned lat_base, int sel, bool full) {
  Smem2 &sm = x.sm;
  TableLds &t = sm.u.t;
  const int lane = lane_id() & 63;
  const unsigned long long lt = (1ull << lane) - 1ull;
  if (__ballot(win) == 0ull) return;
  int li = win ? (int)sm.tokof[slot] : 0, gx = 0;
  int fresh = win & (int)(li == 0xFFFF);
  const unsigned long long mn = __ballot(fresh), mw = __ballot(win & (int)((unsigned)rec.x >> 31));
  // places: lane 0 takes the new tokens' local numbers, lane 1 the worklist's, lane 2 the numbers in the set (from
  // the cluster's counter)
  int at = 0;
  if (lane == 0 && mn) at = atomicAdd(&sm.n_loc, __popcll(mn));
  if (lane == 1 && mw) at = atomicAdd(&sm.made[2], __popcll(mw));
  if (kCl && lane == 2 && mn) at = (int)__hip_atomic_fetch_add(set_size_of(x), (unsigned)__popcll(mn), __ATOMIC_RELAXED, kStoreScope);
  const int rank = __popcll(mn & lt);
  if (fresh) { li = __builtin_amdgcn_readlane(at, 0) + rank; gx = kCl ? __builtin_amdgcn_readlane(at, 2) + rank : li; }
  else if (win) {
    gx = kCl ? uni(sm.gbase) + li : li;
    if (kCl && li >= x.n_emit) gx = NGI[li];     // (made by the closure)
  }
  unsigned ms = kOrdNone;
  if (win) {
    bool room = gx < x.c.qcap && li < x.c.qcap;
    // (the last token of a full set has the number that stands for none: there is no room for a new one, but it may be meant)
    if (full && fresh && key_of(NQ[kQueueMax - 1].x) == key_of(rec.x)) {
      li = kQueueMax - 1; gx = kCl ? NGI[li] : li;
      fresh = 0; room = gx < x.c.qcap;
    }
    if (!room) atomicOr(&sm.status, kStCapacity);
    else {
      if (fresh) { NQ[li] = make_int2(rec.x, rec.y); if (kCl) NGI[li] = gx; }
      else NQ[li].y = rec.y;
      if (lat_base + (unsigned)gx >= x.lat_cap) atomicOr(&sm.status, kStLattice);
      else put_lat<kCl>(x.lat + lat_base + (unsigned)gx, rec.z, rec.w);
      t.vals[slot] = ((unsigned long long)f2ord(__int_as_float(rec.y)) << 32) | kRefTok | (unsigned)li;
      sm.tokof[slot] = (unsigned short)li;
      if ((unsigned)rec.x & kFlagSimple) ms = f2ord(__int_as_float(rec.y));
    }
    if ((unsigned)rec.x & kFlagHasEps) {
      const int wi = __builtin_amdgcn_readlane(at, 1) + __popcll(mw & lt);
      list_eps(x, sel, wi, room ? make_int4(gx, key_of(rec.x), rec.y, fresh) : make_int4(0, 0, __float_as_int(INFINITY), 0));
    }
  }
  const unsigned cur = __hip_atomic_load(&sm.min_simple, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  if (__ballot(ms < cur) != 0ull) {
    const unsigned m = wave_min(ms);
    if (lane == 0) atomicMin(&sm.min_simple, m);
  }
}

// Candidates of kU arcs per lane over epsilon arcs.
template <bool kCl>
__device__ __forceinline__ void emit_eps2(Cx &x, int (&ok)[kU], const float (&tc)[kU], const int (&src)[kU], int (&arc)[kU],
                                          const Cutoff &cut, bool boosted, int buf) {
  int next[kU]; float nc[kU]; int4 a[kU]; int more = 0;
#pragma unroll
  for (int u = 0; u < kU; ++u) { a[u] = make_int4(0, 0, 0, 0); if (ok[u]) a[u] = x.g.unit[arc[u]]; }
#pragma unroll
  for (int u = 0; u < kU; ++u) {
    nc[u] = canon(tc[u] + __int_as_float(a[u].y));
    next[u] = a[u].x; arc[u] |= (int)kArcEps;
    if (boosted) {                           // epsilon arcs can carry output labels too
      const int b = (int)((unsigned)src[u] >> 16);
      int nb = b;
      if (ok[u] && a[u].w != 0) nc[u] = canon(nc[u] + boost_step2(x.sm, b, a[u].w, nb));
      next[u] |= nb << x.g.blk_bits;
    }
    ok[u] &= (int)(nc[u] < INFINITY) & (int)cut.keep(nc[u]);
    more |= ok[u] & (int)((unsigned)next[u] >> 31);
  }
  if (__ballot(more) != 0ull) x.sm.more = 1;
  push_cands2<kCl, kU>(x, ok, next, nc, src, arc, buf);
}

// Least fixpoint under the frozen predicate `cut`.  The worklist holds the tokens created or
// improved in the previous round that have epsilon arcs.  The set's tokens that an epsilon arc can
// enter sit in the LDS table (put there when they were made), so a round's candidates meet them
// directly.  If they do not fit, every round's candidates go into an empty table and all tokens look
// themselves up.  On entry the first worklist holds sm.made[2] entries: kWlLds in sm.wl[0], the others in wl0.
//
// A round is bound by its chain (worklist, state, arcs, exchange, table, tokens), and every barrier adds to that the
// wait for the slowest of 16 waves.  So each wave flattens the arcs of its own items (a flattening
// over the block took three barriers more), and where no candidate's state has epsilon arcs the
// round is the last, without one to find that out.  What only that exchange would tell, the size of the
// set, comes with the next frame's first one: returns true if it is still to come (never with `last`, a launch's last frame).
// The two sets of segments are used in turn, also from one frame to the next: what another workgroup may still be reading
// when a frame ends is not what the next frame's arcs are written to.
// (One utterance of 10.8 k tokens per frame 10.57 -> 9.93 ms, of 900 tokens 2.03 -> 1.90 ms, 64 on a graph that branches
// everywhere 30.1 -> 28.4 ms.)
template <bool kCl, bool kBoost, bool kProf>
__device__ __forceinline__ bool closure2(Cx &x, int2 *NQ, int *NGI, unsigned lat_base, const Cutoff &cut, bool last) {
  Smem2 &sm = x.sm;
  TableLds &t = sm.u.t;
  const int tid = lane_id(), lane = tid & 63, wave = uni(tid >> 6);
  const bool boosted = kBoost && x.s.boost_n > 0;
  const int lg = kCl ? x.lg : 0;
  for (int round = 1;; ++round) {
    const int sel = (round - 1) & 1, buf = kCl ? seg_set(x) ^ 1 : 0;
    const int n_wl = uni(min(sm.made[2], x.c.qcap));
    if (!kCl && n_wl == 0) { __syncthreads(); break; }        // (the size of the set is known)
    if (n_wl > 0) {                                           // (with nothing to do, what the others have is asked for at once)
      // ---- every wave expands items of its own; at least four, so that short lists don't keep all waves busy
      const int size = min(kEpsTok, max(4, (n_wl + kWaves - 1) / kWaves));
      WaveEps &we = sm.v.ek.w[wave];
      unsigned xsum = 0;
      for (int r = wave; r * size < n_wl; r += kWaves) {
        const int i = r * size + lane;
        int4 w = make_int4(0, 0, 0, 0);
        unsigned deg = 0;
        if (lane < size && i < n_wl) {
          w = sm.wl[sel][min(i, kWlLds - 1)];                   // w.y is the token's key: (state in B, block)
          asm volatile("" : "+v"(w.x), "+v"(w.y), "+v"(w.z), "+v"(w.w));     // (or both would be one load of a generic address)
          if (i >= kWlLds) w = (x.wl0 + sel * x.c.qcap)[i];
          deg = (unsigned)x.g.unit[2 * (size_t)((unsigned)w.y & x.g.blk_mask)].w >> kPackXShift;   // the state's header
        }
        int first = 2 * (int)((unsigned)w.y & x.g.blk_mask) + 1;
        const float cost = __int_as_float(w.z);                 // the token's cost when it was listed
        const int src = w.x | (int)(((unsigned)w.y >> x.g.blk_bits) << 16);
        xsum += w.w ? deg : 0u;
        if (deg > (unsigned)kEpsDeg) {                          // to the shared list, as far as it has room
          const int n = ((int)deg + kEpsSeg - 1) / kEpsSeg;
          const int h = atomicAdd(&sm.n_eseg, n), fit = max(0, min(n, kEpsSegs - h));
          for (int q = 0; q < fit; ++q, first += kEpsSeg) {
            sm.v.ek.seg[h + q] = WaveItem{first, cost, src, min(kEpsSeg, (int)deg)};
            deg -= min((unsigned)kEpsSeg, deg);
          }
        }
        do {
          const unsigned take = min(deg, (unsigned)kEpsDeg);
          const int M = list_items(we, take, first, cost, src);
          for (int f0 = 0, q = 0, before = 0; f0 < M; f0 += 64 * kU) {
            int ok[kU], isrc[kU], arc[kU]; float tc[kU];
#pragma unroll
            for (int u = 0; u < kU; ++u) {
              const int f = f0 + u * 64 + lane;
              const WaveItem it = item_of(we, q++, before);
              ok[u] = f < M; isrc[u] = it.src; tc[u] = it.tcost; arc[u] = it.abase + f;
            }
            emit_eps2<kCl>(x, ok, tc, isrc, arc, cut, boosted, buf);
          }
          __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
          __builtin_amdgcn_wave_barrier();
          deg -= take; first += (int)take;
        } while (__ballot(deg != 0) != 0ull);
      }
      // epsilon arcs out of the set (a counter): every token is listed as new exactly once
      xsum = wave_sum(xsum);
      if (lane == 0 && xsum) atomicAdd((unsigned long long *)&sm.ctr[kCtXarc], (unsigned long long)xsum);
      if (kCl) stores_done();
      __syncthreads();
      const int n_seg = uni(min(sm.n_eseg, kEpsSegs));
      if (n_seg > 0) {                                          // ---- segments of states with many arcs
        for (int q = wave; q < n_seg; q += kWaves) {
          const WaveItem it = sm.v.ek.seg[q];
          int ok[kU], isrc[kU], arc[kU]; float tc[kU];
#pragma unroll
          for (int u = 0; u < kU; ++u) { ok[u] = u * 64 + lane < it.pad; isrc[u] = it.src; tc[u] = it.tcost; arc[u] = it.abase + u * 64 + lane; }
          emit_eps2<kCl>(x, ok, tc, isrc, arc, cut, boosted, buf);
        }
        if (kCl) stores_done();
        __syncthreads();
        if (tid == 0) sm.n_eseg = 0;
      }
    } else if (kCl && round == 1) stores_done();              // (nothing to expand: the set's counter alone)
    if (tid == 0) sm.made[2] = 0;
    mark<kProf>(x, kPhEpsExpand);
    post_sizes<kCl>(x);
    take_sizes<kCl>(x);
    // An overflow (or a cluster that has broken up) ends the closure, and with the frame the channel: a token that
    // found no room has left the number of its candidate in the table, which would now be looked for among this
    // round's candidates.
    const int2 told = sm.told[kCl ? x.xc & 1u : 0];
    const int n_own = uni(told.x), what = uni(told.y);
    if (what & 1) break;
    const bool more = (what & 2) != 0;
    mark<kProf>(x, kPhEpsRecombine);
    if (n_own > 0) {
      const int n_map = uni(sm.made[3]), n_loc0 = uni(sm.n_loc);
      // (in the map as long as it may do: half of the candidates new ones; if they are more than it holds, the round begins again.
      // One workgroup takes it only for as many as it has room for; with that rule in clusters one utterance took 8.83 instead of 8.74
      // ms and a stream 4.79 instead of 4.74.  Room is not enough: of 6,144 keys at regular distances, as the states of a
      // list have them, some find no free slot within kProbeLimit probes in up to 97 of 100 orders.)
      bool map = !uni(sm.map_bad) && (kCl ? n_map + n_own / 2 <= kTabSlots * 7 / 8 : n_map + n_own <= kMapMax);
      int P = map ? 1 : max(1, (n_own + kGroupTarget - 1) / kGroupTarget);
      for (int g = 0; g < P; ++g) {
        if (!map) {
          __syncthreads();
          clear_table(sm);
          if (tid == 0) { sm.map_bad = 1; sm.overfull = 0; }
          __syncthreads();
        }
        // a lane's first candidate stays in registers (usually it is the only one)
        int4 rec0 = make_int4(0, 0, 0, 0); int slot0 = -1;
#pragma unroll 1
        for (int i0 = 0; i0 < n_own; i0 += kBlock) {
          if (map && i0 > 0 && uni(sm.overfull)) break;
          const int i = i0 + tid;
          int4 cd = make_int4(0, 0, 0, 0); int sl = -1;
          if (i < n_own) {
            cd = get4<kCl>(cand_at<kCl>(x, i));
            const int key = key_of(cd.x);
            if (P == 1 || group2(key, lg, P) == g) sl = insert2<kCl, true>(x, key, __int_as_float(cd.y), cd.w, cd.z, i, NGI, lat_base);
          }
          if (i0 == 0) { rec0 = cd; slot0 = sl; }
        }
        __syncthreads();
        if (map && __builtin_expect(uni(sm.overfull), 0)) {     // some destination found no slot: without the map, from the start
          map = false; P = max(1, (n_own + kGroupTarget - 1) / kGroupTarget); g = -1;
          continue;
        }
        if (!map) {
          if (uni(sm.overfull) && P < 4096) {      // more destinations than planned: smaller sub-groups, from the start
            // (nothing has been applied for this sub-group yet; what the earlier ones applied does not beat itself)
            __syncthreads();
            P *= 2; g = -1;
            continue;
          }
          // the set's tokens look their keys up: a token whose key is there stays if it is the better
          // one, and otherwise is the one that improves
          const int n_now = uni(min(sm.n_loc, x.c.qcap));
          int2 nxt = make_int2(0, 0);
          if (tid < n_now) nxt = NQ[tid];
          for (int i = tid; i < n_now; i += kBlock) {
            const int2 q = nxt;
            if (i + kBlock < n_now) nxt = NQ[i + kBlock];
            const int key = key_of(q.x);
            const int sl = ((unsigned)q.x & kFlagEpsIn) ? find2(sm, key) : -1;
            if (sl < 0) continue;
            const unsigned long long v = t.vals[sl];
            const unsigned oc = f2ord(__int_as_float(q.y)), cc = (unsigned)(v >> 32);
            bool stays = oc < cc;
            if (oc == cc) {
              const int4 cd = get4<kCl>(cand_at<kCl>(x, (int)(unsigned)v));
              const unsigned at = (unsigned)(kCl ? NGI[i] : i);
              const int2 bp = at < (unsigned)x.c.qcap && lat_base + at < x.lat_cap ? get_lat<kCl>(x.lat + lat_base + at) : make_int2(0, 0);
              stays = !((unsigned)cd.w < (unsigned)bp.y || (cd.w == bp.y && ((unsigned)cd.z >> 16) < ((unsigned)bp.x >> 16)));
            }
            if (stays) t.vals[sl] = ((unsigned long long)oc << 32) | kRefTok | (unsigned)i;
            sm.tokof[sl] = (unsigned short)i;
          }
          __syncthreads();
        }
        mark<kProf>(x, kPhEpsTabFill);
#pragma unroll 1
        for (int i0 = 0; i0 < n_own; i0 += kBlock) {
          const int i = i0 + tid;
          int4 cd = rec0; int sl = slot0, win = 0;
          if (i0 > 0) {
            sl = -1;
            if (i < n_own) {
              cd = get4<kCl>(cand_at<kCl>(x, i));
              const int key = key_of(cd.x);
              if (P == 1 || group2(key, lg, P) == g) sl = find2(sm, key);
            }
          }
          if (sl >= 0) win = (int)((unsigned)t.vals[sl] == (unsigned)i);
          apply2<kCl>(x, win, cd, sl, NQ, NGI, lat_base, sel ^ 1, n_loc0 >= kQueueMax && x.c.qcap == kQueueMax);
        }
        __syncthreads();
        mark<kProf>(x, kPhEpsTabScan);
      }
      if (tid == kResetTid && map) sm.made[3] = n_map + uni(sm.n_loc) - n_loc0;
    }
    if (!more && !(kCl && last)) { mark<kProf>(x, kPhEpsRecombine); return kCl; }
  }
  mark<kProf>(x, kPhEpsRecombine);
  return false;
}

// The closed token set becomes A_f (f = x.s.frame): the workgroup's own part of that.  `bad`: some tokens found no room, and
// were not written or have a number beyond the arena.
template <bool kCl, bool kOpt>
__device__ __forceinline__ void finish2(Cx &x, const int2 *NQ, const int *NGI, int n_loc, unsigned lat_base, bool bad) {
  Smem2 &sm = x.sm;
  const int tid = lane_id();
  const int n = min(n_loc, x.c.qcap);
  const int f = x.s.frame;
  if (kOpt && !bad) {
    if (x.dig_sum && f <= x.c.max_frames) {
      unsigned long long s = 0;
      for (int i = tid; i < n; i += kBlock) {
        const int2 sc = NQ[i];
        const int state = x.g.unit[2 * (size_t)((unsigned)sc.x & x.g.blk_mask)].x;     // the header names the state
        const unsigned b = ((unsigned)sc.x & kKeyMask) >> x.g.blk_bits;   // the token's state in the boosting acceptor
        s += mix64((((unsigned long long)(unsigned)state << 32) | (unsigned)sc.y) ^ ((unsigned long long)b * 0x9E3779B97F4A7C15ull));
      }
      if (s) atomicAdd(&x.dig_sum[f], s);        // (zeroed when the launch began)
    }
    if (x.c.tokrec) {                              // lattice output wants the closed set's final records
      int2 *rec = x.c.tokrec + (x.lat - x.c.lattice) + lat_base;
      for (int i = tid; i < n; i += kBlock) {
        const int2 q = NQ[i]; const unsigned at = (unsigned)(kCl ? NGI[i] : i);
        if (lat_base + at < x.lat_cap) rec[at] = make_int2((int)((unsigned)q.x & (kKeyMask | kFlagSimple)), q.y);
      }
    }
  }
  if (tid == kStoredTid) count2(sm, kCtStored, n);
  x.s.cur ^= 1;
  x.n = n;
}
// Its size and its place in the lattice: the newest set's, which starts at x.s.lat_used.
template <bool kCl, bool kOpt>
__device__ __forceinline__ void publish2(Cx &x, bool stop) {
  const Smem2 &sm = x.sm;
  const unsigned lat_base = x.s.lat_used;
  const int total = uni(min(sm.n_emit_all + (kCl ? sm.x_made : sm.n_loc - x.n_emit), x.c.qcap));
  const int f = x.s.frame;
  if (threadIdx.x == kPublishTid && (!kCl || x.me == 0)) {
    const int F = x.c.max_frames + 2;            // the per-frame tables are rings (a recycled channel outlives them)
    x.frame_off[ring_at(f, F)] = lat_base;
    x.frame_off[ring_at(f + 1, F)] = lat_base + (unsigned)total;
    x.c.frame_ep[(x.frame_off - x.c.frame_off) + ring_at(f, F)] = x.s.lat_epoch;
    if (kOpt && !stop && x.dig_sum && f <= x.c.max_frames) x.dig_cnt[f] = total;
  }
  x.s.lat_used = lat_base + (unsigned)total;
  x.s.n_tok = total;
}

// ------------------------------------------------------------------ final choice + traceback
// Best token by (cost + final cost, state) if any token is final, else by (cost, state)
// (block numbers grow with state ids, so they order the same way);
// then the backpointers are followed to the start token and the non-zero output labels of
// the arcs are written in path order.
template <bool kCl>
__device__ __forceinline__ void trace2(Cx &x, const LaunchArgs &a, int io, const int2 *Q, const int *GI) {
  Smem2 &sm = x.sm;
  const int tid = lane_id(), lane = tid & 63;
  const int n = x.n;
  int *words = a.words + (long long)io * a.max_words;
  int flags = x.s.status;
  if (x.s.n_tok == 0) {
    if (tid == 0 && (!kCl || x.me == 0)) { a.nwords[io] = 0; a.cost[io] = INFINITY; a.flags[io] = flags | WFST_FLAG_DEAD; }
    return;
  }
  if (tid == 0) { sm.red64 = ~0ull; sm.red64b = ~0ull; sm.sel_idx = -1; sm.trace_from = -1; }
  __syncthreads();
  // ties go to the lower graph state, then to the lower state of the boosting acceptor: the key
  // (B state, block) is turned round for the comparison
  const int bbits = x.g.blk_bits, sbits = 29 - x.g.blk_bits; const unsigned bm = x.g.blk_mask;
  unsigned long long mf = ~0ull, mr = ~0ull;
  for (int i = tid; i < n; i += kBlock) {
    const int2 t = Q[i];
    const float c = __int_as_float(t.y);
    const unsigned blk = (unsigned)t.x & bm, turned = (blk << sbits) | (((unsigned)t.x & kKeyMask) >> bbits);
    mr = min(mr, ((unsigned long long)f2ord(c) << 32) | turned);
    if (a.finalize) {
      const float fc = x.g.has_final ? __int_as_float(x.g.unit[2 * (size_t)blk].y) : 0.0f;
      const float f = c + fc;
      if (f < INFINITY) mf = min(mf, ((unsigned long long)f2ord(f) << 32) | turned);
    }
  }
  if (mf != ~0ull) atomicMin(&sm.red64, mf);
  if (mr != ~0ull) atomicMin(&sm.red64b, mr);
  __syncthreads();
  {
    // number in the set of the workgroup's best final token (sel_idx) and best token (trace_from)
    const unsigned long long bf = sm.red64, br = sm.red64b;
    for (int i = tid; i < n; i += kBlock) {
      const unsigned key = (unsigned)key_of(Q[i].x), turned = ((key & bm) << sbits) | (key >> bbits);
      if (bf != ~0ull && turned == (unsigned)bf) sm.sel_idx = kCl ? GI[i] : i;
      if (br != ~0ull && turned == (unsigned)br) sm.trace_from = kCl ? GI[i] : i;
    }
  }
  if (kCl) stores_done();                        // the backpointers the first workgroup is going to read
  __syncthreads();
  if (kCl) {
    ++x.xc;
    if (tid < 6) post(x, tid, tid == 0 ? (unsigned)(sm.red64 >> 32) : tid == 1 ? (unsigned)sm.red64 : tid == 2 ? (unsigned)(sm.red64b >> 32)
                               : tid == 3 ? (unsigned)sm.red64b : tid == 4 ? (unsigned)sm.sel_idx : (unsigned)sm.trace_from);
    if (x.me != 0) return;
    if (tid < 64) {
      unsigned v = 0;
      const int r = lane >> 3, wd = lane & 7;
      if (r < x.G && wd < 6) v = poll(sm, box_of(x, r) + wd, x.xc);
      unsigned long long bf = ~0ull, br = ~0ull; int jf = -1, jr = -1;
      for (int q = 0; q < x.G; ++q) {
        const unsigned long long f = ((unsigned long long)(unsigned)__shfl((int)v, q * 8) << 32) | (unsigned)__shfl((int)v, q * 8 + 1);
        const unsigned long long r2 = ((unsigned long long)(unsigned)__shfl((int)v, q * 8 + 2) << 32) | (unsigned)__shfl((int)v, q * 8 + 3);
        const int fi = __shfl((int)v, q * 8 + 4), ri = __shfl((int)v, q * 8 + 5);
        if (f < bf) { bf = f; jf = fi; }
        if (r2 < br) { br = r2; jr = ri; }
      }
      __builtin_amdgcn_wave_barrier();
      if (lane == 0) { sm.red64 = bf; sm.red64b = br; sm.sel_idx = jf; sm.trace_from = jr; }
    }
    __syncthreads();
    if (uni(sm.dead)) return;                    // (the entry will be reported as lost)
  }
  const bool any_final = sm.red64 != ~0ull;
  const unsigned long long best = any_final ? sm.red64 : sm.red64b;
  const int first_tok = any_final ? sm.sel_idx : sm.trace_from;
  __syncthreads();
  // One lane follows the backpointers.  The words come out last to first: they go into a ring
  // in LDS (the recombination table is idle now) that keeps the latest max_words of them, i.e.
  // the first max_words of the path, and all lanes then write them out in path order.  Only
  // when max_words exceeds the ring is the chain walked twice (count, then write).
  // The walk is incremental: the previous traceback of the channel left, per frame, the token
  // with which its path entered that frame's set and the number of words up to there, and
  // its words.  Backpointers of stored frames never change, so when the new walk reaches such a
  // token the rest of the path is the old one: the walk stops and the old words are kept.  A
  // partial result after every chunk then costs a walk over the new frames (plus the distance
  // to where the two paths join) instead of over the whole stream.
  int *ring = sm.u.t.keys;
  const bool one_walk = a.max_words <= kTabSlots;
  const bool inc = one_walk && x.c.path_tok != nullptr && a.max_words == x.c.max_words;
  const size_t chan = (size_t)(x.frame_off - x.c.frame_off) / (size_t)(x.c.max_frames + 2);
  int *ptok = inc ? x.c.path_tok + chan * (size_t)(x.c.max_frames + 1) : nullptr;
  int *pnw = inc ? x.c.path_nw + chan * (size_t)(x.c.max_frames + 1) : nullptr;
  int *pwords = inc ? x.c.path_words + chan * (size_t)x.c.max_words : nullptr;
  if (tid == 0) {
    int nw = 0, f_stop = 0, w_stop = 0;
    bool broken = false, gone = false;
    const int F = x.c.max_frames + 2, FM = x.c.max_frames + 1;   // the per-frame tables are rings
    const int *fep = x.c.frame_ep + (x.frame_off - x.c.frame_off);
    for (int pass = one_walk ? 1 : 0; pass < 2; ++pass) {
      int f = x.s.frame, i = first_tok, k = 0;
      for (unsigned step = 0;; ++step) {
        // every chain ends at the start token; the bounds only guard against a damaged lattice
        if (f < 0 || i < 0 || step > 0x40000000u) { broken = true; break; }
        const unsigned off = x.frame_off[f % F];
        if (x.c.recycle) {
          // is the frame still there?  Its slot of the per-frame tables, and its tokens: stored in
          // this epoch, or in the one before at a place the write position has not reached again
          const int ep = fep[f % F];
          const bool here = x.s.frame - f <= x.c.max_frames &&
                            (ep == x.s.lat_epoch || (ep == x.s.lat_epoch - 1 && off >= x.s.lat_used));
          if (!here) { gone = true; break; }
        } else if (off + (unsigned)i >= x.s.lat_used) { broken = true; break; }
        const unsigned li = off + (unsigned)i;
        if (li >= x.lat_cap) { broken = true; break; }
        const int2 bp = get_lat<kCl>(x.lat + li);
        if (bp.y < 0) break;
        const bool emitting = !((unsigned)bp.y & kArcEps);
        if (inc && emitting) {
          if (f <= x.s.path_frames && ptok[f % FM] == i) { f_stop = f; w_stop = pnw[f % FM]; break; }   // the old path from here on
          ptok[f % FM] = i; pnw[f % FM] = k;        // k: words after this arc; turned into words up to it below
        }
        const int ol = x.g.unit[(unsigned)bp.y & kArcMask].w;
        if (ol != 0) {
          if (one_walk) ring[k % a.max_words] = ol;
          else if (pass == 1) { const int pos = nw - 1 - k; if (pos < a.max_words) words[pos] = ol; }
          ++k;
        }
        i = bp.x & 0xffff;                                      // (the upper half: the source's state in the boosting acceptor)
        if (emitting) --f;                                      // an emitting arc consumed a frame
      }
      nw = k;
    }
    nw += w_stop;
    if (any_final) flags |= WFST_FLAG_REACHED_FINAL;
    if (nw > a.max_words) flags |= WFST_FLAG_TRUNCATED;
    if (broken) { flags |= WFST_FLAG_CAPACITY; nw = 0; }
    // a recycled arena no longer holds the frames this path runs through before it meets the path of
    // the previous result (results were asked for too rarely for the arena's size)
    if (gone) { flags |= WFST_FLAG_LATTICE_OVERFLOW; nw = 0; broken = true; }
    a.nwords[io] = min(nw, a.max_words);
    a.cost[io] = x.c.cost_offset ? (float)((double)ord2f((unsigned)(best >> 32)) + x.s.offset) : ord2f((unsigned)(best >> 32));
    a.flags[io] = flags;
    sm.sel_idx = nw;
    sm.trace_from = f_stop; sm.trace_words = w_stop;
    sm.path_frames = (inc && !broken) ? x.s.frame : 0;
  }
  __syncthreads();
  if (one_walk) {
    const int nw = sm.sel_idx, w_stop = sm.trace_words;   // new word k of the walk (0 = last word) sits in ring[k % max_words]
    const int k_new = nw - w_stop;
    if (inc) {
      // marks of the frames walked: words after the arc -> words up to and including it
      const int FM = x.c.max_frames + 1;
      for (int f = sm.trace_from + 1 + tid; f <= x.s.frame; f += kBlock) pnw[f % FM] = nw - pnw[f % FM];
      for (int p = w_stop + tid; p < min(nw, a.max_words); p += kBlock) pwords[p] = ring[(k_new - 1 - (p - w_stop)) % a.max_words];
      __syncthreads();
      for (int p = tid; p < min(nw, a.max_words); p += kBlock) words[p] = pwords[p];
    } else {
      for (int p = tid; p < min(nw, a.max_words); p += kBlock) words[p] = ring[(nw - 1 - p) % a.max_words];
    }
  }
  __syncthreads();
}

// The next entry of the launch's list (for all workgroups of a cluster); ends with a barrier.  The first
// workgroup takes it when the others have come here too: an entry without a frame or a result has no other
// exchange, and a mailbox keeps the words of two exchanges only, so the first workgroup could be two
// entries ahead and overwrite a word that another has yet to read.  (1 us per utterance.)  A cluster
// that has broken up takes none, and the first workgroup knows behind this whether the others have
// done their part of the last entry.
template <bool kCl>
__device__ __forceinline__ int next_job2(Cx &x, const LaunchArgs &a) {
  Smem2 &sm = x.sm;
  if (kCl) {
    if (uni(sm.dead)) return a.n_jobs;
    ++x.xc;
    if (x.me == 0) {
      if (threadIdx.x > 0 && (int)threadIdx.x < x.G) poll(sm, box_of(x, threadIdx.x), x.xc);
      __syncthreads();
      if (uni(sm.dead)) return a.n_jobs;
    }
  }
  if (threadIdx.x == 0) {
    if (!kCl || x.me == 0) { sm.job = atomicAdd(a.lists + 4 * a.n_jobs, 1); if (kCl) post(x, 0, (unsigned)sm.job); }
    else { post(x, 0, 0u); sm.job = (int)poll(sm, box_of(x, 0), x.xc); }
  }
  __syncthreads();
  const int job = uni(sm.job);
  return kCl && uni(sm.dead) ? a.n_jobs : job;
}

// An entry that no cluster has finished: its channel stops, and its result says so.
__device__ __forceinline__ void report_lost(const DevChannels &c, const LaunchArgs &a, int ch, int io) {
  ChanState &s = c.st[ch];
  const int status = (a.mode & kModeInit ? 0 : s.status) | kStCapacity;
  s.status = status; s.n_tok = 0; s.path_frames = 0;
  if (a.mode & kModeInit) { s.frame = -1; s.lat_used = 0; }
  if (a.mode & kModeFinal) { a.nwords[io] = 0; a.cost[io] = INFINITY; a.flags[io] = status | WFST_FLAG_DEAD; }
}
// What the first workgroup of a cluster that has broken up leaves behind: a report for its entry (ch; -1:
// it has none), and, if the other clusters that have started have gone the same way, for the entries left.
__device__ __forceinline__ void give_up2(const DevChannels &c, const LaunchArgs &a, const ClusterArgs &w, int ch, int io) {
  if (threadIdx.x != 0) return;
  if (ch >= 0) report_lost(c, a, ch, io);
  int *const n_started = a.lists + 4 * a.n_jobs + 1, *const n_gone = a.lists + 6 * a.n_jobs + 2 + kXcds;
  const int gone = atomicAdd(n_gone, 1) + 1;
  if (gone < min(__hip_atomic_load(n_started, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), w.n_clusters)) return;
  for (int j; (j = atomicAdd(a.lists + 4 * a.n_jobs, 1)) < a.n_jobs;) report_lost(c, a, a.lists[j], a.lists[2 * a.n_jobs + j]);
}

// ------------------------------------------------------------------ the channel kernel
// kCl: clusters of up to w.G workgroups per channel; without it a workgroup is on its own and all of
// its data are the channel's.  kBoost: some channel of the launch has a boosting table or acceptor.  kProf: the phases
// are timed (a debug hook).  kOpt: the decoder has one of its options on (cost offsets, token records
// for lattices, a recycled arena, frame digests).  kQueue: workgroups (clusters always) take more than one entry
// of the launch's list.  Every one of these costs the frame loop a percent or two when it is a
// run-time test.
template <bool kCl, bool kBoost, bool kProf, bool kOpt, bool kQueue>
__global__ __launch_bounds__(kBlock, WFST_MIN_WAVES) void wfst_channel_kernel2(DevGraph g, DevChannels c_arg, LaunchArgs a, ClusterArgs w) {
  __shared__ Smem2 sm;
  const int tid = lane_id();
  DevChannels c = c_arg;
  if (!kOpt) {                                 // (the host launches this instance only when all of these are off)
    c.cost_offset = 0; c.recycle = 0; c.tokrec = nullptr; c.frame_best = nullptr; c.dig_sum = nullptr; c.dig_cnt = nullptr;
  }
  Cx x{g, c, w, sm};
  int job = blockIdx.x;
  x.G = 1; x.lg = 0; x.me = 0; x.xc = 0; x.hc = 0;
  if (kCl) {
    // Clusters are formed on every XCD from the workgroups that start there, in the order in which they
    // start, and nobody waits for one that has not started: the first of a cluster waits a
    // fixed time for the others and goes on with those that are there (a power of two); who comes
    // later, or is not needed, ends.  The launch has as many workgroups on every XCD as the fullest
    // XCD needs; clusters without a ticket end.
    const int xcd = (int)__builtin_amdgcn_s_getreg(kHwXccId) & (kXcds - 1);
    const int cap = (int)gridDim.x / kXcds;      // workgroups per XCD: a multiple of w.G
    if (tid == 0) { sm.job = atomicAdd(a.lists + 6 * a.n_jobs + 2 + xcd, 1); sm.polls = w.polls; sm.dead = 0; }
    __syncthreads();
    const int arrival = uni(sm.job);
    if (arrival >= cap) return;
    const int slot = xcd * cap + arrival, s0 = xcd * cap + arrival / w.G * w.G;
    x.me = slot - s0;
    unsigned long long *box = w.box + (size_t)slot * 2 * kBoxWords;
    for (int i = tid; i < 2 * kBoxWords; i += kBlock) astore(box + i, 0ull);
    stores_done();
    __syncthreads();
    if (tid == 0) {
      if (x.me == 0) {
        const int ticket = atomicAdd(a.lists + 4 * a.n_jobs + 1, 1);
        int eff = 0;
        if (ticket < w.n_clusters) {
          const long long t0 = (long long)wall_clock64();
          int n = 1;
          while (n < w.G) {
            if ((unsigned)(aload(w.hello + 2 * (size_t)(s0 + n)) >> 32) == w.seq) ++n;
            else if ((long long)wall_clock64() - t0 > (long long)w.ticks) break;
          }
          for (eff = 1; 2 * eff <= n;) eff *= 2;
        }
        sm.job = eff | ticket << 4;
        astore(w.hello + 2 * (size_t)s0 + 1, u64_of(sm.job, (int)w.seq));
      } else {
        astore(w.hello + 2 * (size_t)slot, u64_of(1, (int)w.seq));
        sm.job = (int)poll_word(sm, w.hello + 2 * (size_t)s0 + 1, w.seq, kPolls);
      }
    }
    __syncthreads();
    x.G = uni(sm.job) & 15;
    if (x.me >= x.G) return;
    const size_t first = (size_t)(uni(sm.job) >> 4) * w.G;      // the cluster's place in the work memory
    x.lg = 31 - __clz(x.G);
    x.seg_stride = (size_t)w.G * w.seg_cap;
    x.seg_cap = w.seg_cap * (w.G / x.G);
    x.box0 = w.box + (size_t)s0 * 2 * kBoxWords;
    x.cand = w.cand + first * 2 * x.seg_stride;
    x.tq = w.tok + (first + x.me) * 2 * c.qcap;
    x.gi = w.gi + (first + x.me) * 2 * c.qcap;
    x.wl0 = w.wl + (first + x.me) * 2 * c.qcap;
    job = next_job2<kCl>(x, a);
    if (x.me == 0 && uni(sm.dead)) give_up2(c, a, w, -1, 0);
    if (job >= a.n_jobs) return;
  }
  for (;;) {
  const int ch = uni(a.lists[job]);
  const int nfr = uni(a.lists[a.n_jobs + job]), io = uni(a.lists[2 * a.n_jobs + job]);
  x.lat_cap = uni((unsigned)a.lists[3 * a.n_jobs + job]);
  x.lat = c.lattice + uni64(reinterpret_cast<const unsigned long long *>(a.lists + 4 * a.n_jobs + 2)[job]);
  x.q0 = c.queue + (size_t)ch * 2 * c.qcap;
  x.win = c.win + (size_t)ch * c.win_cap; x.win_cap = c.win_cap;
  if (kCl) {
    // recombined tokens that do not fit registers: a part of the channel's own buffers each
    if (x.G == 8 && x.me >= 4) { x.win = c.cand + (size_t)ch * c.cand_cap + (size_t)(x.me - 4) * c.region_cap; x.win_cap = c.region_cap; }
    else { x.win_cap = x.G == 8 ? c.region_cap : c.win_cap / x.G; x.win += (size_t)x.me * x.win_cap; }
  } else {
    x.cand = c.cand + (size_t)ch * c.cand_cap;
    x.tq = x.q0; x.gi = nullptr;
    x.wl0 = c.wl + (size_t)ch * 2 * c.qcap;
  }
  x.frame_off = c.frame_off + (size_t)ch * (c.max_frames + 2);
  x.dig_sum = c.dig_sum ? c.dig_sum + (size_t)ch * (c.max_frames + 1) : nullptr;
  x.dig_cnt = c.dig_cnt ? c.dig_cnt + (size_t)ch * (c.max_frames + 1) : nullptr;
  const bool leader = !kCl || x.me == 0;
  x.s = c.st[ch];
  x.s.frame = uni(x.s.frame); x.s.n_tok = uni(x.s.n_tok); x.s.cur = uni(x.s.cur); x.s.status = uni(x.s.status);
  x.s.lat_used = uni(x.s.lat_used); x.s.max_active = uni(x.s.max_active); x.s.beam = uni(x.s.beam);
  x.s.scale = uni(x.s.scale); x.s.sel_ratio = uni(x.s.sel_ratio); x.s.offset = uni(x.s.offset);
  x.s.boost_n = uni(x.s.boost_n); x.s.boost_states = uni(x.s.boost_states); x.s.lat_epoch = uni(x.s.lat_epoch);
  x.s.path_frames = uni(x.s.path_frames);
  if (kBoost && x.s.boost_n > 0)
    for (int i = tid; i < kBoostSlots; i += kBlock) {
      sm.bk[i] = c.boost_keys[(size_t)ch * kBoostSlots + i];
      sm.bv[i] = c.boost_vals[(size_t)ch * kBoostSlots + i];
      sm.bft[i] = c.boost_from_to[(size_t)ch * kBoostSlots + i];
    }
  if (tid == 0) {
    sm.best_ord = kOrdNone; sm.min_simple = kOrdNone; sm.x_minsimple = kOrdNone;
    sm.n_hub = 0; sm.made[0] = 0; sm.made[1] = 0; sm.n_loc = 0; sm.made[2] = 0; sm.made[3] = 0; sm.n_win = 0;
    sm.more = 0; sm.status_before = 0; sm.n_eseg = 0; sm.x_before = 0;
    sm.map_bad = 0; sm.status = 0; sm.x_status = 0; sm.overfull = 0; sm.redo = 0; sm.n_emit = 0; sm.n_emit_all = 0; sm.x_made = 0;
    if (!kCl) sm.dead = 0;
    for (int r = 0; r < kMaxG; ++r) sm.n_seg[r] = 0;
    for (int i = 0; i < 16; ++i) sm.prof[i] = 0;
    for (int i = 0; i < 8; ++i) sm.ctr[i] = 0;
    sm.prof_t0 = (long long)wall_clock64();
  }
  if (tid < 256) sm.hist[tid] = 0;
  __syncthreads();

  // the buffers of the current set and of the one under construction
  int cur = kCl ? 0 : x.s.cur;
  bool stop = false, open = false;               // open: the newest set's size is still to come
  x.n = 0; x.n_front = 0; x.n_emit = 0;
  if (kOpt && x.dig_sum && leader)               // the workgroups of a cluster add their parts of a digest
    for (int f = (a.mode & kModeInit ? 0 : x.s.frame + 1) + tid; f <= min(c.max_frames, (a.mode & kModeInit ? 0 : x.s.frame) + nfr); f += kBlock)
      __hip_atomic_store(&x.dig_sum[f], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (kOpt) stores_done();
  if (a.mode & kModeInit) {
    x.s.frame = -1; x.s.n_tok = 0; x.s.cur = 1; x.s.status = 0; x.s.lat_used = 0; x.s.offset = 0.0; x.s.path_frames = 0;
    x.s.lat_epoch = 0;
    x.s.beam = a.beam; x.s.scale = a.scale; x.s.max_active = a.max_active; x.s.sel_ratio = 1.5f;
    if (!kCl) cur = 1;
  } else if (x.s.n_tok > 0) {
    // the channel's token set as the last launch left it; a cluster shares it out by owner
    const int2 *q = x.q0 + (size_t)x.s.cur * c.qcap;
    unsigned ms = kOrdNone;
    for (int i0 = 0; i0 < x.s.n_tok; i0 += kBlock) {
      const int i = i0 + tid;
      int2 t = make_int2(0, 0);
      if (i < x.s.n_tok) t = q[i];
      int own[1] = {(int)(i < x.s.n_tok)}, li[1];
      if (kCl) {
        own[0] &= (int)(part_of(key_of(t.x), x.lg) == x.me);
        wave_alloc_n<1>(&sm.n_loc, own, li);
        if (own[0]) { x.tq[li[0]] = t; x.gi[li[0]] = i; }
      }
      if (own[0] && ((unsigned)t.x & kFlagSimple)) ms = min(ms, f2ord(__int_as_float(t.y)));
    }
    if (ms != kOrdNone) atomicMin(&sm.x_minsimple, ms);
    __syncthreads();
    x.n = kCl ? uni(sm.n_loc) : x.s.n_tok;
  }

  // A frame's row, two classes per lane, is loaded while the frame before waits for the sizes of its segments, and kept as it
  // is in memory until it is needed: what is converted (or negated) at once is waited for at once.
  const long long ll0 = (long long)io * a.ll_stride;
  auto load_row = [&](int t, int v, unsigned &raw) {
    const long long at = ll0 + (long long)t * a.V;
    if (a.ll_dtype == WFST_LOGLIKE_F32) raw = (static_cast<const unsigned *>(a.ll) + at)[v];
    else raw = (static_cast<const unsigned short *>(a.ll) + at)[v];
  };
  auto row_cost = [&](unsigned raw) -> float {       // 16-bit rows are widened exactly
    if (a.ll_dtype == WFST_LOGLIKE_F32) return -__uint_as_float(raw);
    if (a.ll_dtype == WFST_LOGLIKE_F16) return -(float)__builtin_bit_cast(_Float16, (unsigned short)raw);
    return -__uint_as_float(raw << 16);
  };
  static_assert(kMaxV <= 2 * kBlock, "two classes per lane");
  unsigned row0 = 0, row1 = 0;
  if (nfr > 0) {
    const int v = lane_id();
    if (v < a.V) load_row(0, v, row0);
    if (v + kBlock < a.V) load_row(0, v + kBlock, row1);
  }
  // (step -1 of an initialisation makes the start token's set)
  for (int t = a.mode & kModeInit ? -1 : 0; t < nfr; ++t) {
    if (stop || x.s.status) break;
    if (t >= 0 && x.s.frame >= c.max_frames && !c.recycle) { if (tid == 0) atomicOr(&sm.x_status, kStCapacity); break; }
    if (t >= 0) {
      const int vs = g.simple_il - 1;          // the class of the simple states' self-loop
      if (tid < a.V) sm.u.e.ac[tid] = row_cost(row0);
      if (tid + kBlock < a.V) sm.u.e.ac[tid + kBlock] = row_cost(row1);
      if (tid == (vs & (kBlock - 1))) {
        const float ac = row_cost(vs < kBlock ? row0 : row1);
        sm.stay_ac = ac;
        // the best of the simple states' candidates: costs are added monotonically (the cluster's, as far as the last
        // exchange told, and the workgroup's own)
        const unsigned ms = min(sm.x_minsimple, sm.min_simple);
        sm.x_minsimple = kOrdNone; sm.min_simple = kOrdNone;
        const float nc = ms == kOrdNone ? INFINITY : canon((ord2f(ms) + g.simple_w) + ac);
        sm.best_ord = nc < INFINITY ? f2ord(nc) : kOrdNone;
      }
    }
    for (int h = tid; h < kHubCap; h += kBlock) { sm.u.e.hub.ready[h] = 0; sm.u.e.hub.seg_next[h] = 0; }
    if (kCl && tid < 256) { sm.v.s.all[tid] = 0; sm.v.s.before[tid] = 0; }
    for (int h = tid; h <= (x.n >> 5); h += kBlock) sm.v.s.hasstay[h & (kQueueMax / 32 - 1)] = 0u;
    if (tid == kResetTid) {
      sm.next_run = kWaves; sm.done_waves = 0; sm.n_hub = 0; sm.status_before = sm.status; sm.earc_before = sm.ctr[kCtEarc];
      sm.made[0] = 0; sm.made[1] = 0; sm.made[2] = 0; sm.made[3] = 0; sm.map_bad = 0; sm.n_win = 0; sm.overfull = 0;
      count2(sm, kCtTok, x.n);
      if (leader && t >= 0) count2(sm, kCtFrames, 1);
    }
    const int2 *Q = x.tq + (size_t)cur * c.qcap; int2 *NQ = x.tq + (size_t)(cur ^ 1) * c.qcap;
    const int *GI = x.gi + (size_t)cur * c.qcap; int *NGI = x.gi + (size_t)(cur ^ 1) * c.qcap;
    const Run run = load_run<kCl>(x, Q, GI, uni(tid >> 6), run_size(x));     // (ahead of the barrier)
    __syncthreads();
    mark<kProf>(x, kPhOther);
    Cutoff cut;
    if (t >= 0) {
      expand2<kCl, kBoost>(x, Q, GI, run);
      if (kCl) stores_done();
      __syncthreads();
      mark<kProf>(x, kPhExpSetup);
      post_sizes<kCl>(x);
      clear_table(sm);
      if (t + 1 < nfr) {
        const int v = lane_id();
        if (v < a.V) load_row(t + 1, v, row0);
        if (v + kBlock < a.V) load_row(t + 1, v + kBlock, row1);
      }
      take_sizes<kCl>(x);
      asm volatile("" : "+v"(row0), "+v"(row1));   // (waited for here, where it has come: later it would be with the stores in between)
      mark<kProf>(x, kPhExpand);
      if (open) {                                // the last frame's set, and an overflow of its last round
        const int before = uni(sm.x_before);
        publish2<kCl, kOpt>(x, before != 0);
        open = false;
        if (__builtin_expect(before, 0)) {       // it has no digest, and what was expanded from it does not count
          __syncthreads();
          if (tid == 0) { sm.x_status = before; sm.ctr[kCtEarc] = sm.earc_before; count2(sm, kCtTok, -x.n); if (leader) count2(sm, kCtFrames, -1); }
          if (kOpt && x.dig_sum && leader && tid == 0 && x.s.frame <= c.max_frames)
            __hip_atomic_store(&x.dig_sum[x.s.frame], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          break;
        }
      }
    } else {
      clear_table(sm);
      if (tid == 0) sm.x_best = kOrdNone;
      __syncthreads();
    }
    // a recycled arena is a ring over whole frames: a frame's tokens (at most qcap) never straddle
    // its end, the write position goes back to the start instead and the epoch counts that
    if (c.recycle && x.s.lat_used + (unsigned)c.qcap > x.lat_cap) { x.s.lat_used = 0; x.s.lat_epoch++; }
    const unsigned lat_base = x.s.lat_used;
    prune2<kCl, kProf, kOpt>(x, Q, GI, NQ, NGI, lat_base, cut, t < 0);
    const bool last = t + 1 >= nfr || (x.s.frame + 1 >= c.max_frames && !c.recycle);
    open = closure2<kCl, kBoost, kProf>(x, NQ, NGI, lat_base, cut, last);
    x.s.frame++;
    cur ^= 1;
    // (one wait for all of these; the workgroup's own status is final behind the closure's last barrier)
    const int n_loc = sm.n_loc, own = sm.status, of_cluster = sm.x_status, is_dead = sm.dead;
    if (!kCl && tid == 0) sm.x_status = own;
    const bool bad = uni(own) != 0, gone = kCl && uni(is_dead) != 0;
    stop = gone || (kCl ? !open && uni(of_cluster) != 0 : bad);
    finish2<kCl, kOpt>(x, NQ, NGI, uni(n_loc), lat_base, stop || bad);
    // If the set's size is still to come, the cluster learns of an overflow with it, behind ExpandArcs of the next
    // frame: until then the workgroup has the tokens of the emitting step, all of them written, and none to expand.
    if (kCl && bad) { x.n_front = 0; x.n = x.n_emit; }
    if (!open) publish2<kCl, kOpt>(x, stop);
    mark<kProf>(x, kPhFinish);
    if (gone) break;
  }
  __syncthreads();
  if (kCl && uni(sm.dead)) { if (tid == 0) sm.x_status |= kStCapacity; __syncthreads(); }
  if (uni(sm.x_status)) {     // overflow: the channel stops with an empty token set
    x.s.status |= uni(sm.x_status);
    x.s.n_tok = 0; x.n = 0;
  }
  {
    const int2 *Q = x.tq + (size_t)cur * c.qcap; const int *GI = x.gi + (size_t)cur * c.qcap;
    if (kCl)                                     // the set goes back to the channel's queue
      for (int i = tid; i < x.n; i += kBlock) x.q0[(size_t)x.s.cur * c.qcap + GI[i]] = Q[i];
    mark<kProf>(x, kPhOther);
    if (a.mode & kModeFinal) {
      // The traceback works on copies of the context, so that the pointers of the frame loop above
      // never live in memory on its account (only then does the compiler know they are global and
      // keep them in registers).
      const DevGraph g2 = g; const DevChannels c2 = c; const LaunchArgs a2 = a; const ClusterArgs w2 = w;
      Cx x2{g2, c2, w2, sm};
      x2.lat = x.lat; x2.frame_off = x.frame_off; x2.s = x.s; x2.lat_cap = x.lat_cap; x2.n = x.n;
      x2.G = x.G; x2.lg = x.lg; x2.me = x.me; x2.xc = x.xc; x2.box0 = x.box0;
      if (tid == 0) sm.path_frames = x.s.path_frames;
      __syncthreads();
      trace2<kCl>(x2, a2, io, Q, GI);
      x.xc = x2.xc;
      __syncthreads();
      x.s.path_frames = uni(sm.path_frames);
    }
  }
  mark<kProf>(x, kPhTrace);
  if (tid == 0) {
    if (leader) {
      c.st[ch] = x.s;
      for (int i = 0; i < 16; ++i) if (sm.prof[i]) atomicAdd((unsigned long long *)&c.counters[8 + i], (unsigned long long)sm.prof[i]);
    }
    for (int i = 0; i < 8; ++i) if (sm.ctr[i]) atomicAdd((unsigned long long *)&c.counters[i], (unsigned long long)sm.ctr[i]);
  }
  if (!kCl && !kQueue) break;
  job = next_job2<kCl>(x, a);  // (also: nobody is still reading this channel's tables when the next one's are set up)
  if (kCl && x.me == 0 && uni(sm.dead)) give_up2(c, a, w, ch, io);
  if (job >= a.n_jobs) break;
  }
}
