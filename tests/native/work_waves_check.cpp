// host-only check of build_work_waves over random layouts: every sub-block of every tile belongs to
// exactly one wavefront of the launch that carries its parameter group, runs name the wavefronts of
// one parameter tile, or of one chunk's RAW tiles, that share a workgroup, launches begin at workgroups; and of
// build_step_tickets on the same lists
#include "layout.hpp"
#include <algorithm>
#include <cstdio>
#include <random>
using namespace ffsnap;

// The tickets of a step in one launch: every contribution to a chunk's checksum has a bit of its own in a word of the
// chunk's, the words know when they are full, and summed up in any order they deliver every chunk once, with the sum
// of its contributions, and are zero again.  refused: a chunk has more contributions than the words take.
static const char* check_tickets(const std::vector<WorkTile>& tiles, const std::vector<WorkWave>& waves, uint64_t n_chunks, std::mt19937_64& rng, bool& refused){
  struct Contribution { uint32_t chunk; StepTicket t; };
  std::vector<StepTicket> runs, heads;
  uint64_t words=0;
  refused = !build_step_tickets(tiles, waves, n_chunks, runs, heads, words);
  // who contributes, from the lists alone: the last wavefront of a run for each stream (for all, if they are in one
  // chunk), and the halves of split elements
  std::vector<Contribution> all;
  std::vector<uint32_t> count(n_chunks, 0);
  for(size_t i=0;i<waves.size();i++){
    if(waves[i].tile==kNoTile) continue;
    const size_t begin = i/kWavesPerGroup*kWavesPerGroup + (waves[i].info>>4&7);
    const uint32_t len = waves[i].info>>8&15;
    if(i != begin+len-1) continue;
    const WorkTile& t=tiles[waves[i].tile];
    bool one = true;
    for(int x=1;x<4 && t.kind==kWorkParam;x++) one = one && t.chunk[x]==t.chunk[0];
    for(int x=0;x<(one?1:4);x++){ all.push_back({t.chunk[x], refused ? StepTicket{} : runs[4*begin+x]}); count[t.chunk[x]]++; }
  }
  for(size_t i=0;i<tiles.size();i++)
    for(int x=1;x<4;x++)
      if(tiles[i].kind==kWorkParam && (tiles[i].head_split>>x&1)){ all.push_back({tiles[i].chunk[3+x], refused ? StepTicket{} : heads[3*i+x-1]}); count[tiles[i].chunk[3+x]]++; }
  const uint32_t most = *std::max_element(count.begin(), count.end());
  if(refused != (most > 1024)) return "refused";
  if(refused) return nullptr;
  for(uint64_t c=0;c<n_chunks;c++) if(!count[c]) return "chunk without contributions";
  struct Word { uint64_t chunk=~0ull; uint32_t bits=0, full=0; };
  std::vector<Word> seen(words);
  auto take=[&](uint32_t word, uint32_t chunk, uint32_t bit, bool shared) -> bool {
    if(word>=words || (seen[word].chunk!=~0ull && seen[word].chunk!=chunk)) return false;
    if(!shared && (seen[word].bits>>bit&1)) return false;
    seen[word].chunk=chunk; seen[word].bits|=1u<<bit;
    return true;
  };
  for(const Contribution& k: all){
    const uint32_t leaves=k.t.bits>>8&63;
    if(leaves != (count[k.chunk]+31)/32) return "leaves";
    if(!take(k.t.leaf, k.chunk, k.t.bits&31, false)) return "leaf bit";
    if(seen[k.t.leaf].full && seen[k.t.leaf].full!=k.t.leaf_full) return "leaf full";
    seen[k.t.leaf].full=k.t.leaf_full;
    if(leaves>1){
      if(!take(k.t.root, k.chunk, k.t.bits>>16&31, true) || k.t.root==k.t.leaf) return "root bit";
      seen[k.t.root].full = leaves==32 ? 0xFFFFFFFFu : (1u<<leaves)-1;
    }
  }
  for(const Word& w: seen) if(w.bits!=w.full) return "a word that fills too early or never";
  std::vector<uint64_t> tally(words, 0);
  std::vector<uint32_t> want(n_chunks, 0), got(n_chunks, 0), delivered(n_chunks, 0);
  std::shuffle(all.begin(), all.end(), rng);
  for(const Contribution& k: all){
    const uint32_t v=rng();
    want[k.chunk]^=v;
    uint64_t now = tally[k.t.leaf]^=uint64_t(1u<<(k.t.bits&31))<<32|v;
    if(now>>32 != k.t.leaf_full) continue;
    tally[k.t.leaf]=0;
    const uint32_t leaves=k.t.bits>>8&63;
    if(leaves>1){
      now = tally[k.t.root]^=uint64_t(1u<<(k.t.bits>>16&31))<<32|uint32_t(now);
      if(now>>32 != (leaves==32 ? 0xFFFFFFFFu : (1u<<leaves)-1)) continue;
      tally[k.t.root]=0;
    }
    got[k.chunk]=uint32_t(now);
    delivered[k.chunk]++;
  }
  for(uint64_t c=0;c<n_chunks;c++) if(delivered[c]!=1 || got[c]!=want[c]) return "delivery";
  for(uint64_t w: tally) if(w) return "a word that is left";
  return nullptr;
}

int main(){
  std::mt19937_64 rng(2);
  // so many contributions to one chunk: a parameter whose workgroups are whole, alone or with a tensor that is only copied
  for(uint64_t n: {1, 2, 31, 32, 33, 63, 64, 65, 1023, 1024, 1025})
    for(bool raw: {false, true}){
      const uint64_t ne=(n-raw)*kWavesPerGroup*kSubElems;
      std::vector<ff_segment> segs;
      if(raw) segs.push_back({(void*)4096, 1000, FF_BF16, FF_KIND_RAW, 0, 0});
      for(uint32_t k=FF_KIND_W16;k<=FF_KIND_V;k++)
        if(ne) segs.push_back({(void*)4096, (k==FF_KIND_W16?2:4)*ne, k==FF_KIND_W16?FF_BF16:FF_F32, k, 0, 0});
      Layout L;
      if(build_layout(segs.data(), segs.size(), 1<<26, 0, L)!=FF_OK){ printf("layout\n"); return 1; }
      std::vector<WorkTile> tiles; build_work_tiles(L,tiles);
      std::vector<WorkWave> w; std::vector<uint32_t> begin;
      bool refused=false;
      if(!build_work_waves(tiles, std::max<size_t>(L.params.size(),1), 2048, w, begin)){ printf("waves\n"); return 1; }
      const char* wrong=check_tickets(tiles, w, L.n_chunks, rng, refused);
      if(wrong || refused!=(n>1024)){ printf("tickets of %llu: %s\n", (unsigned long long)n, wrong?wrong:"refused"); return 1; }
    }
  static char arena[1<<16];
  for(int it=0; it<2000; it++){
    std::vector<ff_segment> segs;
    const uint64_t chunk = 1024ull << (rng()%14);
    const uint32_t per_launch = 1 + rng()%5;
    const int np = 1 + rng()%12;
    for(int p=0;p<np;p++){
      const uint64_t ne = rng()%3==0 ? 1 + rng()%5 : 1 + rng()%40000;
      segs.push_back({arena+2, 2*ne, FF_BF16, FF_KIND_W16, (uint32_t)p, 0});
      for(uint32_t k=FF_KIND_MASTER;k<=FF_KIND_V;k++) segs.push_back({arena+4, 4*ne, FF_F32, k, (uint32_t)p, 0});
      if(rng()%3==0) segs.push_back({arena+2, 2*(rng()%60000), FF_BF16, FF_KIND_RAW, 0, 0});
      for(uint64_t k=rng()%30; k-- && rng()%8;) segs.push_back({arena+2, 2*(1+rng()%3000), FF_BF16, FF_KIND_RAW, 0, 0});
    }
    Layout L;
    if(build_layout(segs.data(), segs.size(), chunk, 0, L)!=FF_OK) continue;
    std::vector<WorkTile> tiles; build_work_tiles(L,tiles);
    std::vector<WorkWave> w; std::vector<uint32_t> begin;
    if(!build_work_waves(tiles, L.params.size(), per_launch, w, begin)){ printf("refused\n"); return 1; }
    { // the limit is on the entries themselves, whatever their number for each tile
      std::vector<WorkWave> w2; std::vector<uint32_t> begin2;
      if(!build_work_waves(tiles, L.params.size(), per_launch, w2, begin2, w.size()) || begin2!=begin ||
         build_work_waves(tiles, L.params.size(), per_launch, w2, begin2, w.size()-1)){ printf("limit\n"); return 1; }
    }
    {
      bool refused;
      if(const char* wrong=check_tickets(tiles, w, L.n_chunks, rng, refused)){ printf("tickets: %s\n", wrong); return 1; }
    }
    const uint64_t launches = (L.params.size()+per_launch-1)/per_launch;
    if(begin.size()!=launches+1 || begin[0]!=0 || begin.back()!=w.size()){ printf("launches\n"); return 1; }
    std::vector<uint32_t> seen(tiles.size(), 0);
    for(uint64_t k=0;k<launches;k++){
      if(begin[k]%kWavesPerGroup || begin[k]>begin[k+1]){ printf("launch begin\n"); return 1; }
      for(uint32_t i=begin[k];i<begin[k+1];i++){
        if(w[i].tile==kNoTile) continue;
        const WorkTile& t=tiles[w[i].tile];
        if(t.kind==kWorkParam ? t.grad_index/per_launch!=k : k+1!=launches){ printf("launch of a tile\n"); return 1; }
        // the place of its gradient among the launch's (a RAW tile has none)
        if(w[i].info>>16 != (t.kind==kWorkParam ? t.grad_index-k*per_launch : 0)){ printf("group\n"); return 1; }
        const uint32_t sub=w[i].info&15, first=(w[i].info>>4)&7, len=(w[i].info>>8)&15;
        if(seen[w[i].tile]&(1u<<sub)){ printf("twice\n"); return 1; }
        seen[w[i].tile]|=1u<<sub;
        const uint32_t slot=i%kWavesPerGroup, base=i-slot;
        if(slot<first || slot>=first+len || first+len>kWavesPerGroup){ printf("run place\n"); return 1; }
        for(uint32_t s=0;s<kWavesPerGroup;s++){
          const bool in = s>=first && s<first+len;
          const uint32_t o=w[base+s].tile;
          // RAW tiles of one chunk share a run, they are neighbours in the stream
          const bool mates = o==w[i].tile || (o!=kNoTile && t.kind==kWorkRaw && tiles[o].kind==kWorkRaw && tiles[o].chunk[0]==t.chunk[0]);
          if(in != mates){ printf("run members\n"); return 1; }
          if(in && ((w[base+s].info>>4)!=(w[i].info>>4))){ printf("run of a mate\n"); return 1; }
        }
      }
    }
    for(size_t i=0;i<tiles.size();i++){
      const WorkTile& t=tiles[i];
      const bool par=t.kind==kWorkParam;
      const uint64_t a = par ? t.e0%kParamTileElems : t.soff[0]%kRawTileBytes, size = par ? kSubElems : kSubRawBytes;
      if(t.n==0 || a+t.n > (par?kParamTileElems:kRawTileBytes)){ printf("block\n"); return 1; }
      uint32_t want=0;
      for(uint64_t s=a/size; s<=(a+t.n-1)/size; s++) want|=1u<<s;
      if(seen[i]!=want){ printf("cover %zu\n",i); return 1; }
    }
  }
  printf("ok\n"); return 0;
}
